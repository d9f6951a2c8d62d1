"""The kept device blocks (csrc/cdugks_pool.cpp) without a device: the file is
compiled into a small host program whose hipMalloc and hipFree hand out host
addresses, count, and can be told to run out of memory or to take their time."""
import subprocess

import pytest

from tests.test_launch_rules import build

SOURCE = r"""
#include "cdugks_pool.cpp"

#include <atomic>
#include <chrono>
#include <cstdio>
#include <cstdlib>
#include <map>
#include <string>
#include <thread>
#include <vector>

namespace {
std::mutex mu;
std::map<void*, size_t> live;
size_t used = 0, device = 3200;  // the bound on idle bytes is 1/32 of it: 100
int mallocs = 0, frees = 0, free_ms = 0;
std::atomic<int> freeing{0};
uintptr_t next = 4096;
}  // namespace

extern "C" hipError_t hipMalloc(void** p, size_t bytes) {
    std::lock_guard<std::mutex> lock(mu);
    if (used + bytes > device) return hipErrorOutOfMemory;
    *p = (void*)(next += 4096);
    live[*p] = bytes;
    used += bytes;
    ++mallocs;
    return hipSuccess;
}
extern "C" hipError_t hipFree(void* p) {
    ++freeing;
    if (free_ms) std::this_thread::sleep_for(std::chrono::milliseconds(free_ms));
    std::lock_guard<std::mutex> lock(mu);
    if (!live.count(p)) {
        printf("a block freed twice or never allocated\n");
        exit(1);
    }
    used -= live[p];
    live.erase(p);
    ++frees;
    --freeing;
    return hipSuccess;
}
extern "C" hipError_t hipGetLastError() { return hipSuccess; }
extern "C" hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600* prop, int) {
    prop->totalGlobalMem = device;
    return hipSuccess;
}

#define CHECK(x)                                                    \
    do {                                                            \
        if (!(x)) {                                                 \
            printf("line %d: %s\n", __LINE__, #x);                  \
            exit(1);                                                \
        }                                                           \
    } while (0)

using namespace cdg;

static void* take(size_t bytes, size_t keep = SIZE_MAX) {
    void* p = nullptr;
    return pool_take(0, bytes, keep, &p) == hipSuccess ? p : nullptr;
}

static void exact() {
    void* a = take(50);
    pool_give(0, a, 50);
    CHECK(frees == 0 && used == 50);
    // a smaller and a larger request get blocks of their own
    void *b = take(49), *c = take(51);
    CHECK(b != a && c != a && used == 150);
    CHECK(take(50) == a && mallocs == 3);
}

static void bound() {
    void* p[5];
    for (int k = 0; k < 5; ++k) p[k] = take(30 + k);
    for (int k = 0; k < 5; ++k) pool_give(0, p[k], 30 + k);
    // 30, 31 and 32 fit 100 bytes; 33 and 34 put the oldest out
    CHECK(frees == 2 && used == 32 + 33 + 34);
    CHECK(take(30) != p[0] && take(34) == p[4] && take(33) == p[3]);
    // a block above the bound is never kept, and costs the others nothing
    void* big = take(101);
    pool_give(0, big, 101);
    CHECK(frees == 3 && take(32) == p[2]);
}

static void count() {
    void* p[70];
    for (int k = 0; k < 70; ++k) p[k] = take(100 + k);
    for (int k = 0; k < 70; ++k) pool_give(0, p[k], 100 + k);
    CHECK(frees == 6);
    CHECK(take(106) == p[6] && take(169) == p[69] && take(105) != p[5]);
}

static void last_user() {
    void *a = take(40), *b = take(41);
    pool_give(0, a, 40);
    pool_user(0, 1);
    pool_user(0, -1);
    CHECK(frees == 0);
    pool_user(0, -1);  // the last: everything idle goes
    CHECK(frees == 1 && used == 41);
    pool_give(0, b, 41);  // and nothing is kept without one
    CHECK(frees == 2 && used == 0);
}

static void out_of_memory() {
    void *a = take(60), *b = take(3000);
    pool_give(0, a, 60);
    CHECK(take(200) != nullptr && frees == 1);  // 3060 + 200 > 3200: the idle block makes room
    CHECK(take(200) == nullptr && used == 3200);
    pool_give(0, b, 3000);
    CHECK(take(3000) != nullptr);
}

static void budget() {
    void *a = take(40), *b = take(35), *c = take(20);
    pool_give(0, a, 40);
    pool_give(0, b, 35);
    pool_give(0, c, 20);
    // a budget of 60: the request's own block is taken, not freed and
    // allocated again, and of the rest only what the budget leaves stays
    CHECK(take(40, 60 - 40) == a && mallocs == 3 && frees == 1 && used == 60);
    // nothing that fits: the idle blocks go first
    CHECK(take(50, 10) != nullptr && frees == 2 && used == 90);
}

static void two_threads() {
    void *a = take(100), *b = take(3060);
    CHECK(b != nullptr);
    pool_give(0, a, 100);
    free_ms = 200;
    // the first thread gives the idle block back for its 50 bytes; the second
    // comes while the block is still on its way and there is nothing idle left
    void* p[2] = {nullptr, nullptr};
    std::thread first([&] { p[0] = take(50); });
    while (freeing == 0) std::this_thread::sleep_for(std::chrono::milliseconds(1));
    p[1] = take(50);
    first.join();
    CHECK(p[0] && p[1] && used == 3160);
}

int main(int, char** argv) {
    const std::string what = argv[1];
    if (what == "count") device = 3200000;  // bound 100000 bytes: the number of blocks is what counts
    pool_user(0, 1);
    if (what == "exact") exact();
    else if (what == "bound") bound();
    else if (what == "count") count();
    else if (what == "last_user") last_user();
    else if (what == "out_of_memory") out_of_memory();
    else if (what == "budget") budget();
    else if (what == "two_threads") two_threads();
    else return 2;
    return 0;
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    return build(str(tmp_path_factory.mktemp("pool")), SOURCE, ["-pthread"])


@pytest.mark.parametrize("what", ["exact", "bound", "count", "last_user", "out_of_memory", "budget", "two_threads"])
def test_pool(program, what):
    r = subprocess.run([program, what], stdout=subprocess.PIPE, text=True, timeout=60)
    assert r.returncode == 0, r.stdout
