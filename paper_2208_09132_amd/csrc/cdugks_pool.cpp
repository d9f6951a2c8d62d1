// Device memory of contexts and batch tables: blocks released by one object
// are handed to the next.
//
// Freeing device memory waits until the driver has cleared it, which takes
// about 29 ms per GB once a process has cycled through the card's memory: a
// refit of a 128^2 x 28^2 problem that took 3.4 ms spent 29 ms more in the
// release of its 1.1 GB context, and the server pays the same per request.
//
// Per device, idle blocks are kept while the library has a live context or
// server there, up to 1/32 of the device's memory in all, the oldest going
// first; with the last of them (and whenever an allocation fails) everything
// idle is given back.  A block is reused for a request of exactly its size, so
// an object never holds more than it asked for: what fitted the device or a
// server's budget without kept blocks fits with them.  An object releases its block only after waiting for the streams that
// used it, so a block taken here has no work in flight.
#include "cdugks_host.h"

#include <mutex>

namespace cdg {
namespace {

constexpr int MAX_DEVICES = 64;  // beyond these, blocks are never kept
constexpr int MAX_IDLE = 64;     // idle blocks per device

struct Block {
    void* ptr;
    size_t bytes;
};
// fixed size, so nothing here allocates host memory (or throws)
struct DevicePool {
    Block idle[MAX_IDLE];  // oldest first
    int count;
    size_t held;           // bytes of the idle blocks
    size_t limit;
    long long users;
    bool known;
};
struct Pools {
    std::mutex mu;
    // held while idle blocks are freed, so that a thread that finds nothing
    // left to free has waited for what others were freeing; taken before mu
    std::mutex freeing;
    DevicePool dev[MAX_DEVICES];
};
// constant-initialised and without a destructor to run: usable whatever order
// the process's other objects go in
Pools g_pools;

DevicePool* pool_of(int d) {
    if (d < 0 || d >= MAX_DEVICES) return nullptr;
    DevicePool& p = g_pools.dev[d];
    if (!p.known) {
        hipDeviceProp_t prop;
        if (hipGetDeviceProperties(&prop, d) == hipSuccess) p.limit = prop.totalGlobalMem / 32;
        else (void)hipGetLastError();
        p.known = true;
    }
    return &p;
}

Block remove(DevicePool& p, int k) {
    const Block b = p.idle[k];
    p.held -= b.bytes;
    --p.count;
    for (int j = k; j < p.count; ++j) p.idle[j] = p.idle[j + 1];
    return b;
}

// Free idle blocks, oldest first, until at most `keep` bytes and `most`
// blocks are left; false if there was nothing to free.
bool cut(int device, size_t keep, int most = MAX_IDLE) {
    Block drop[MAX_IDLE];
    int n = 0;
    std::lock_guard<std::mutex> free_lock(g_pools.freeing);
    {
        std::lock_guard<std::mutex> lock(g_pools.mu);
        DevicePool* p = pool_of(device);
        while (p && p->count > 0 && (p->held > keep || p->count > most)) drop[n++] = remove(*p, 0);
    }
    // outside mu: a free waits for the device
    for (int k = 0; k < n; ++k) (void)hipFree(drop[k].ptr);
    return n > 0;
}

}  // namespace

hipError_t pool_take(int device, size_t bytes, size_t keep, void** ptr) {
    void* found = nullptr;
    {
        std::lock_guard<std::mutex> lock(g_pools.mu);
        DevicePool* p = pool_of(device);
        for (int k = 0; p && !found && k < p->count; ++k)
            if (p->idle[k].bytes == bytes) found = remove(*p, k).ptr;
    }
    if (keep != SIZE_MAX) cut(device, keep);
    if (found) {
        *ptr = found;
        return hipSuccess;
    }
    hipError_t e = hipMalloc(ptr, bytes);
    // idle blocks, of this thread's freeing or another's, may have been in the
    // way; again while there were any
    for (bool freed = true; e != hipSuccess && freed;) {
        (void)hipGetLastError();
        freed = cut(device, 0);
        e = hipMalloc(ptr, bytes);
    }
    return e;
}

void pool_give(int device, void* ptr, size_t bytes) {
    if (!ptr) return;
    size_t keep = 0;
    {
        std::lock_guard<std::mutex> lock(g_pools.mu);
        DevicePool* p = pool_of(device);
        if (p && p->users > 0 && bytes <= p->limit) keep = p->limit - bytes + 1;
    }
    if (keep > 0) {
        cut(device, keep - 1, MAX_IDLE - 1);
        std::lock_guard<std::mutex> lock(g_pools.mu);
        DevicePool* p = pool_of(device);
        // another thread may have filled the room just made
        if (p->users > 0 && p->count < MAX_IDLE && p->held + bytes <= p->limit) {
            p->idle[p->count++] = Block{ptr, bytes};
            p->held += bytes;
            return;
        }
    }
    (void)hipFree(ptr);
}

void pool_user(int device, int change) {
    bool last = false;
    {
        std::lock_guard<std::mutex> lock(g_pools.mu);
        DevicePool* p = pool_of(device);
        if (!p) return;
        p->users += change;
        last = p->users <= 0;
    }
    if (last) cut(device, 0);
}

}  // namespace cdg
