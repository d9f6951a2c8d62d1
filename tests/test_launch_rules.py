"""Launch rules of the library's host side, asked of the built library without
a GPU: a small program includes the library's internal header, links the
library and prints what a rule answers."""
import os
import shutil
import subprocess

import pytest

from paper_2208_09132_amd import cdugks as cd
from tests.conftest import ROOT

CSRC = os.path.join(ROOT, "paper_2208_09132_amd", "csrc")
INCLUDES = ["-D__HIP_PLATFORM_AMD__", "-isystem", "/opt/rocm/include", "-I", os.path.join(ROOT, "include"), "-I", CSRC]


def build(tmp, source, extra):
    """Compile a host program with g++ and return its path."""
    if shutil.which("g++") is None:
        pytest.skip("no g++")
    src, exe = os.path.join(tmp, "rules.cpp"), os.path.join(tmp, "rules")
    with open(src, "w") as f:
        f.write(source)
    subprocess.run(["g++", "-std=c++17", "-O1", *INCLUDES, src, "-o", exe, *extra], check=True)
    return exe


@pytest.fixture(scope="module")
def lanes(tmp_path_factory):
    exe = build(str(tmp_path_factory.mktemp("rules")), r"""
#include "cdugks_host.h"
#include <cstdio>
#include <cstdlib>
int main(int argc, char** argv) {
    cdg::Resolved r{};
    r.D = atoi(argv[1]);
    for (int d = 0; d < 3; ++d) r.nv[d] = d < r.D ? atoi(argv[2 + d]) : 1;
    for (int k = 2 + r.D; k < argc; ++k) printf("%d ", cdg::close_lanes(r, atoll(argv[k])));
}
""", [cd.LIB_PATH, "-Wl,-rpath," + os.path.dirname(cd.LIB_PATH)])

    def ask(nv, *faces):
        args = [str(len(nv))] + [str(x) for x in (*nv, *faces)]
        out = subprocess.run([exe, *args], check=True, stdout=subprocess.PIPE, text=True).stdout
        return [int(x) for x in out.split()]

    return ask


def test_one_thread_closes_a_face_where_groups_would_queue(lanes):
    # two workgroups of 256 on each of 256 CUs: 8192 groups of 16
    assert lanes([28, 28], 8192, 8193, 131072) == [16, 1, 1]
    # more than 256 nodes: groups of 16 for up to three (1-D) or two (2-D, 3-D)
    # rounds of that, never for any number of faces
    assert lanes([257], 8192, 24576, 24577, 200000, 16000000) == [16, 16, 1, 1, 1]
    assert lanes([129, 129], 16384, 16385, 80000) == [16, 1, 1]
    assert lanes([100, 100, 100], 16384, 16385) == [16, 1]
    assert lanes([16385], 128, 24577) == [256, 1]


def test_streaming_stores(tmp_path):
    exe = build(str(tmp_path), r"""
#include "cdugks_host.h"
#include <cstdio>
#include <cstdlib>
int main(int argc, char** argv) {
    for (int k = 1; k + 3 < argc; k += 4) {
        cdg::Resolved r{};
        r.D = atoi(argv[k]);
        r.storage = atoi(argv[k + 1]);
        r.ne[0] = atoi(argv[k + 2]);
        r.V = atoi(argv[k + 3]);
        printf("%d ", cdg::fv_streams(r) ? 1 : 0);
    }
}
""", [cd.LIB_PATH, "-Wl,-rpath," + os.path.dirname(cd.LIB_PATH)])

    def ask(*problems):
        args = [str(x) for p in problems for x in p]
        return [int(x) for x in
                subprocess.run([exe, *args], check=True, stdout=subprocess.PIPE, text=True).stdout.split()]

    # dimension, storage form, faces of a row, velocities
    assert ask((2, 0, 256, 784), (2, 0, 257, 784), (2, 0, 8, 4)) == [1, 0, 1]
    assert ask((2, 1, 256, 4095), (2, 1, 256, 4096), (2, 1, 257, 4096), (2, 2, 256, 16641)) == [0, 1, 0, 1]
    assert ask((3, 1, 64, 512), (3, 1, 65, 512), (3, 0, 24, 64)) == [1, 0, 1]


@pytest.mark.parametrize("storage, n, bc", [
    ("f64", [31, 2 ** 24], ["outflow", "periodic"]),
    ("f64", [2 ** 15, 2 ** 14], ["periodic", "periodic"]),
    ("f64", [1, 15, 2 ** 24], ["outflow", "outflow", "periodic"]),
    ("f32", [63, 2 ** 24], ["outflow", "periodic"]),
    ("f32", [2 ** 15, 2 ** 15], ["periodic", "periodic"]),
])
def test_velocity_rows_of_4_gb_belong_to_problems_no_device_holds(storage, n, bc):
    # the smallest velocity grid on the fewest cells whose face rows reach 4 GB,
    # the reach of the kernels' 32-bit offsets in a row
    D = len(n)
    p = dict(dim=D, n=n, lo=[0.0] * D, hi=[1.0] * D, bc=bc, nv=[2] * D, vmin=[-5.0] * D, vmax=[5.0] * D,
             relax="tau", tau=1.0, storage=storage)
    assert cd.cdugks_required_bytes(p) > 288 * 2 ** 30
