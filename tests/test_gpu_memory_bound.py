"""Kept device blocks on the device itself: contexts that together pass the
bound of 1/32 of its memory, no two of a size, leave at most that behind, the
last released among it, and a context of a kept size allocates nothing."""
import ctypes

import pytest

from paper_2208_09132_amd import cdugks as cd
from paper_2208_09132_amd import workloads as wl

pytestmark = pytest.mark.gpu

SLACK = 64 << 20


def memory():
    free, total = ctypes.c_size_t(), ctypes.c_size_t()
    assert cd.load_library().hipMemGetInfo(ctypes.byref(free), ctypes.byref(total)) == 0
    return free.value, total.value


def of_bytes(target):
    """A 2-D problem that needs about `target` bytes."""
    def make(n):
        return wl.random_fourier(2, [n, n], [28, 28], wl.SplitMix64(3))
    per_cell = cd.cdugks_required_bytes(make(256)) / 256 ** 2
    p = make(int((target / per_cell) ** 0.5))
    need = cd.cdugks_required_bytes(p)
    assert 0.8 * target < need < 1.2 * target, (need, target)
    return p, need


def test_the_bound_puts_the_oldest_blocks_out():
    cd.Solver(wl.sod(n=16, nv=16)).close()  # library and queues loaded
    free0, total = memory()
    bound = total // 32
    keep = cd.Solver(wl.sod(n=16, nv=16))
    problems = [of_bytes(bound * f) for f in (0.26, 0.30, 0.34, 0.38, 0.42, 0.46)]
    assert sum(need for _, need in problems) > 2 * bound
    for p, need in problems:
        print(f"{need / 2**30:.2f} GiB of {bound / 2**30:.2f}", flush=True)
        cd.Solver(p).close()
        assert free0 - memory()[0] <= bound + SLACK
    # the last two stay, the four before them are gone
    kept = problems[-1][1] + problems[-2][1]
    assert abs((free0 - memory()[0]) - kept) <= SLACK
    again = cd.Solver(problems[-2][0])
    assert abs((free0 - memory()[0]) - kept) <= SLACK
    again.close()
    keep.close()
    assert free0 - memory()[0] <= SLACK
