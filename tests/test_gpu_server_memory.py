"""The server's memory budget with kept device blocks about: requests count with
the bytes they ask for, so a budget of three requests runs three at a time
whatever blocks lie idle, and blocks and requests together stay within it."""
import ctypes
import time

import pytest

from paper_2208_09132_amd import cdugks as cd
from paper_2208_09132_amd import workloads as wl

pytestmark = pytest.mark.gpu

MIB = 1 << 20


def problem(n):
    return wl.random_fourier(2, [n, n], [20, 20], wl.SplitMix64(n), Kn=1e-2)


def free_memory():
    free, total = ctypes.c_size_t(), ctypes.c_size_t()
    assert cd.load_library().hipMemGetInfo(ctypes.byref(free), ctypes.byref(total)) == 0
    return free.value


def poll(srv, ticket, timeout=60.0):
    t0 = time.time()
    while time.time() - t0 < timeout:
        r = srv.poll(ticket)
        if r is not None:
            return r
        time.sleep(0.002)
    raise AssertionError("request still pending")


def test_a_larger_idle_block_leaves_the_budget_to_the_requests():
    p, larger = problem(128), problem(140)
    need, more = cd.cdugks_required_bytes(p), cd.cdugks_required_bytes(larger)
    assert need < more < 1.25 * need
    budget = 3 * need + MIB
    keep = cd.Solver(wl.sod(n=16, nv=16))  # idle blocks are kept while something lives
    srv = cd.Server(budget, max_active=3, chunk_steps=20)
    # a short request first: queues, code and batch tables are there
    poll(srv, srv.submit(p, 2))
    cd.Solver(larger).close()
    free0 = free_memory()  # with what lies idle
    steps = 4000
    tickets, least = [], free0
    for _ in range(3):
        tickets.append(srv.submit(p, steps))
        time.sleep(0.1)  # admitted one after another, not in one go
        least = min(least, free_memory())
    results = [poll(srv, t) for t in tickets]
    queued, served = [r[3] for r in results], [r[4] for r in results]
    print(f"queued {queued} served {served} held {(free0 - least) / need:.2f} requests' bytes", flush=True)
    assert served[0] > 0.5  # long enough to overlap
    assert max(queued) < 0.25 * served[0], (queued, served)
    srv.close()
    keep.close()


def test_requests_and_idle_blocks_stay_within_the_budget():
    sizes = [128, 140, 118, 133, 125, 140, 118]
    problems = [problem(n) for n in sizes]
    budget = int(2.5 * max(cd.cdugks_required_bytes(p) for p in problems))
    cd.Solver(problems[0]).close()  # queues and code loaded, nothing kept
    free0 = free_memory()
    srv = cd.Server(budget, max_active=4, chunk_steps=10)
    tickets, least = [], free0
    for p in problems:
        tickets.append(srv.submit(p, 200))
    waiting = set(tickets)
    while waiting:
        waiting -= {t for t in waiting if srv.poll(t) is not None}
        least = min(least, free_memory())
        time.sleep(0.001)
    least = min(least, free_memory())
    srv.close()
    held = free0 - least
    # batch tables and the runtime's own allocations beside the requests
    assert held <= budget + 64 * MIB, (held, budget)
    assert free0 - free_memory() <= 64 * MIB
