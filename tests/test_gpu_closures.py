"""The face closure's groups of threads (one thread, 16, 64 or a whole
workgroup per face, chosen from the face count and the number of velocity
nodes) and the cell closure inside the update, against the FP64 oracle:
moments within 1e-12 and g, b within 1e-12 of each velocity row's largest
value, the parity bound of the other FP64 tests (a group adds up in the order
of one thread, so no bound of its own is needed).  Each size sits at an edge of
the rule or of the groups' work: node counts at and past a chunk, blocks of 16
nodes left partly empty, more velocity slices than one pass over them holds,
the face count from which one thread takes a face, and faces outside the grid
(outflow) beside groups that close theirs."""
import numpy as np
import pytest

from paper_2208_09132_amd import cdugks as cd
from paper_2208_09132_amd import workloads as wl
from tests.test_gpu_accel import parity

pytestmark = pytest.mark.gpu


def problem(n, nv, bc=None, accel=None):
    p = wl.random_fourier(len(n), n, nv, wl.SplitMix64(17), amp=0.2, Kn=1e-2)
    if bc:
        p["bc"] = bc
    p["accel"] = accel or [0.0] * len(n)
    return p


@pytest.mark.parametrize("n, nv, bc, accel, slices", [
    ([5], [31], None, None, 0),                # 16 threads per face
    ([7], [33], ["outflow"], [0.5], 33),       # 64, one node past two blocks, a slice per velocity
    ([130], [128], None, None, 128),           # 64, a whole chunk, more slices than a pass
    ([3], [129], ["outflow"], None, 0),        # a workgroup, one node past
    ([600], [511], None, [0.3], 70),           # 64, several chunks
    ([1], [513], ["outflow"], None, 513),      # a workgroup, one node past a chunk
    ([33], [2050], None, [0.3], 0),            # a workgroup per face, ragged
    ([6, 5], [33, 9], ["outflow", "periodic"], [0.2, -0.1], 60),
    ([3, 4], [9, 129], ["periodic", "outflow"], None, 0),
    ([40, 50], [17, 16], ["periodic", "outflow"], None, 5),  # 16, more than one chunk
    ([256, 128], [7, 7], None, None, 0),       # 2^16 faces: one thread per face
    ([3, 4, 5], [33, 9, 9], ["outflow", "outflow", "periodic"], [0.1, 0.2, -0.1], 0),
])
def test_closures_match_the_oracle(n, nv, bc, accel, slices):
    p = problem(n, nv, bc, accel)
    p["velocity_slices"] = slices
    parity(p, 3, 1e-12, distributions=True)


def test_closures_in_a_batch_equal_solo_runs():
    probs = [problem([5], [31]), problem([70], [200], ["outflow"]), problem([9], [700]), problem([11, 6], [9, 35]),
             problem([3, 4, 5], [9, 9, 9])]
    solo = [cd.Solver(p) for p in probs]
    many = [cd.Solver(p) for p in probs]
    batch = cd.Batch(many, chunk_steps=4)
    batch.step(7)
    for p, s, m in zip(probs, solo, many):
        s.step(7)
        for a, b in zip(s.moments() + s.distributions(), m.moments() + m.distributions()):
            assert np.array_equal(a, b), p["n"]
    batch.close()
