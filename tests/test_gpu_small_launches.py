"""Problems that leave most of the device idle: a single run stores its face
values in short velocity slices and sums them in a second launch, and updates
in short slices; in a batch the same problem takes one launch with the sums'
own slices.  Both have to give bitwise the same moments and distributions, and
the FP64 oracle's moments within the parity tests' bounds (1e-12; FP32 forms
1e-5).  Sizes: velocity counts a slice of 4 does not divide, slices starting
inside a block of the Maxwellian recurrence (8 nodes), one tile and ragged
tiles, every kernel variant (Dirichlet sides, single slope, acceleration)."""
import numpy as np
import pytest

from paper_2208_09132_amd import cdugks as cd
from paper_2208_09132_amd import workloads as wl
from tests.helpers import dt_checked, make_oracle, moment_errors

pytestmark = pytest.mark.gpu


def problem(n, nv, storage, bc=None, **kw):
    D = len(n)
    p = wl.random_fourier(D, n, nv, wl.SplitMix64(29), amp=0.2, Kn=1e-2, storage=storage)
    if bc:
        p["bc"] = bc
        side = [[1.0] + [0.05] * D + [1.0], [0.9] + [-0.05] * D + [1.1]]
        p["dirichlet"] = [side if b == "dirichlet" else None for b in bc]
    return dict(p, **kw)


CASES = [
    ([40], [24], None, {}),
    ([257], [61], ["outflow"], {}),
    ([300], [200], ["dirichlet"], {}),
    ([300], [97], ["dirichlet"], {"reconstruction": "single_slope"}),
    ([130], [65], ["dirichlet"], {"accel": [0.3]}),
    ([13, 9], [9, 13], None, {}),
    ([33, 17], [13, 15], ["outflow", "dirichlet"], {}),
    ([20, 40], [11, 12], ["periodic", "dirichlet"], {"reconstruction": "single_slope"}),
    ([35, 20], [12, 14], ["dirichlet", "outflow"], {"accel": [0.1, -0.2]}),
]


@pytest.mark.parametrize("storage", ["f64", "f32", "f32_bf16tail"])
@pytest.mark.parametrize("n, nv, bc, kw", CASES)
def test_split_launches_equal_the_batched_ones(n, nv, bc, kw, storage):
    p = problem(n, nv, storage, bc, **kw)
    solo, one = cd.Solver(p), cd.Solver(p)
    batch = cd.Batch([one], chunk_steps=2)
    solo.step(5)
    batch.step(5)
    for a, b in zip(solo.moments() + solo.distributions(), one.moments() + one.distributions()):
        assert np.array_equal(a, b)
    o = make_oracle(p, dt=dt_checked(p, solo.dt))
    assert o.step(5) == 0
    assert max(moment_errors(o.moments(), solo.moments())) <= (1e-12 if storage == "f64" else 1e-5)
    batch.close()
