"""How face values are stored (streaming on rows of whole 64-byte sectors,
ordinary otherwise; 2-D FP32 forms always ordinary, 3-D kernels either) never
changes a value: rows on and off the sectors give bitwise what a batch, whose
kernels choose for themselves, gives, and the FP64 oracle's moments within the
parity tests' bounds.  Row lengths: whole sectors, one value more, one less,
and an outflow axis, whose rows hold one face more than cells."""
import numpy as np
import pytest

from paper_2208_09132_amd import cdugks as cd
from paper_2208_09132_amd import workloads as wl
from tests.helpers import dt_checked, make_oracle, moment_errors

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("storage", ["f64", "f32", "f32_bf16tail"])
@pytest.mark.parametrize("n, nv, bc", [
    ([32, 19], [10, 9], None),
    ([33, 19], [10, 9], None),
    ([31, 19], [10, 9], ["outflow", "periodic"]),
    ([32, 7, 5], [7, 8, 7], None),
    ([17, 7, 5], [7, 8, 7], ["periodic", "outflow", "periodic"]),
    ([15, 18, 6], [7, 8, 7], ["outflow", "periodic", "outflow"]),
])
def test_rows_on_and_off_whole_sectors(n, nv, bc, storage):
    p = wl.random_fourier(len(n), n, nv, wl.SplitMix64(31), amp=0.2, Kn=1e-2, storage=storage)
    if bc:
        p["bc"] = bc
    # short slices of the sums, so the 2-D runs take the one-launch kernels
    p["velocity_slices"] = 2 if len(n) == 3 else int(np.prod(nv)) // 8
    solo, one = cd.Solver(p), cd.Solver(p)
    batch = cd.Batch([one], chunk_steps=2)
    solo.step(3)
    batch.step(3)
    for a, b in zip(solo.moments() + solo.distributions(), one.moments() + one.distributions()):
        assert np.array_equal(a, b)
    o = make_oracle(p, dt=dt_checked(p, solo.dt))
    assert o.step(3) == 0
    assert max(moment_errors(o.moments(), solo.moments())) <= (1e-12 if storage == "f64" else 1e-5)
    batch.close()
