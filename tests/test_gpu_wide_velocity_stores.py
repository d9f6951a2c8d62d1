"""2-D FP32 forms stream their face values over 4096 velocities and more on
rows of whole 64-byte sectors: the bits of the 32 x 8 tile, whose kernel stores
ordinarily, on both sides of the line and on ragged rows."""
import numpy as np
import pytest

from paper_2208_09132_amd import cdugks as cd
from paper_2208_09132_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("storage", ["f32", "f32_bf16tail"])
@pytest.mark.parametrize("n0, nv", [(64, [64, 64]), (64, [65, 63]), (63, [64, 64])])
@pytest.mark.parametrize("form", ["plain", "outflow"])
def test_streamed_and_ordinary_stores_agree(storage, n0, nv, form):
    out = []
    for tile in (1, 2):
        p = wl.random_fourier(2, [n0, 40], nv, wl.SplitMix64(9), Kn=1e-2, storage=storage)
        # one launch for values and sums, whatever the device's size
        p.update(face_tile=tile, velocity_slices=256)
        if form == "outflow":
            p["bc"] = ["periodic", "outflow"]
        s = cd.Solver(p)
        s.step(3)
        out.append(s.moments() + s.distributions())
        s.close()
    for a, b in zip(*out):
        assert np.array_equal(a, b)
