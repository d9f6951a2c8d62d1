"""The timing helper: a duration for each of the four phases, and steps like
any other's."""
import numpy as np
import pytest

from paper_2208_09132_amd import cdugks as cd
from paper_2208_09132_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dim", [1, 2, 3])
@pytest.mark.parametrize("storage", ["f64", "f32_bf16tail"])
def test_four_phases_and_the_same_state(dim, storage):
    p = wl.random_fourier(dim, [19, 17, 11][:dim], [9, 8, 7][:dim], wl.SplitMix64(dim), Kn=1e-2, storage=storage)
    a, b = cd.Solver(p), cd.Solver(p)
    a.step(3)
    ms = b.profile_phases(3)
    print(f"dim {dim} {storage}: {ms}", flush=True)
    assert ms.shape == (4,) and np.all(ms > 0.0) and np.all(ms < 100.0), ms
    assert b.info() == a.info()
    for x, y in zip(a.moments() + a.distributions(), b.moments() + b.distributions()):
        assert np.array_equal(x, y)
    a.close()
    b.close()
