"""Columns of the 3-D face sums chosen for the grid's extents: grids of one
ragged column, of columns of up to 192 and of up to 256 cells, narrow grids
along either axis and rows of whole 64-byte sectors give bitwise what the box
shape gives, and the FP64 oracle's moments within the parity tests' bounds; so
do Dirichlet sides and the single-slope option on such a grid."""
import numpy as np
import pytest

from paper_2208_09132_amd import cdugks as cd
from paper_2208_09132_amd import workloads as wl
from tests.helpers import dt_checked, make_oracle, moment_errors

pytestmark = pytest.mark.gpu

GRIDS = [([17, 9, 5], None, {}),
         ([20, 20, 4], None, {}),
         ([33, 33, 3], ["outflow", "outflow", "periodic"], {}),
         ([5, 41, 4], ["periodic", "outflow", "outflow"], {}),
         ([67, 5, 4], ["outflow", "periodic", "outflow"], {}),
         ([16, 18, 4], None, {}),
         ([32, 17, 4], None, {}),
         ([3, 4, 3], None, {}),
         ([21, 18, 4], ["periodic", "dirichlet", "outflow"],
          {"dirichlet": [None, [[1.1, 0.1, -0.1, 0.05, 1.1], [0.9, -0.1, 0.05, 0.0, 0.9]], None]}),
         ([18, 21, 4], None, {"reconstruction": "single_slope"})]


@pytest.mark.parametrize("storage", ["f64", "f32", "f32_bf16tail"])
@pytest.mark.parametrize("n, bc, more", GRIDS)
def test_columns_give_the_box_shape_s_results(n, bc, more, storage):
    p = dict(wl.random_fourier(3, n, [7, 8, 7], wl.SplitMix64(17), amp=0.2, Kn=1e-2, storage=storage), **more)
    if bc:
        p["bc"] = bc
    box, column = cd.Solver(dict(p, face_tile=1)), cd.Solver(p)
    assert column.launch_info()[0] == 7
    for s in (box, column):
        s.step(3)
    for a, b in zip(box.moments() + box.distributions(), column.moments() + column.distributions()):
        assert np.array_equal(a, b)
    o = make_oracle(p, dt=dt_checked(p, column.dt))
    assert o.step(3) == 0
    assert max(moment_errors(o.moments(), column.moments())) <= (1e-12 if storage == "f64" else 1e-5)
    for s in (box, column):
        s.close()
