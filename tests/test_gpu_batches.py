"""Batches against the same problems alone, bit for bit, in the forms whose
kernels are compiled differently for batches: 3-D FP64 with and without an
acceleration (register limits, face-value stores) and 2-D FP64 (face-value
stores), on face grids whose rows fill whole 64-byte sectors and on ragged
ones, and one of each together."""
import numpy as np
import pytest

from paper_2208_09132_amd import cdugks as cd
from paper_2208_09132_amd import workloads as wl

pytestmark = pytest.mark.gpu


def fourier(n, nv, storage, seed, **kw):
    p = wl.random_fourier(len(n), n, nv, wl.SplitMix64(seed), Kn=1e-2, storage=storage)
    p.update(kw)
    return p


def state(s):
    return s.moments() + s.distributions()


def check(problems, steps=3):
    alone = []
    for p in problems:
        s = cd.Solver(p)
        s.step(steps)
        alone.append(state(s))
        s.close()
    first = cd.Solver(problems[0])
    solvers = [first] + [cd.Solver(p) for p in problems[1:]]
    b = cd.Batch(solvers, chunk_steps=2)
    b.step(steps)
    got = [state(s) for s in solvers]
    b.close()
    for s in solvers:
        s.close()
    for p, x, y in zip(problems, got, alone):
        assert all(np.array_equal(u, v) for u, v in zip(x, y)), (p["n"], p["storage"])


SECTORS, RAGGED = [16, 8, 8], [17, 6, 9]


@pytest.mark.parametrize("accel", [None, [0.1, 0.0, -0.05]])
@pytest.mark.parametrize("sizes", [[SECTORS], [RAGGED], [SECTORS, RAGGED]])
def test_3d_fp64(sizes, accel):
    kw = {} if accel is None else dict(accel=accel)
    check([fourier(n, [7, 6, 5], "f64", 3 + k, **kw) for k, n in enumerate(sizes)])


@pytest.mark.parametrize("form", ["plain", "accel", "single_slope", "dirichlet"])
@pytest.mark.parametrize("n0", [[24, 40], [23, 33], [24, 23]])
def test_2d_fp64(n0, form):
    kw = {"plain": {}, "accel": dict(accel=[0.1, -0.05]), "single_slope": dict(reconstruction="single_slope"),
          "dirichlet": dict(bc=["periodic", "dirichlet"], dirichlet=[None, [[1.0, 0.0, 0.0, 1.0]] * 2])}[form]
    # with a 1-D problem beside them, whose rows do not count
    check([fourier([m, 19], [8, 7], "f64", m, **kw) for m in n0] +
          ([wl.sod(n=50, nv=12)] if form == "plain" else []))
