"""FP64 distributions at the bottom of the number range: a limited slope that
eq. VanLeer rejects is exactly zero, so nothing is added to tails that are
subnormal or have underflowed to zero.

Blocks of hot, coldest and cold gas stand side by side: towards the ends of the
velocity box the coldest cell is a strict minimum between a large value and a
subnormal one, and every slope of the row is zero.  A residue of the rejected
slope (any multiple of the smallest subnormal) would reach the first cold cell
through its face.  (The last cold cell is left out: its face to the hot gas has
an equilibrium of ordinary size, whose rounding is all that is left there.)"""
import numpy as np
import pytest

from paper_2208_09132_amd import cdugks as cd
from paper_2208_09132_amd import workloads as wl
from tests.helpers import dt_checked, make_oracle

pytestmark = pytest.mark.gpu

TINY = 2.0 ** -1074


def problem(dim):
    rng = wl.SplitMix64(17)
    T = []
    for _ in range(8):
        cold = rng.uniform(0.1395, 0.1412)  # g near 1e-312..1e-308 at |xi| = 10
        T += [20.0] * 4 + [rng.uniform(0.125, 0.1338)] + [cold] * 4
    T = np.array(T)
    n = [len(T)] + [5] * (dim - 1)
    Tc = np.tile(T, 5 ** (dim - 1))
    p = dict(dim=dim, n=n, lo=[0.0] * dim, hi=[1.0] + [5.0 / len(T)] * (dim - 1), bc=["periodic"] * dim,
             nv=[81] + [9] * (dim - 1), vmin=[-10.0] + [-1.0] * (dim - 1), vmax=[10.0] + [1.0] * (dim - 1),
             relax="tau", tau=float("inf"), rho=np.ones(len(Tc)), u=np.zeros((dim, len(Tc))), T=Tc)
    return p


@pytest.mark.parametrize("dim", [1, 2])
def test_a_rejected_slope_adds_nothing_to_subnormal_tails(dim):
    p = problem(dim)
    s = cd.Solver(p)
    o = make_oracle(p, dt=dt_checked(p, s.dt))
    # both sides from the library's own initial state: one step's arithmetic
    g0, b0 = s.distributions()
    o.set_state(np.ascontiguousarray(g0.T), np.ascontiguousarray(b0.T), s.conserved())
    s.step(1)
    assert o.step(1) == 0
    g, b = s.distributions()
    s.close()
    og, ob, _ = o.state()
    cold = np.isin(np.arange(g.shape[1]) % p["n"][0] % 9, (5, 6, 7))[None, :]
    for name, start, ref, got in (("g", g0, og.T, g), ("b", b0, ob.T, b)):
        tail = cold & (ref > 0.0) & (ref < 1e-306) & (start < 1e-306)
        assert tail.sum() >= 24, (name, int(tail.sum()))
        err = np.abs(got[tail] - ref[tail])
        # the step's roundings: relative, and of the smallest subnormal each
        worst = float(np.max(err / (1e-12 * ref[tail] + 64 * TINY)))
        print(f"dim {dim} {name}: {int(tail.sum())} values below 1e-306, error/bound {worst:.3g}", flush=True)
        assert worst <= 1.0, (name, worst)
