"""An autotuned context launches like a fresh one of its tile shape: whatever
shape it was set up with, the split of face values and sums (which small
problems have in shape 0 alone) is that of the shape it ends with."""
import os
import subprocess

import pytest

from paper_2208_09132_amd import cdugks as cd
from tests.test_launch_rules import build

pytestmark = pytest.mark.gpu

SOURCE = r"""
#include "cdugks_host.h"
#include <cstdio>
#include <cstdlib>
#include <vector>
int main(int argc, char** argv) {
    const int n = atoi(argv[1]), nv = atoi(argv[2]), tile = atoi(argv[3]);
    cdugks_space sp{};
    cdugks_velocity ve{};
    cdugks_params pa{};
    sp.dim = 2;
    for (int d = 0; d < 2; ++d) {
        sp.n[d] = n;
        sp.hi[d] = 1.0;
        ve.nv[d] = nv;
        ve.vmin[d] = -5.0;
        ve.vmax[d] = 5.0;
    }
    pa.gamma = 5.0 / 3.0;
    pa.Pr = 2.0 / 3.0;
    pa.R = 0.5;
    pa.omega = 0.5;
    pa.relax_mode = CDUGKS_RELAX_TAU;
    pa.tau = 0.1;
    pa.cfl = 0.5;
    pa.face_tile = tile;
    std::vector<double> one(n * n, 1.0), u(2 * n * n, 0.0);
    cdugks_ctx* c = nullptr;
    if (cdugks_init(&sp, &ve, &pa, one.data(), u.data(), one.data(), nullptr, nullptr, 0, &c)) return 1;
    const int before = c->P.value_slices, want_before = cdg::value_slices(c->r);
    if (cdugks_autotune(c, 20)) return 2;
    printf("%d %d %d %d %d", before, want_before, c->r.tile, c->P.value_slices, cdg::value_slices(c->r));
    cdugks_destroy(c);
    return 0;
}
"""


@pytest.mark.parametrize("n, nv", [(32, 20), (16, 24), (41, 13), (24, 40)])
def test_the_split_follows_the_tuned_shape(tmp_path, n, nv):
    exe = build(str(tmp_path), SOURCE, [cd.LIB_PATH, "-Wl,-rpath," + os.path.dirname(cd.LIB_PATH),
                                        "-Wl,--allow-shlib-undefined"])
    env = {k: v for k, v in os.environ.items() if k != "CDUGKS_TUNE_CACHE"}
    out = subprocess.run([exe, str(n), str(nv), "2"], check=True, stdout=subprocess.PIPE, text=True, env=env,
                         timeout=60).stdout
    before, want_before, tile, after, want = (int(x) for x in out.split())
    print(f"{n}^2 x {nv}^2: set up with {before} slices, tuned to shape {tile} with {after}", flush=True)
    assert before == want_before == 0  # shape 1 has no split
    assert after == want
