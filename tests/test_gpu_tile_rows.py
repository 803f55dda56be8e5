"""GPU test of the tile builds' row queue: particles spread at random, so that
stencil rows are empty, end within a group of four, or span several groups, in
every order; bitwise the fields and lists of the global walk."""
import numpy as np
import pytest

import paper_1909_04504_amd as sph
import sph_workloads as W
from test_gpu_list_tiles import csr
from test_gpu_tiles import FIELDS, ON, case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", [sph.FP64, sph.FP32_MIXED])
@pytest.mark.parametrize("name", ["cube32_cd1", "cube32_cd2"])
@pytest.mark.parametrize("keep", [0.02, 0.3, 1.0])
def test_random_rows_bitwise_equal_to_walk(name, keep, prec):
    p, s = case("cube32_cd2")
    if name == "cube32_cd1":
        p = p.replace(cell_div=1)
    rng = np.random.default_rng(7)
    n = int(keep * s.n)
    x = np.stack([p.lo[k] + rng.random(n) * (p.hi[k] - p.lo[k]) for k in range(3)])
    s = W.State(x, s.u[:, :n].copy(), s.m[:n].copy(), s.ptype[:n].copy(), s.pid[:n].copy())
    outs = []
    for tiles in (-1, ON):
        prm = sph.make_params(p, prec, 192, pair_tiles=tiles)
        dp = sph.DeviceParticles.from_state(s, prec)
        ws = sph.workspace(prm, s.n)
        sph.step(prm, dp, 0, ws, prime=True)
        sph.check(ws)
        outs.append((dp.numpy(), csr(p, s, prec, 192, tiles)))
    a, b = outs
    for f in FIELDS:
        assert np.array_equal(a[0][f], b[0][f]), f
    assert np.array_equal(a[1][0], b[1][0]) and np.array_equal(a[1][1], b[1][1])
