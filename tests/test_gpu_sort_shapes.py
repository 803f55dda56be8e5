"""GPU test of the sort's launch shapes: grids that count in the gather (up to
16,384 cells) and just above, grids with more groups of cells than one scan
takes, sparse grids, and cells that outgrow their table row, the gather's
entries and its rounds; twice on one workspace.  Bit-exact against the stable
sort."""
import numpy as np
import pytest

import oracle
import paper_1909_04504_amd as sph
import sph_workloads as W
from test_gpu_parity import gpu_sorted

pytestmark = pytest.mark.gpu

# cells per axis, particles spread at random, particles in one cell
SHAPES = [((128, 128), 40000, 0), ((128, 129), 40000, 0), ((128, 128), 3000, 2500),
          ((129, 131), 30000, 2500), ((400, 400), 5000, 0), ((400, 400), 300, 2500),
          ((900, 900), 900000, 400), ((24, 25, 27), 50000, 1500), ((25, 26, 27), 2000, 1500),
          ((90, 90, 90), 800000, 0), ((90, 90, 90), 20000, 700)]


@pytest.mark.parametrize("nc,spread,packed", SHAPES)
@pytest.mark.parametrize("prec", [sph.FP64, sph.FP32_MIXED])
def test_sort_shapes_bit_exact(nc, spread, packed, prec):
    d = len(nc)
    p, _ = W.taylor_green(16) if d == 2 else W.periodic_cube(n_side=14, cell_div=2)
    cell = 2 * p.h / p.cell_div
    lo = np.array(p.lo[:d], float)
    p = p.replace(hi=tuple(lo[k] + (nc[k] + 1e-6) * cell for k in range(d)) + tuple(p.hi[d:]))
    rng = np.random.default_rng(sum(nc) + packed)
    size = np.array(nc) * cell
    x = lo[:, None] + rng.random((d, spread)) * size[:, None]
    if packed:
        at = (np.array(nc) // 3)[:, None] + 0.1 + 0.8 * rng.random((d, packed))
        x = np.concatenate([x, lo[:, None] + at * cell], axis=1)
    n = x.shape[1]
    x = x[:, rng.permutation(n)]
    s = W.State(x, rng.standard_normal((d, n)), rng.random(n) + 1.0,
                np.zeros(n, np.uint8), rng.permutation(n).astype(np.int32))
    _, perm, cs_ref, ce_ref = oracle.bin_sort(p, s.x)
    assert cs_ref.size == np.prod(nc)
    prm, dp, ws, cs, ce = gpu_sorted(p, s, prec)
    for again in (False, True):
        if again:  # on the other buffer of counts, already in order
            cs.zero_()
            ce.zero_()
            sph.bin_sort(prm, dp, ws, cs, ce)
        out = dp.numpy()
        assert np.array_equal(out["id"], s.pid[perm])
        assert np.array_equal(out["x"], s.x[:, perm])
        assert np.array_equal(out["u"], s.u[:, perm])
        assert np.array_equal(out["m"], s.m[perm])
        assert np.array_equal(cs.cpu().numpy().view(np.uint32), cs_ref)
        assert np.array_equal(ce.cpu().numpy().view(np.uint32), ce_ref)
    sph.check(ws)
