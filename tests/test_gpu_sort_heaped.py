"""GPU tests of the sort's other forms: cells that hold many times the mean
(k_cell_gather's listed particles, in cells with and without table rows to
spare, several of them at once), cells full on average, thinly filled and very
large grids (chunk sums scanned by a launch, in more than one round), each
bit-exact against the stable sort; and the time of a sort with 20,000
particles in one cell, which must not be a wave's own work."""
import time

import numpy as np
import pytest
import torch

import oracle
import paper_1909_04504_amd as sph
import sph_workloads as W
from test_gpu_parity import gpu_sorted

pytestmark = pytest.mark.gpu


def grid_params(nc, cell_div=1):
    d = len(nc)
    p, _ = W.taylor_green(16) if d == 2 else W.periodic_cube(n_side=14, cell_div=2)
    p = p.replace(cell_div=cell_div)
    cell = 2 * p.h / cell_div
    lo = np.array(p.lo[:d], float)
    hi = tuple(lo[k] + (nc[k] + 1e-6) * cell for k in range(d)) + tuple(p.hi[d:])
    return p.replace(hi=hi), lo, cell


def heaped_state(nc, spread, heaps, cell_div=1, seed=0):
    """spread particles at random, and heaps of (cell, particles)."""
    p, lo, cell = grid_params(nc, cell_div)
    d = len(nc)
    rng = np.random.default_rng(seed)
    x = [lo[:, None] + rng.random((d, spread)) * (np.array(nc) * cell)[:, None]]
    for at, k in heaps:
        x.append(lo[:, None] + (np.array(at)[:, None] + 0.1 + 0.8 * rng.random((d, k))) * cell)
    x = np.concatenate(x, axis=1)
    n = x.shape[1]
    x = x[:, rng.permutation(n)]
    return p, W.State(x, rng.standard_normal((d, n)), rng.random(n) + 1.0,
                      np.zeros(n, np.uint8), rng.permutation(n).astype(np.int32))


def check_sort(p, s, prec):
    _, perm, cs_ref, ce_ref = oracle.bin_sort(p, s.x)
    prm, dp, ws, cs, ce = gpu_sorted(p, s, prec)
    for again in (False, True):
        if again:  # on what the first sort left in the workspace
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


# cells per axis, particles spread, heaps, cell_div; cells a wave: 8 in the
# plane, 16 or 32 (half cells) and 4 in space, so that 96, 48 or 24 and 192 a
# cell are the most without listed particles
HEAPED = [((64, 64), 20000, [((5, 6), 95)], 1), ((64, 64), 20000, [((5, 6), 140)], 1),
          ((9, 9), 300, [((0, 0), 5000)], 1), ((100, 100), 50000, [((k, 3 * k), 300 + 40 * k)
                                                                 for k in range(30)], 1),
          ((300, 300), 600000, [((299, 299), 3000), ((0, 0), 700), ((150, 20), 97)], 1),
          ((30, 31, 32), 70000, [((29, 30, 31), 60), ((3, 3, 3), 2000)], 2),
          ((70, 70, 70), 700000, [((0, 0, 0), 25), ((69, 69, 69), 4000)], 2),
          ((20, 20, 20), 140000, [((19, 0, 7), 250)], 1), ((3, 3), 1, [((1, 1), 3000)], 1)]


@pytest.mark.parametrize("nc,spread,heaps,cell_div", HEAPED)
@pytest.mark.parametrize("prec", [sph.FP64, sph.FP32_MIXED])
def test_heaped_cells_bit_exact(nc, spread, heaps, cell_div, prec):
    p, s = heaped_state(nc, spread, heaps, cell_div, seed=spread)
    check_sort(p, s, prec)


# full cells (36 a cell is the line, and above), thinly filled grids, and grids
# above 256 chunks of 4,096 cells (dense and sparse) and above 2,048 of them
SHAPES = [((24, 24), 24 * 24 * 36, 1), ((24, 24), 24 * 24 * 36 + 1, 1), ((150, 150), 40 * 22500, 1),
          ((11, 12, 13), 64 * 1716, 1), ((60, 61), 3000, 1), ((200, 201), 150000, 1),
          ((30, 30, 30), 200000, 1), ((30, 30, 30), 290000, 1), ((1100, 1100), 5000000, 1),
          ((1100, 1100), 1300000, 1), ((1300, 1300), 20000, 1), ((3000, 3000), 4000, 1)]


@pytest.mark.parametrize("nc,n,cell_div", SHAPES)
def test_sort_forms_bit_exact(nc, n, cell_div):
    p, s = heaped_state(nc, n, [], cell_div, seed=n)
    check_sort(p, s, sph.FP32_MIXED)


def test_heaped_run_equals_single_steps():
    """Steps on a grid with a heap: the epilogue of the momentum pass lists the
    particles of the next sort, and both count buffers see heaps."""
    p, s = W.taylor_green(40, jitter=0.2, seed=3)
    rng = np.random.default_rng(1)
    k = rng.permutation(s.n)[:200]  # 200 of the 1600 into two cells
    s.x[:, k] = 0.31 + 0.02 * rng.random((2, k.size))
    p = p.replace(dt=1e-9)
    prm = sph.make_params(p, sph.FP64)
    out = []
    for calls in ([4], [1, 1, 1, 1]):
        dp = sph.DeviceParticles.from_state(s, sph.FP64)
        ws = sph.workspace(prm, s.n)
        sph.step(prm, dp, 0, ws, prime=True)
        for c in calls:
            sph.step(prm, dp, c, ws, prime=False)
        torch.cuda.synchronize()
        out.append(dp.numpy())
    _, perm, _, _ = oracle.bin_sort(p, out[0]["x"])
    assert np.array_equal(perm, np.arange(s.n))  # in sorted order
    for f in ("x", "u", "a", "rho", "p", "id"):
        assert np.array_equal(out[0][f], out[1][f]), f


@pytest.mark.parametrize("nc,spread", [((100, 100), 60000), ((400, 400), 1000000)])
def test_heap_does_not_serialise(nc, spread):
    """20,000 particles of one cell: 1.5 to 1.7 ms with a thread per particle; as
    one wave's work 4,000 took 20 ms, and the time goes with their square."""
    p, s = heaped_state(nc, spread, [((30, 30), 20000)])
    prm, dp, ws, cs, ce = gpu_sorted(p, s, sph.FP64)
    torch.cuda.synchronize()
    t = time.perf_counter()
    sph.bin_sort(prm, dp, ws, cs, ce)
    torch.cuda.synchronize()
    assert time.perf_counter() - t < 0.05
