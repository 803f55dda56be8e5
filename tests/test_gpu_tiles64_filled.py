"""GPU tests of the FP64 tiles where the fluid is denser than the mean of its
grid, so that the boxes chosen by the mean overflow: partly filled periodic
boxes (the tile passes leave every target to the fallback, which writes lists),
boxes of which a part is compressed, and lists too short for their targets.
Everything bitwise the passes over global lists, and not slower than them by
more than the probe."""
import time

import numpy as np
import pytest
import torch

import paper_1909_04504_amd as sph
import sph_workloads as W

pytestmark = pytest.mark.gpu


def filled(side, hdx, cell_div, frac, squeeze=0.0):
    """The part z < frac of a periodic cube; squeeze: the part x < squeeze of it
    pressed to half its width."""
    p, s = W.periodic_cube(n_side=side, hdx=hdx, cell_div=cell_div)
    keep = s.x[2] < frac
    x = s.x[:, keep]
    if squeeze:
        x[0] = np.where(x[0] < squeeze, 0.5 * x[0], x[0])
    n = x.shape[1]
    # nothing moves far, whatever the pressure
    return p.replace(dt=1e-9), W.State(x, s.u[:, keep], s.m[keep], np.zeros(n, np.uint8),
                                       np.arange(n, dtype=np.int32))


def steps(p, s, pair_tiles, nbr_cap, n=2):
    prm = sph.make_params(p, sph.FP64, pair_tiles=pair_tiles, nbr_cap=nbr_cap)
    dp = sph.DeviceParticles.from_state(s, sph.FP64)
    ws = sph.workspace(prm, s.n)
    diag = torch.zeros((n, 4), dtype=torch.float64, device="cuda")
    sph.step(prm, dp, n, ws, prime=True, diag=diag)
    out = dp.numpy()
    sph.check(ws)
    return out, diag.cpu().numpy(), sph.read_interactions(ws)


# (side, h/dx, cell_div, filled, squeezed, pair_tiles, nbr_cap)
CASES = [(24, 1.5, 1, 0.5, 0, 0, 0), (24, 1.7, 2, 0.5, 0, 0, 0), (24, 1.5, 2, 1.0, 0.6, 0, 400),
         (26, 1.5, 1, 1.0, 0.5, 0, 400), (24, 1.5, 2, 1.0, 0.1, 1900, 400),
         (24, 1.5, 2, 0.5, 0, 700, 0), (24, 1.5, 2, 1.0, 0, 0, 80), (24, 1.5, 1, 0.5, 0, 1500, 104)]


@pytest.mark.parametrize("side,hdx,cell_div,frac,squeeze,tiles,cap", CASES)
def test_denser_than_the_mean(side, hdx, cell_div, frac, squeeze, tiles, cap):
    p, s = filled(side, hdx, cell_div, frac, squeeze)
    got, dg, ng = steps(p, s, tiles, cap)
    ref, dr, nr = steps(p, s, -1, cap)
    for f in ("x", "u", "a", "rho", "p", "id"):
        assert np.array_equal(got[f], ref[f]), f
    assert ng == nr
    assert np.abs(dg - dr).max() <= 1e-13 * np.abs(dr).max()  # sums in another order

    # the terms one by one on the sorted state
    out = []
    for t in (tiles, -1):
        prm = sph.make_params(p, sph.FP64, pair_tiles=t, nbr_cap=cap)
        dp = sph.DeviceParticles.from_state(s, sph.FP64)
        ws = sph.workspace(prm, s.n)
        cs, ce = sph.cell_arrays(prm)
        sph.bin_sort(prm, dp, ws, cs, ce)
        sph.density(prm, dp, cs, ce, ws)
        sph.eos(prm, dp)
        off = torch.zeros(s.n + 1, dtype=torch.int64, device="cuda")
        nbr = torch.zeros(s.n * 400, dtype=torch.int32, device="cuda")
        total = sph.neighbors(prm, dp, cs, ce, nbr.numel(), off, nbr, ws)
        sph.momentum(prm, dp, cs, ce, ws)
        d = dp.numpy()
        out.append((d["rho"], d["p"], d["a"], off.cpu().numpy(), nbr[:total].cpu().numpy()))
    for a, b in zip(*out):
        assert np.array_equal(a, b)


@pytest.mark.parametrize("hdx,cell_div,frac", [(1.5, 1, 0.5), (1.5, 1, 0.75), (1.7, 2, 0.25),
                                               (1.7, 2, 0.5), (1.1, 1, 0.25)])
def test_partly_filled_box_is_not_slower(hdx, cell_div, frac):
    """At most 1.4 times the passes over global lists (measured 0.93 to 1.12;
    1.3 to 2.5 before)."""
    p, s = filled(64, hdx, cell_div, frac)
    best = {}
    for again in range(3):
        for tiles in (0, -1):
            prm = sph.make_params(p, sph.FP64, pair_tiles=tiles)
            dp = sph.DeviceParticles.from_state(s, sph.FP64)
            ws = sph.workspace(prm, s.n)
            sph.step(prm, dp, 5, ws, prime=True)
            torch.cuda.synchronize()
            t = time.perf_counter()
            sph.step(prm, dp, 20, ws, prime=False)
            torch.cuda.synchronize()
            best[tiles] = min(best.get(tiles, 1e9), time.perf_counter() - t)
    assert best[0] <= 1.4 * best[-1]
