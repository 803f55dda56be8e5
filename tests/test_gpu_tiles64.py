"""GPU tests of the LDS-tiled 3D passes in FP64: bitwise the fields of the
global-list passes (the same records, pair terms and neighbour order) for
boxes that wrap a periodic grid onto themselves, partial boxes, walls, a wide
support, unions above the staging capacity and lists above theirs, Z-order
keys, and particles clamped into edge cells from near and far outside."""
import numpy as np
import pytest
import torch

import paper_1909_04504_amd as sph
import sph_workloads as W
from helpers import shuffled
from test_gpu_tiles import CASES, FIELDS, ON, case

pytestmark = pytest.mark.gpu


def run(p, s, tiles, nsteps, cap=0, code=0):
    prm = sph.make_params(p, sph.FP64, cap, pair_tiles=tiles)
    dp = sph.DeviceParticles.from_state(s, sph.FP64)
    ws = sph.workspace(prm, s.n)
    diag = torch.zeros((max(nsteps, 1), 4), dtype=torch.float64, device="cuda")
    sph.read_interactions(ws, reset=True)
    sph.step(prm, dp, nsteps, ws, prime=True, diag=diag if nsteps else None)
    if code:
        with pytest.raises(sph.SphError) as ei:
            sph.check(ws)
        assert ei.value.code == code
    else:
        sph.check(ws)
    return dp.numpy(), sph.read_interactions(ws, reset=True), diag.cpu().numpy()


def same(a, b, fields=FIELDS):
    assert a[1] == b[1]
    for f in fields:
        assert np.array_equal(a[0][f], b[0][f]), f


@pytest.mark.parametrize("name", CASES)
@pytest.mark.parametrize("tiles,cap", [(ON, 0), (64, 0), (700, 0), (ON, 72)])
def test_tiles_fp64_bitwise_equal_to_global_lists(name, tiles, cap):
    p, s = case(name)
    s = shuffled(s, 3)
    ref = run(p, s, -1, 3)
    out = run(p, s, tiles, 3, cap)
    same(out, ref)
    assert np.abs(out[2] / ref[2] - 1)[:, 0].max() < 1e-13
    assert np.abs(out[2] - ref[2])[:, 1:].max() <= 1e-13 * np.abs(ref[2][:, 0]).max()


def test_tiles_fp64_zorder_and_standalone():
    p, s = case("cube32_cd2")
    p = p.replace(cell_order=W.Z_ORDER)
    same(run(p, s, ON, 2), run(p, s, -1, 2))
    outs = []
    for tiles in (-1, ON):
        prm = sph.make_params(p, sph.FP64, 0, pair_tiles=tiles)
        dp = sph.DeviceParticles.from_state(shuffled(s, 4), sph.FP64)
        ws = sph.workspace(prm, s.n)
        cs, ce = sph.cell_arrays(prm)
        sph.bin_sort(prm, dp, ws, cs, ce)
        sph.density(prm, dp, cs, ce, ws)
        sph.eos(prm, dp)
        sph.momentum(prm, dp, cs, ce, ws)
        outs.append(dp.numpy())
    for f in FIELDS:
        assert np.array_equal(outs[1][f], outs[0][f]), f


@pytest.mark.parametrize("out", [0.3, 0.9, 30.0, 1e6])
def test_tiles_fp64_with_particles_outside_box(out):
    """Two neighbouring particles beyond the lower x face, near (the tile
    walks whole rows) and far (the tile is left to the fallback)."""
    p, s = case("dam_cd2")
    x = s.x.copy()
    fl = np.where(s.ptype == 0)[0]
    x[:, fl[0]] = (p.lo[0] - out * p.h, x[1, fl[0]], x[2, fl[0]])
    x[:, fl[1]] = (p.lo[0] - out * p.h, x[1, fl[0]] + 0.2 * p.h, x[2, fl[0]])
    s = W.State(x, s.u, s.m, s.ptype, s.pid)
    same(run(p, s, ON, 0, code=sph.SPH_EDOMAIN), run(p, s, -1, 0, code=sph.SPH_EDOMAIN),
         ("a", "rho", "p", "id"))
