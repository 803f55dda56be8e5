"""GPU tests of the tiled build of the global-format lists (3D) and of the CSR
lists formed from stored lists: sph_neighbors gives entry for entry the lists
of the cell walks (no tiles, no stored lists), whatever the staging and list
capacities; the continuity scheme's fields over tiled lists are bitwise those
over walked ones."""
import numpy as np
import pytest
import torch

import paper_1909_04504_amd as sph
import sph_workloads as W
from helpers import shuffled
from test_gpu_tiles import CASES, ON, case


def csr(p, s, prec, cap, tiles):
    prm = sph.make_params(p, prec, cap, pair_tiles=tiles)
    dp = sph.DeviceParticles.from_state(s, prec)
    ws = sph.workspace(prm, s.n)
    cs, ce = sph.cell_arrays(prm)
    sph.bin_sort(prm, dp, ws, cs, ce)
    off = torch.zeros(s.n + 1, dtype=torch.int64, device="cuda")
    with pytest.raises(sph.SphError) as ei:
        sph.neighbors(prm, dp, cs, ce, 0, off, None, ws)
    assert ei.value.code == sph.SPH_ECAPACITY
    nbr = torch.full((ei.value.total,), -1, dtype=torch.int32, device="cuda")
    assert sph.neighbors(prm, dp, cs, ce, nbr.numel(), off, nbr, ws) == nbr.numel()
    return off.cpu().numpy(), nbr.cpu().numpy()


@pytest.mark.gpu
@pytest.mark.parametrize("prec", [sph.FP64, sph.FP32_MIXED])
@pytest.mark.parametrize("name", CASES)
def test_neighbors_from_tiled_lists_equal_walks(name, prec):
    p, s = case(name)
    s = shuffled(s, 8)
    off, nbr = csr(p, s, prec, -1, -1)  # walks
    mid = int(np.median(np.diff(off)))
    # staging for every union, for some and for none; lists for every count,
    # for about half of them (odd to the octets), and of one row
    for cap, tiles in ((0, ON), (0, 700), (0, 64), (mid, ON), (4, ON), (0, -1), (mid, -1)):
        o, q = csr(p, s, prec, cap, tiles)
        assert np.array_equal(o, off), (cap, tiles)
        assert np.array_equal(q, nbr), (cap, tiles)


@pytest.mark.gpu
@pytest.mark.parametrize("prec", [sph.FP64, sph.FP32_MIXED])
def test_neighbors_from_lists_2d_and_zorder(prec):
    p, s = W.taylor_green(33, jitter=0.3, seed=5)
    off, nbr = csr(p, s, prec, -1, -1)
    for cap in (0, int(np.median(np.diff(off)))):
        o, q = csr(p, s, prec, cap, 0)
        assert np.array_equal(o, off) and np.array_equal(q, nbr)
    p, s = case("cube32_cd2")
    p = p.replace(cell_order=W.Z_ORDER)
    off, nbr = csr(p, s, prec, -1, -1)
    o, q = csr(p, s, prec, 0, ON)
    assert np.array_equal(o, off) and np.array_equal(q, nbr)


@pytest.mark.gpu
@pytest.mark.parametrize("prec", [sph.FP64, sph.FP32_MIXED])
@pytest.mark.parametrize("name", ["cube32_cd2", "dam_cd2", "dam_cd1"])
def test_continuity_fields_over_tiled_lists(name, prec):
    p, s = case(name)
    p = p.replace(scheme=W.CONTINUITY)
    rho = p.rho0 * (1 + 1e-3 * np.random.default_rng(3).standard_normal(s.n))
    outs = []
    for tiles in (-1, ON, 64):
        prm = sph.make_params(p, prec, 0, pair_tiles=tiles)
        dp = sph.DeviceParticles(s.x, s.u, s.m, s.ptype, s.pid, prec, rho=rho, scheme=sph.CONTINUITY)
        ws = sph.workspace(prm, s.n)
        sph.step(prm, dp, 2, ws, prime=True)
        sph.check(ws)
        outs.append((dp.numpy(), sph.read_interactions(ws)))
    for o, inter in outs[1:]:
        assert inter == outs[0][1]
        for f in ("x", "u", "a", "rho", "p", "id", "arho"):
            assert np.array_equal(o[f], outs[0][0][f]), f
