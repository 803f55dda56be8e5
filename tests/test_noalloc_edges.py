"""What sph_step_noalloc takes and refuses at the edge of its limit, which is
counted without the sort's tables (two words per cell and six per particle):
mostly empty grids of eight million cells, and FP64 calls that ask for tiles on
them.  Without a device the call still tells a refused size (workspace) from one
that it takes (no device); on one, the largest sizes it takes run and agree with
the oracle."""
import ctypes

import numpy as np
import pytest
import torch

import oracle
import paper_1909_04504_amd as sph
import sph_workloads as W

LIMIT = 64 << 20


def thin_plane(size):
    """1,600 particles on a plane of (size * 15.38)^2 cells."""
    p, s = W.taylor_green(40, jitter=0.2, seed=40)
    return p.replace(hi=tuple(size * v for v in p.hi)), s


def thin_box(n, cells=200):
    """n particles in a corner of cells^3 whole cells."""
    p, s = W.periodic_cube(n_side=10, jitter=0.2)
    p = p.replace(cell_div=1, periodic=(0, 0, 0))
    cell = (3 if p.kernel == W.QUINTIC else 2) * p.h
    p = p.replace(hi=tuple(p.lo[k] + cells * cell * (1 + 1e-9) for k in range(3)))
    return p, W.State(s.x[:, :n].copy(), s.u[:, :n].copy(), s.m[:n].copy(), s.ptype[:n].copy(),
                      s.pid[:n].copy())


# (state, precision, pair_tiles, taken)
EDGES = [(lambda: thin_plane(185), sph.FP32_MIXED, 0, True),
         (lambda: thin_plane(186), sph.FP32_MIXED, 0, True),
         (lambda: thin_plane(187), sph.FP32_MIXED, 0, True),
         (lambda: thin_plane(188), sph.FP32_MIXED, 0, False),
         (lambda: thin_plane(186), sph.FP64, 0, True),
         (lambda: thin_box(1000), sph.FP32_MIXED, 0, True),
         (lambda: thin_box(100), sph.FP64, 0, True),
         (lambda: thin_box(1000), sph.FP64, 2000, True),
         (lambda: thin_box(1000, 205), sph.FP32_MIXED, 0, False)]


@pytest.mark.skipif(torch.cuda.is_available(), reason="the arrays of the call are not real ones")
@pytest.mark.parametrize("state,prec,tiles,taken", EDGES)
def test_limit_without_device(state, prec, tiles, taken):
    p, s = state()
    prm = sph.make_params(p, prec, pair_tiles=tiles)
    c = sph.Particles()
    c.n = s.n
    for k in range(3):
        c.x[k] = c.u[k] = c.a[k] = 4096  # never read: there is no device
    c.rho = c.p = c.m = c.type = c.id = c.arho = 4096
    rc = sph.lib().sph_step_noalloc(ctypes.byref(prm), ctypes.byref(c), 1, 1, None, None)
    assert rc == (sph.SPH_EDEVICE if taken else sph.SPH_EWORKSPACE)
    if not taken:  # the message names a need above what is there
        words = sph.lib().sph_last_error().decode().replace(",", "").split()
        need, have = [int(w) for w in words if w.isdigit()]
        assert need > have == LIMIT


@pytest.mark.gpu
@pytest.mark.parametrize("state,prec,tiles,taken", EDGES)
def test_limit_on_device(state, prec, tiles, taken):
    p, s = state()
    prm = sph.make_params(p, prec, pair_tiles=tiles)
    dp = sph.DeviceParticles.from_state(s, prec)
    if not taken:
        with pytest.raises(sph.SphError) as ei:
            sph.step_noalloc(prm, dp, 1, prime=True)
        assert ei.value.code == sph.SPH_EWORKSPACE
        return
    sph.step_noalloc(prm, dp, 2, prime=True)
    torch.cuda.synchronize()
    out = dp.numpy()
    _, perm, _, _ = oracle.bin_sort(p, out["x"])
    assert out["x"].shape[1] == s.n
    ref = oracle.step(p, s.x, s.u, s.m, s.ptype, 2)
    o, tol = np.argsort(out["id"]), 1e-12 if prec == sph.FP64 else 1e-4
    assert np.array_equal(out["id"][o], np.sort(s.pid))
    for f in ("x", "u", "a"):
        got, want = out[f][:, o].astype(np.float64), ref[f][:, np.argsort(s.pid)]
        assert np.abs(got - want).max() <= tol * np.abs(want).max(), f
    # the order is the sort's of the step's positions (drifted once more by none)
    assert np.array_equal(perm, np.arange(s.n))
