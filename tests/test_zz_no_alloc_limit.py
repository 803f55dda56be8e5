"""The limit of sph_step_noalloc at its edge: what the static scratch takes is
counted without the sort's tables (three words per particle stand for them), so
it takes 416 particles a side of a 2D lattice and a mostly empty grid of seven
million cells, whose tables double the workspace, and refuses one more."""
import numpy as np
import pytest
import torch

import paper_1909_04504_amd as sph
import sph_workloads as W

pytestmark = pytest.mark.gpu


def case(kind, size):
    if kind == "dense":
        return W.taylor_green(size, jitter=0.2, seed=1)
    p, s = W.taylor_green(40, jitter=0.2, seed=40)
    return p.replace(hi=tuple(size * v for v in p.hi)), s


@pytest.mark.parametrize("kind,takes,refuses", [("dense", 416, 417), ("sparse", 185, 190)])
def test_noalloc_limit(kind, takes, refuses):
    prec = sph.FP32_MIXED
    p, s = case(kind, takes)
    prm = sph.make_params(p, prec)
    out = []
    for noalloc in (False, True):
        dp = sph.DeviceParticles.from_state(s, prec)
        if noalloc:
            sph.step_noalloc(prm, dp, 1, prime=True)
        else:
            ws = sph.workspace(prm, s.n)
            sph.step(prm, dp, 1, ws, prime=True)
        torch.cuda.synchronize()
        out.append(dp.numpy())
    for f in ("x", "u", "a", "rho", "p", "id"):
        assert np.array_equal(out[0][f], out[1][f]), f
    p, s = case(kind, refuses)
    with pytest.raises(sph.SphError) as ei:
        sph.step_noalloc(sph.make_params(p, prec), sph.DeviceParticles.from_state(s, prec), 1,
                         prime=True)
    assert ei.value.code == sph.SPH_EWORKSPACE
