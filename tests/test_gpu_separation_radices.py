"""MB separation with every radix of the two-pass form that the other size tests leave out,
as both passes of a frame count (10, 12, 14, 18 and 21 twice, 24 beside 20) and beside a
prime, against the oracle."""
from dataclasses import replace

import numpy as np
import pytest

from synth import arrays, cfg_tiny, with_blocks, with_frames
from oracle import separation
from gpu_util import rel_l2, say

pytestmark = pytest.mark.gpu

TOL = 1e-5          # relative L2 per subset, as the other comparisons


@pytest.mark.parametrize("F,nz,nu,S", [
    (12, 5, 7, 2), (20, 3, 11, 1), (36, 4, 8, 3), (63, 3, 11, 2), (64, 2, 16, 4), (100, 5, 13, 3),
    (144, 4, 9, 2), (196, 3, 11, 3), (256, 2, 17, 3), (324, 3, 11, 2), (441, 4, 8, 1), (480, 3, 11, 3),
    (486, 1, 33, 2), (490, 2, 16, 3), (504, 3, 5, 2)])
def test_separation_radices(F, nz, nu, S):
    import torch
    import paper_2511_21647_amd as ulm
    cfg = with_blocks(with_frames(cfg_tiny(), F), 1)
    cfg = cfg.with_(grid=replace(cfg.grid, nz=nz, nu=nu, nv=max(nu, 2)))
    ctx = ulm.Context(cfg)
    x = arrays.complex_normal(ctx.proj_shape, seed=131 + F)
    out = torch.full((2 * S,) + tuple(ctx.proj_shape), float("nan"), dtype=torch.complex64, device="cuda")
    got = ulm.ulm_separate(ctx, torch.from_numpy(x).cuda(), S, out).cpu().numpy()
    ref = separation.separate(x.astype(np.complex128), S)
    assert np.isfinite(got).all()
    worst = max(rel_l2(got[i], ref[i]) for i in range(2 * S))
    say(f"[separation radices F={F} {nz}x{nu} S={S}] worst subset rel-L2 {worst:.2e}")
    assert worst <= TOL
