"""MB separation over the frame counts' two-radix splits against the oracle: the smallest,
even and uneven splits, every base radix twice in one factor, one work-group row shorter
than the others' (large second radix), the largest counts, and the counts without a split;
planes of one pixel, of a whole number of work-groups and of one pixel more."""
from dataclasses import replace

import numpy as np
import pytest

from synth import arrays, cfg_tiny, with_blocks, with_frames
from oracle import separation
from gpu_util import rel_l2, say

pytestmark = pytest.mark.gpu

TOL = 1e-5          # relative L2 per subset, as the other comparisons


@pytest.mark.parametrize("F,nz,nu,blocks,S", [
    (4, 8, 9, 1, 1), (6, 4, 8, 1, 2), (7, 5, 13, 1, 3), (25, 3, 11, 2, 8), (49, 16, 16, 1, 2), (81, 7, 11, 1, 3),
    (105, 1, 33, 1, 4), (125, 2, 16, 1, 1), (245, 5, 7, 1, 3), (300, 9, 11, 2, 3), (343, 3, 11, 1, 2),
    (375, 1, 65, 1, 5), (405, 2, 16, 1, 2), (448, 3, 11, 1, 3), (500, 1, 32, 1, 2), (512, 1, 17, 2, 8)])
def test_separation_sizes(F, nz, nu, blocks, S):
    import torch
    import paper_2511_21647_amd as ulm
    cfg = with_blocks(with_frames(cfg_tiny(), F), blocks)
    if nz < nu and nz < 4:              # flat planes, the other way round
        nz, nu = nu, nz
    cfg = cfg.with_(grid=replace(cfg.grid, nz=nz, nu=nu, nv=max(nu, 2)))
    ctx = ulm.Context(cfg)
    x = arrays.complex_normal(ctx.proj_shape, seed=81 + F)
    out = torch.full((2 * S,) + tuple(ctx.proj_shape), float("nan"), dtype=torch.complex64, device="cuda")
    got = ulm.ulm_separate(ctx, torch.from_numpy(x).cuda(), S, out).cpu().numpy()
    ref = separation.separate(x.astype(np.complex128), S)
    assert np.isfinite(got).all()
    errs = [rel_l2(got[i], ref[i]) for i in range(2 * S) if np.linalg.norm(ref[i]) > 0]
    say(f"[separation sizes F={F} {nz}x{nu} B={blocks} S={S}] worst subset rel-L2 {max(errs):.2e}")
    assert max(errs) <= TOL
    for i in range(2 * S):
        if np.linalg.norm(ref[i]) == 0:            # an empty speed range gives zeros
            assert np.all(got[i] == 0)
