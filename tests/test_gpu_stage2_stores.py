"""Stage 2 of narrow slabs on either side of the rule for its stores (rows of whole 64-byte
pieces or not, four and five transmits), against the FP64 oracle on the same slices."""
from dataclasses import replace

import numpy as np
import pytest

from synth import arrays, cfg_tiny, with_angles, with_blocks, with_frames
from oracle import beamform
from gpu_util import rel_l2, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nu,angles", [
    (16, (0.0,)), (40, (0.0,)), (48, (-4.0, 4.0)), (33, (0.0,)), (47, (-6.0, -2.0, 2.0, 6.0)),
    (50, (-8.0, -4.0, 0.0, 4.0, 8.0))])
def test_stage2_stores(nu, angles):
    import torch
    import paper_2511_21647_amd as ulm
    cfg = with_blocks(with_angles(with_frames(cfg_tiny(), 3), angles), 7)
    g = cfg.grid
    nz = 66
    cfg = cfg.with_(grid=replace(g, nz=nz, nu=nu, nv=nu, dz=1e-4, u0=-(nu - 1) / 2 * g.du,
                                 v0=-(nu - 1) / 2 * g.dv),
                    seq=replace(cfg.seq, n_samp=1024))
    S = arrays.complex_normal((2, len(angles), 3, nz, nu), 700 + nu)
    ref = beamform.stage2_project(S.astype(np.complex128), cfg)
    ctx = ulm.Context(cfg)
    ulm.ulm_stage1_slices(ctx).copy_(torch.from_numpy(S).cuda())
    got = ulm.rca_beamform_stage2(ctx)
    torch.cuda.synchronize()
    # FP32 sums of at most 5 x 8 products: 40 * 2^-24 * sqrt(terms) stays far below 1e-5
    e = rel_l2(got.cpu().numpy(), ref)
    say(f"[stage 2 stores {nz}x{nu} angles {angles}] rel-L2 {e:.2e}")
    assert e <= 1e-5
