"""Stage 2 of many narrow slabs (unrolled by tap count) at the edges of its rule:
slab counts that leave a partial group and an empty last slab, steering angles that
give one tap (0 degrees) up to the largest count of the unrolled form and beyond it,
planes of less than and just over one tile, against the FP64 oracle on the same
stage-1 slices."""
from dataclasses import replace

import numpy as np
import pytest

from synth import arrays, cfg_tiny, with_angles, with_blocks, with_frames
from oracle import beamform
from gpu_util import rel_l2, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("blocks,nz,nu,angles", [
    (5, 64, 40, (0.0, 8.0)),            # one whole group
    (6, 65, 33, (-8.0, 0.0, 8.0)),      # a partial group, one row and column over a tile
    (13, 30, 65, (-6.0, 2.0)),          # less than a tile of rows
    (9, 70, 73, (-3.0, 0.0, 3.0)),      # the last slab has one slice
    (8, 64, 64, (-30.0, 30.0)),         # steep: more taps than the unrolled form takes
    (35, 48, 274, (-8.0, -4.0, 0.0, 4.0, 8.0))])
def test_stage2_narrow_slabs(blocks, nz, nu, angles):
    import torch
    import paper_2511_21647_amd as ulm
    cfg = with_blocks(with_angles(with_frames(cfg_tiny(), 3), angles), blocks)
    g = cfg.grid
    cfg = cfg.with_(grid=replace(g, nz=nz, nu=nu, nv=nu, dz=1e-4, u0=-(nu - 1) / 2 * g.du,
                                 v0=-(nu - 1) / 2 * g.dv),
                    seq=replace(cfg.seq, n_samp=1024))
    S = arrays.complex_normal((2, len(angles), 3, nz, nu), 900 + blocks)
    ref = beamform.stage2_project(S.astype(np.complex128), cfg)
    ctx = ulm.Context(cfg)
    ulm.ulm_stage1_slices(ctx).copy_(torch.from_numpy(S).cuda())
    got = ulm.rca_beamform_stage2(ctx)
    torch.cuda.synchronize()
    # FP32 sums of at most 2 x 274 products: 274 * 2^-24 * sqrt(terms) stays far below 1e-5
    e = rel_l2(got.cpu().numpy(), ref)
    say(f"[stage 2 B={blocks} {nz}x{nu} angles {angles}] rel-L2 {e:.2e}")
    assert e <= 1e-5
