"""Clutter filter where the Gram's pixel chunks are shorter than the usual 2048 (small
planes, few frames): one chunk, a last chunk of one pixel, the shortest chunk, and the
sizes on either side of a halving, in both precisions, against the FP64 oracle."""
from dataclasses import replace

import numpy as np
import pytest

from synth import arrays, cfg_tiny, with_frames
from oracle import clutter
from gpu_util import rel_l2, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["fp64", "bf16x3"])
@pytest.mark.parametrize("F,nz,nu,c", [
    (5, 7, 9, 2), (20, 5, 13, 2), (33, 16, 128, 4), (64, 1, 2049, 3), (65, 64, 257, 5),
    (20, 129, 127, 2)])
def test_filter_short_chunks(F, nz, nu, c, precision):
    import torch
    import paper_2511_21647_amd as ulm
    cfg = with_frames(cfg_tiny(), F)
    if nu > 550:                         # a plane this flat, the other way round
        nz, nu = nu, nz
    cfg = cfg.with_(grid=replace(cfg.grid, nz=nz, nu=nu, nv=nu), svd_cutoff=c)
    x = np.stack([arrays.clutter_stack(nz * nu, F, c, 40 + o, decay=0.5) for o in range(2)])
    x = np.ascontiguousarray(x.reshape(2, 1, F, nz, nu))
    ref, lam = clutter.filter_planes(x.astype(np.complex128), c)
    ctx = ulm.Context(cfg, precision=ulm.ULM_PREC_BF16X3 if precision == "bf16x3" else ulm.ULM_PREC_FP64GRAM)
    d = torch.from_numpy(x).cuda()
    eig = ulm.svd_clutter_filter(ctx, d)
    ulm.ulm_check_status(ctx)
    e = rel_l2(d.cpu().numpy(), ref)
    el = np.abs(eig.cpu().numpy() - lam).max() / lam.max()
    say(f"[filter chunks {precision} F={F} {nz}x{nu} c={c}] rel-L2 {e:.2e}, eigenvalues {el:.2e}")
    # the tolerances of the filter's other comparisons
    assert e <= (2e-5 if precision == "fp64" else 1e-3)
    assert el <= (1e-10 if precision == "fp64" else 1e-6)


@pytest.mark.parametrize("F", [1, 16, 17, 48, 49, 64, 80, 81, 96, 112, 113, 128, 145])
def test_filter_gram_tiles(F):
    """The FP64 Gram's tile shares: every number of 16-frame tiles in the last block, on and
    off the diagonal."""
    test_filter_short_chunks(F, 16, 33, min(F, 3), "fp64")
