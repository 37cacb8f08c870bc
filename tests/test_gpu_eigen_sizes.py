"""Clutter filter over the eigensolver's sizes against the FP64 oracle: either side of each
change of work-group shape (20/21 and 32/33 frames: columns per wave of one work-group;
64/65: one work-group or several; 384/385: columns per wave), of a row block (128/129), the
smallest and largest sizes, more planes than XCDs, no cutoff and the largest; and both
exchange modes between work-groups, bit for bit."""
from dataclasses import replace

import numpy as np
import pytest

from synth import arrays, cfg_tiny, with_frames
from oracle import clutter
from gpu_util import say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("F,blocks,c", [
    (1, 1, 1), (2, 1, 0), (3, 1, 3), (20, 5, 2), (21, 1, 4), (32, 1, 32), (33, 5, 2), (64, 1, 32), (65, 1, 0),
    (65, 5, 3), (128, 1, 5), (129, 5, 4), (300, 1, 32), (384, 1, 2), (385, 1, 3), (512, 5, 2)])
def test_eigen_sizes(F, blocks, c, monkeypatch):
    import torch
    import paper_2511_21647_amd as ulm
    nz, nu = 16, 40
    cfg = with_frames(cfg_tiny(), F)
    cfg = cfg.with_(grid=replace(cfg.grid, nz=nz, nu=nu, nv=nu, n_blocks=blocks), svd_cutoff=c)
    x = np.stack([arrays.clutter_stack(nz * nu, F, max(c, 1), 70 + p, decay=0.85) for p in range(2 * blocks)])
    x = np.ascontiguousarray(x.reshape(2, blocks, F, nz, nu))
    ref, lam = clutter.filter_planes(x.astype(np.complex128), c)
    out = []
    for fenced in (False, True):
        if fenced:
            monkeypatch.setenv("ULMPROJ_EIGEN_AGENT_SCOPE", "1")
        else:
            monkeypatch.delenv("ULMPROJ_EIGEN_AGENT_SCOPE", raising=False)
        ctx = ulm.Context(cfg)
        d = torch.from_numpy(x).cuda()
        eig = ulm.svd_clutter_filter(ctx, d)
        ulm.ulm_check_status(ctx)
        out.append((d.cpu().numpy(), eig.cpu().numpy()))
    # relative to the input where every mode is removed
    scale = np.linalg.norm(x if c == F else ref)
    e = np.linalg.norm((out[0][0] - ref).ravel()) / scale
    el = np.abs(out[0][1] - lam).max() / lam.max()
    say(f"[eigen sizes F={F} planes={2 * blocks} c={c}] rel-L2 {e:.2e}, eigenvalues {el:.2e}")
    # the tolerances of the filter's other comparisons
    assert e <= 2e-5
    assert el <= 1e-10
    assert np.array_equal(out[0][0], out[1][0])
    assert np.array_equal(out[0][1], out[1][1])
