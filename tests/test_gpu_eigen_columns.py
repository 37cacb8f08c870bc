"""The eigensolver's columns per wave: sizes and plane counts that choose 3, 4 and 5 (70
planes; 10 planes choose 3), against the FP64 oracle and, bit for bit, against the same
planes two at a time, which always take 3 or, from 385 frames, 4."""
from dataclasses import replace

import numpy as np
import pytest

from synth import arrays, cfg_tiny, with_frames
from oracle import clutter
from gpu_util import rel_l2, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("F,blocks", [
    (65, 35), (96, 35), (128, 35), (160, 35), (200, 35), (256, 35), (300, 35), (321, 35), (352, 35), (384, 35),
    (384, 5), (400, 9)])
def test_eigen_columns(F, blocks):
    import torch
    import paper_2511_21647_amd as ulm
    nz, nu, c = 4, 16, 5           # one Gram chunk whatever the number of planes
    cfg = with_frames(cfg_tiny(), F)
    cfg = cfg.with_(grid=replace(cfg.grid, nz=nz, nu=nu, nv=max(nu, blocks)), svd_cutoff=c)
    x = np.stack([arrays.clutter_stack(nz * nu, F, c, 300 + p, decay=0.7) for p in range(2)])
    x = np.ascontiguousarray(x.reshape(2, 1, F, nz, nu))

    def run(n_blocks):
        ctx = ulm.Context(cfg.with_(grid=replace(cfg.grid, n_blocks=n_blocks)))
        d = torch.from_numpy(np.ascontiguousarray(np.repeat(x, n_blocks, axis=1))).cuda()
        eig = ulm.svd_clutter_filter(ctx, d)
        ulm.ulm_check_status(ctx)
        return d.cpu().numpy(), eig.cpu().numpy()

    want, lam = run(1)
    got, eig = run(blocks)
    ref, _ = clutter.filter_planes(x.astype(np.complex128), c)
    say(f"[eigen columns F={F} planes={2 * blocks}] rel-L2 against the oracle {rel_l2(want, ref):.2e}")
    assert rel_l2(want, ref) <= 2e-5          # as the filter's other comparisons
    assert np.array_equal(got, np.repeat(want, blocks, axis=1))
    assert np.array_equal(eig, np.repeat(lam, blocks, axis=1))
