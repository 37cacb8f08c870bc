"""NCC localiser at the edges of its band and batch shapes: bands of 14, 22 and 38
rows (chosen by the number of images), last bands of one row, planes of one and of
just over one group of eight columns, every template size, values too small for the
fast root, and an empty frame, against the FP64 oracle's localiser."""
from dataclasses import replace

import numpy as np
import pytest

from synth import arrays, cfg_tiny, with_frames
from oracle import localize
from gpu_util import compare_detections, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("F,nz,nu,size,scale", [
    (1, 14, 6, 3, 1.0), (2, 15, 7, 5, 1.0), (1, 1, 70, 7, 1.0), (2, 29, 62, 9, 1.0),
    (1, 28, 56, 13, 1.0), (1, 43, 114, 15, 1.0), (1, 17, 400, 3, 1.0), (2, 30, 40, 9, 1e-16),
    (350, 50, 14, 7, 1.0), (512, 39, 16, 9, 1.0)])
def test_ncc_band_edges(F, nz, nu, size, scale):
    import torch
    import paper_2511_21647_amd as ulm
    # speckle fills the windows of the widest templates, so little of it reaches 0.5 there
    cfg = with_frames(cfg_tiny(), F)
    cfg = cfg.with_(grid=replace(cfg.grid, nz=nz, nu=nu, nv=nu), svd_cutoff=0,
                    loc=replace(cfg.loc, ncc_size=size, tau_ncc=0.5 if size < 13 else 0.1))
    # a few speckle fields, moved from frame to frame so that no two frames are equal
    base = [arrays.speckle_field(nz, nu, 100 * nz + nu + k, smooth=1.0) for k in range(4)]
    x = np.zeros((2, 1, F, nz, nu), dtype=np.complex64)
    for o in range(2):
        for f in range(F):
            a = np.roll(base[(2 * o + f) % 4], (f % max(nz, 1), (3 * f) % nu), axis=(0, 1))
            x[o, 0, f] = (scale / np.abs(a).max()) * a
    if F == 2:
        x[1, 0, 1] = 0.0
    ora, N, I = localize.localize(x.astype(np.complex128), cfg)
    ctx = ulm.Context(cfg)
    d = torch.from_numpy(x).cuda()
    locs, cnt = ulm.ncc_localize(ctx, d, capacity=1 << 18)
    ulm.ulm_check_status(ctx, cnt, 1 << 18)
    got = ulm.locs_to_numpy(locs, cnt)
    # the tolerances of the localiser's other comparisons: decisions within 1e-4 of a
    # threshold are not compared, positions to 1e-3 pixel
    n, nund, err = compare_detections(got, ora, N, I, cfg, delta=1e-4, pos_tol=1e-3)
    say(f"[ncc bands F={F} {nz}x{nu} size {size} scale {scale}] matched {n}, undecidable {nund}, "
        f"max pos err {err:.2e}")
    assert n > 0
    # a short output list holds the first records of the whole one
    cap = max(1, len(got) // 2)
    short, cnt2 = ulm.ncc_localize(ctx, d, capacity=cap)
    torch.cuda.synchronize()
    assert int(cnt2.item()) == len(got)
    assert (ulm.locs_to_numpy(short, cap) == got[:cap]).all()
