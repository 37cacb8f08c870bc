"""Clutter filter where covariances have equal eigenvalues in decoupled parts: more modes
removed than the planes' rank (zeros), frames that light one pixel each (all equal, in two
groups where frames outnumber pixels), and planes of zeros.  The removal is a projection of
the top modes' energy: |planes|^2 - |filtered|^2 is the sum of the largest eigenvalues, and
the filtered planes are orthogonal to what was removed."""
from dataclasses import replace

import numpy as np
import pytest

from synth import cfg_tiny, with_angles, with_frames
from gpu_util import say

pytestmark = pytest.mark.gpu

KINDS = ("static", "rank5", "integers5", "three_phases", "one_hot", "few_frames", "one_pixel", "zeros")


def _planes(kind, F, npix, g):
    field = lambda *s: g.standard_normal(s) + 1j * g.standard_normal(s)
    x = np.zeros((F, npix), complex)
    if kind == "static":
        x[:] = field(1, npix)
    elif kind == "rank5":
        x = field(F, 5) @ field(5, npix)
    elif kind == "integers5":
        x = np.round(field(F, 5)) @ np.round(field(5, npix))
    elif kind == "three_phases":
        x = np.exp(2j * np.pi * np.outer(np.arange(F), np.arange(npix) % 3) / F)
    elif kind == "one_hot":
        x[np.arange(F), np.arange(F) % npix] = 2
    elif kind == "few_frames":
        x[:6] = field(6, npix)[:F]
    elif kind == "one_pixel":
        x[:, npix // 3] = 1 + 1j
    return x


@pytest.mark.parametrize("precision", ["fp64", "bf16x3"])
@pytest.mark.parametrize("F,c", [(8, 8), (20, 20), (21, 8), (33, 32), (50, 20), (65, 32), (128, 20), (150, 4), (200, 32),
                                 (300, 20), (384, 32), (512, 20), (516, 32)])
def test_equal_eigenvalues(F, c, precision):
    import torch
    import paper_2511_21647_amd as ulm
    nz, nu, B = 9, 12, len(KINDS)
    cfg = with_angles(with_frames(cfg_tiny(), F), [0])
    cfg = cfg.with_(grid=replace(cfg.grid, nz=nz, nu=nu, nv=nu, n_blocks=B), svd_cutoff=c)
    g = np.random.default_rng(F + c)
    p = np.stack([_planes(k, F, nz * nu, g) for k in KINDS]).astype(np.complex64)
    ctx = ulm.Context(cfg, ulm.ULM_PREC_BF16X3 if precision == "bf16x3" else ulm.ULM_PREC_FP64GRAM)
    d = torch.from_numpy(np.ascontiguousarray(np.stack([p, p]).reshape(2, B, F, nz, nu))).cuda()
    eig = ulm.svd_clutter_filter(ctx, d)
    ulm.ulm_check_status(ctx)
    q, lam = d.cpu().numpy().reshape(2, B, F, -1).astype(complex), eig.cpu().numpy()
    assert np.isfinite(q).all() and np.isfinite(lam).all()
    p = p.astype(complex)
    worst = 0.0
    for b in range(B):
        w = np.linalg.eigvalsh(p[b] @ p[b].conj().T)[::-1]
        if w[0] == 0:
            assert not q[:, b].any()
            continue
        for o in range(2):
            kept = (np.abs(q[o, b]) ** 2).sum()
            worst = max(worst, abs((np.abs(p[b]) ** 2).sum() - kept - w[:c].sum()) / w[0],
                        abs(np.vdot(q[o, b], p[b]).real - kept) / w[0])
    say(f"[equal eigenvalues F={F} c={c} {precision}] energy and projection {worst:.1e} of the largest")
    # sums over up to 512 modes' FP32-rounded planes (2^-24 each, one-sided at worst: 3e-5)
    assert worst <= 4e-5
