"""Clutter filter of planes whose covariance has low rank exactly, where what the
eigensolver's reduction leaves over shrinks by rounding at every step down to where squares
and reciprocals leave the double range: identical frames (constant, random, very small and
large ones), two alternating frames, a single bright pixel, one frame or pixel that differs.
The eigenvalues are the oracle's and the clutter is gone."""
from dataclasses import replace

import numpy as np
import pytest

from synth import cfg_tiny, with_angles, with_frames
from oracle import clutter
from gpu_util import say

pytestmark = pytest.mark.gpu


def _planes(kind, F, npix, g, small=1e-30):
    def field(*shape):
        return g.standard_normal(shape) + 1j * g.standard_normal(shape)
    base = field(1, npix)
    x = np.repeat(base, F, axis=0)
    if kind == "ones":
        x = np.ones((F, npix), complex)
    elif kind == "small":
        x = x * small
    elif kind == "large":
        x = x * 1e15
    elif kind == "two":
        x = np.where(np.arange(F)[:, None] % 2 == 0, base, field(1, npix))
    elif kind == "pixel":
        x = np.zeros((F, npix), complex)
        x[:, npix // 2] = 3 - 2j
    elif kind == "phase":
        x = base * np.array([1, 1j, -1, -1j])[np.arange(F) % 4][:, None]
    elif kind == "one_frame":
        x[F // 2] *= 2
    elif kind == "ramp":
        x = base * (1.0 + np.arange(F)[:, None])
    return x


KINDS = ("ones", "random", "small", "large", "two", "pixel", "phase", "one_frame", "ramp")


@pytest.mark.parametrize("precision", ["fp64", "bf16x3"])
@pytest.mark.parametrize("F", [2, 3, 5, 16, 20, 33, 50, 64, 65, 100, 129, 200, 300, 385, 512, 513])
def test_static_planes(F, precision):
    import torch
    import paper_2511_21647_amd as ulm
    nz, nu, c = 13, 16, min(3, F)
    cfg = with_angles(with_frames(cfg_tiny(), F), [0])
    # every kind in a plane of its own; the second orientation holds them in reverse
    B = len(KINDS)
    cfg = cfg.with_(grid=replace(cfg.grid, nz=nz, nu=nu, nv=nu, n_blocks=B), svd_cutoff=c)
    g = np.random.default_rng(F)
    # the split form's products are FP32: their squares have to stay in its range
    x = np.stack([_planes(k, F, nz * nu, g, 1e-30 if precision == "fp64" else 1e-12) for k in KINDS])
    x = np.stack([x, x[::-1]]).astype(np.complex64).reshape(2, B, F, nz, nu)
    ctx = ulm.Context(cfg, ulm.ULM_PREC_BF16X3 if precision == "bf16x3" else ulm.ULM_PREC_FP64GRAM)
    d = torch.from_numpy(np.ascontiguousarray(x)).cuda()
    eig = ulm.svd_clutter_filter(ctx, d)
    ulm.ulm_check_status(ctx)
    got, lam = d.cpu().numpy(), eig.cpu().numpy()
    assert np.isfinite(got).all() and np.isfinite(lam).all()
    worst = [0.0, 0.0]
    for o in range(2):
        for b in range(B):
            _, want = clutter.filter_planes(x[o:o + 1, b:b + 1].astype(np.complex128), c)
            top = want.max()
            worst[0] = max(worst[0], np.abs(lam[o, b] - want.ravel()).max() / top)
            worst[1] = max(worst[1], np.linalg.norm(got[o, b].astype(complex)) / np.linalg.norm(x[o, b].astype(complex)))
    say(f"[static planes F={F} {precision}] eigenvalues {worst[0]:.1e}, left over {worst[1]:.1e}")
    # every kind has rank at most two: nothing but rounding is left.  The tolerances of the
    # filter's other comparisons (of the split form's against the planes: 2^-24 per term)
    assert worst[0] <= (1e-10 if precision == "fp64" else 1e-6)
    assert worst[1] <= (2e-5 if precision == "fp64" else 1e-3)
