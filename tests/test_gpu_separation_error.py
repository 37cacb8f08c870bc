"""MB separation's error against 64 bits in its two-pass form: no larger than that of the
plain mixed-radix transform (radices 4, 2, 3, 5, 7 in turn, every constant and twiddle one
float, the sums as fused operations), which the table holds for white noise and three speed
ranges, from an emulation in FP32 on the host."""
from dataclasses import replace

import numpy as np
import pytest

from synth import arrays, cfg_tiny, with_frames
from oracle import separation
from gpu_util import say

pytestmark = pytest.mark.gpu

PLAIN = {36: 1.054e-7, 60: 1.265e-7, 80: 1.164e-7, 120: 1.306e-7, 150: 1.418e-7, 200: 1.349e-7,
         240: 1.355e-7, 300: 1.492e-7, 324: 1.501e-7, 360: 1.414e-7, 400: 1.436e-7, 480: 1.447e-7,
         512: 1.416e-7}


@pytest.mark.parametrize("F", sorted(PLAIN))
def test_separation_error(F):
    import torch
    import paper_2511_21647_amd as ulm
    cfg = with_frames(cfg_tiny(), F)
    cfg = cfg.with_(grid=replace(cfg.grid, nz=24, nu=32, nv=32))
    ctx = ulm.Context(cfg)
    x = arrays.complex_normal(ctx.proj_shape, seed=17 + F)
    got = ulm.ulm_separate(ctx, torch.from_numpy(x).cuda(), 3).cpu().numpy().astype(np.complex128)
    ref = separation.separate(x.astype(np.complex128), 3)
    err = np.linalg.norm(got - ref) / np.linalg.norm(ref)
    say(f"[separation error F={F}] {err:.3e}, the plain transform's {PLAIN[F]:.3e}")
    assert err <= PLAIN[F]
