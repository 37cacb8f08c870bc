"""Low-rank planes at frame counts where the split-precision form's solver met a reflector
too small for its reciprocals, and in the solver of more than 512 frames: finite, and the
clutter gone."""
from dataclasses import replace

import numpy as np
import pytest

from synth import cfg_tiny, with_angles, with_frames
from gpu_util import say
from test_gpu_static_scene import KINDS, _planes

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("F,precision", [(254, "bf16x3"), (336, "bf16x3"), (369, "bf16x3"), (387, "bf16x3"),
                                         (388, "bf16x3"), (389, "bf16x3"), (520, "fp64"), (601, "fp64")])
def test_static_planes_finite(F, precision):
    import torch
    import paper_2511_21647_amd as ulm
    nz, nu, c, B = 7, 9, 3, len(KINDS)
    cfg = with_angles(with_frames(cfg_tiny(), F), [0])
    cfg = cfg.with_(grid=replace(cfg.grid, nz=nz, nu=nu, nv=nu, n_blocks=B), svd_cutoff=c)
    g = np.random.default_rng(F)
    smalls = (1e-30, 1e-20) if precision == "fp64" else (1e-12, 1e-12)
    x = np.stack([np.stack([_planes(k, F, nz * nu, g, s) for k in KINDS]) for s in smalls])
    x = x.astype(np.complex64).reshape(2, B, F, nz, nu)
    ctx = ulm.Context(cfg, ulm.ULM_PREC_BF16X3 if precision == "bf16x3" else ulm.ULM_PREC_FP64GRAM)
    d = torch.from_numpy(x).cuda()
    eig = ulm.svd_clutter_filter(ctx, d)
    ulm.ulm_check_status(ctx)
    got = d.cpu().numpy()
    assert np.isfinite(got).all() and torch.isfinite(eig).all()
    left = max(np.linalg.norm(got[o, b].astype(complex)) / np.linalg.norm(x[o, b].astype(complex))
               for o in range(2) for b in range(B))
    say(f"[static planes F={F} {precision}] left over {left:.1e}")
    assert left <= (2e-5 if precision == "fp64" else 1e-3)
