"""CNN gradients at each number of rows per wave (8 down to 1 by the images' rows and the
precision) and with rows split into column segments, against the FP64 oracle: heights that
leave a wave's band, and widths that leave a segment, partly empty."""
import numpy as np
import pytest

from oracle import cnn
from gpu_util import rel_l2, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec,B,H,W", [
    ("fp32", 43, 33, 65), ("fp32", 40, 33, 65), ("fp32", 20, 33, 65), ("fp32", 3, 13, 70), ("fp32", 1, 3, 700),
    ("bf16", 12, 33, 65), ("bf16", 10, 33, 65), ("bf16", 5, 33, 65), ("bf16", 6, 13, 70), ("bf16", 2, 9, 700)])
def test_gradient_bands(prec, B, H, W):
    import torch
    import paper_2511_21647_amd as ulm
    g = np.random.default_rng(100 * B + H + W)
    p = cnn.init_params(g)
    for k in p:
        if k.startswith("b"):
            p[k] = p[k] + 0.05 * g.standard_normal(p[k].shape)
    flat = ulm.cnn_pack(p)
    p = {k: v.reshape(p[k].shape) for k, v in ulm.cnn_unpack(flat).items()}
    distinct = min(B, 6)                 # the oracle's images; the batch repeats them
    imgs = g.uniform(0, 1, (distinct, H, W)).astype(np.float32)
    mbs = [np.stack([g.uniform(0, H - 1, 4), g.uniform(0, W - 1, 4)], 1).astype(np.float32)
           for _ in range(distinct)]
    images = np.stack([imgs[n % distinct] for n in range(B)])
    zu = np.concatenate([mbs[n % distinct] for n in range(B)])
    img = np.repeat(np.arange(B), 4).astype(np.int32)
    ref, loss = {k: 0.0 for k in p}, 0.0
    for n in range(distinct):
        share = len(range(n, B, distinct)) / B
        l, gr = cnn.loss_and_grad(p, imgs[n].astype(np.float64), cnn.target_map(mbs[n].astype(np.float64), H, W))
        loss += share * l
        for k in ref:
            ref[k] = ref[k] + share * gr[k]
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    lo, gr = ulm.ulm_cnn_gradients(dev(flat), dev(images), dev(zu), dev(img),
                                   ulm.ULM_CNN_FP32 if prec == "fp32" else ulm.ULM_CNN_BF16)
    got = ulm.cnn_unpack(gr)
    # as the other gradient comparisons: FP32 rounding in another order, and 8-bit
    # mantissas of every stored activation
    tol = 1e-5 if prec == "fp32" else 1e-2
    worst = max(rel_l2(got[k], ref[k]) for k in ref)
    say(f"[gradient bands {prec} {B}x{H}x{W}] loss rel {abs(float(lo) - loss) / loss:.2e}, worst tensor {worst:.2e}")
    assert abs(float(lo) - loss) <= tol * loss
    assert worst <= tol
