"""CNN gradients at the edges of the training kernels' tiles, against the FP64 oracle:
images narrower and just wider than a 32-pixel strip, fewer and just more rows than a
wave's or a work-group's band, single rows and columns, more strips than work-groups,
and a last 32-pixel chunk of the head that is partly empty."""
import numpy as np
import pytest

from oracle import cnn
from gpu_util import rel_l2, say

pytestmark = pytest.mark.gpu


SMALL = [(1, 40), (40, 1), (8, 32), (9, 33)]
SHAPES = ([("fp32", 2, h, w) for h, w in SMALL] + [("bf16", 48, h, w) for h, w in SMALL]
          + [(p, b, h, w) for p in ("fp32", "bf16") for b, h, w in [(1, 33, 31), (3, 32, 65), (70, 34, 66)]])


@pytest.mark.parametrize("prec,B,H,W", SHAPES)
def test_gradient_shapes(prec, B, H, W):
    import torch
    import paper_2511_21647_amd as ulm
    g = np.random.default_rng(1000 * B + 10 * H + W)
    p = cnn.init_params(g)
    for k in p:
        if k.startswith("b"):
            p[k] = p[k] + 0.05 * g.standard_normal(p[k].shape)
    flat = ulm.cnn_pack(p)
    p = {k: v.reshape(p[k].shape) for k, v in ulm.cnn_unpack(flat).items()}
    # the large batch of larger images repeats three, so the oracle runs three; the small
    # images are all distinct, because BF16's rounding errors average out over pixels only
    distinct = min(B, 3 if H * W > 400 else 48)
    imgs = g.uniform(0, 1, (distinct, H, W)).astype(np.float32)
    mbs = [np.stack([g.uniform(0, H - 1, 3), g.uniform(0, W - 1, 3)], 1).astype(np.float32)
           for _ in range(distinct)]
    images = np.stack([imgs[n % distinct] for n in range(B)])
    zu = np.concatenate([mbs[n % distinct] for n in range(B)])
    img = np.repeat(np.arange(B), 3).astype(np.int32)
    ref, loss = {k: 0.0 for k in p}, 0.0
    for n in range(distinct):
        share = len(range(n, B, distinct)) / B
        T = cnn.target_map(mbs[n].astype(np.float64), H, W)
        l, gr = cnn.loss_and_grad(p, imgs[n].astype(np.float64), T)
        loss += share * l
        for k in ref:
            ref[k] = ref[k] + share * gr[k]
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    pr = ulm.ULM_CNN_FP32 if prec == "fp32" else ulm.ULM_CNN_BF16
    lo, gr = ulm.ulm_cnn_gradients(dev(flat), dev(images), dev(zu), dev(img), pr)
    got = ulm.cnn_unpack(gr)
    # the tolerances of the other gradient comparison: FP32 rounding in another order, and
    # 8-bit mantissas of every stored activation
    tol = 1e-5 if prec == "fp32" else 1e-2
    worst = max(rel_l2(got[k], ref[k]) for k in ref)
    say(f"[gradients {prec} {B}x{H}x{W}] loss rel {abs(float(lo) - loss) / loss:.2e}, worst tensor {worst:.2e}")
    assert abs(float(lo) - loss) <= tol * loss
    assert worst <= tol
