"""CNN gradients of one row so wide that 32 bits do not count its FP32 activations' bytes.
Without biases a pixel far from any light has no activation and no error, so an image that
is dark but for its two ends has, but for the mean's count, the gradient of the two ends as
images of their own, which the FP64 oracle gives."""
import numpy as np
import pytest

from oracle import cnn
from gpu_util import rel_l2, say

pytestmark = pytest.mark.gpu


def test_gradient_of_a_wide_row():
    import torch
    import paper_2511_21647_amd as ulm
    W, E = (1 << 24) + 33, 96        # width; columns of an end, its outer 64 lit
    g = np.random.default_rng(24)
    p = cnn.init_params(g)
    for k in p:
        if k.startswith("b"):
            p[k] = np.zeros_like(p[k])
    flat = ulm.cnn_pack(p)
    p = {k: v.reshape(p[k].shape) for k, v in ulm.cnn_unpack(flat).items()}
    left, right = np.zeros((1, E), np.float32), np.zeros((1, E), np.float32)
    left[0, :64], right[0, -64:] = g.uniform(0, 1, 64), g.uniform(0, 1, 64)
    # lights beyond 10^6 columns are not labels, so the right end's target is dark
    mb = np.array([[0.0, 3.25], [0.2, 40.5]], np.float32)
    targets = (cnn.target_map(mb.astype(np.float64), 1, E), 0.0)
    ref, loss = {k: 0.0 for k in p}, 0.0
    for img, T in zip((left, right), targets):
        l, gr = cnn.loss_and_grad(p, img.astype(np.float64), T)
        loss += l * E / W
        for k in ref:
            ref[k] = ref[k] + gr[k] * E / W
    image = torch.zeros((1, 1, W), dtype=torch.float32, device="cuda")
    image[0, 0, :E] = torch.from_numpy(left[0]).cuda()
    image[0, 0, W - E:] = torch.from_numpy(right[0]).cuda()
    say(f"[gradients fp32 1x1x{W}]")
    lo, gr = ulm.ulm_cnn_gradients(torch.from_numpy(flat).cuda(), image, torch.from_numpy(mb).cuda(),
                                   torch.zeros(2, dtype=torch.int32, device="cuda"), ulm.ULM_CNN_FP32)
    got = ulm.cnn_unpack(gr)
    worst = max(rel_l2(got[k], ref[k]) for k in ref)
    say(f"  loss rel {abs(float(lo) - loss) / loss:.2e}, worst tensor {worst:.2e}")
    assert abs(float(lo) - loss) <= 1e-5 * loss
    assert worst <= 1e-5
