"""XZ/YZ pairing at each number of threads per (plane, frame) range: few, some and many
ranges, of more records than lanes, some out of row order and some empty: identical to the
oracle's pairs."""
import numpy as np
import pytest

from synth import cfg_tiny, plane_records, with_blocks, with_frames
from oracle import pairing
from gpu_util import say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("frames,blocks,per_frame", [(1, 1, 1500), (128, 1, 300), (129, 1, 40), (129, 8, 160)])
def test_pairing_range_threads(frames, blocks, per_frame):
    import torch
    import paper_2511_21647_amd as ulm
    cfg = with_blocks(with_frames(cfg_tiny(), frames), blocks)
    cfg = cfg.with_(svd_cutoff=1)
    g = cfg.grid
    recs, _ = plane_records(g.nz, g.nv, blocks, frames, per_frame, 41 + frames)
    rng = np.random.default_rng(frames)
    recs = recs[recs["frame"] % 11 != 5]                       # empty frames
    key = recs["plane"].astype(np.int64) * frames + recs["frame"]
    # in every seventh frame two records of a range change places, in every ninth all are shuffled
    tie = np.arange(len(recs), dtype=float)
    for k in np.unique(key):
        at = np.nonzero(key == k)[0]
        if k % 7 == 3 and len(at) > 1:
            tie[at[-1]], tie[at[-2]] = tie[at[-2]], tie[at[-1]]
        elif k % 9 == 4:
            tie[at] = rng.permutation(tie[at])
    recs = recs[np.lexsort((tie, key))]
    want = pairing.pair_localisations(recs, blocks, g.nv)
    locs = torch.from_numpy(np.ascontiguousarray(recs).view(np.int32).reshape(-1, 8).copy()).cuda()
    cnt = torch.tensor([len(recs)], dtype=torch.int32, device="cuda")
    ctx = ulm.Context(cfg)
    out, oc = ulm.ulm_pair_planes(ctx, locs, cnt, len(recs), 2 * len(recs))
    torch.cuda.synchronize()
    got = ulm.loc3d_to_numpy(out, oc)
    say(f"[pairing ranges F={frames} B={blocks}] {len(recs)} records, {len(want)} pairs")
    assert len(got) == len(want) and len(want) > 0
    for f in ("frame", "idx_xz", "idx_yz"):
        assert np.array_equal(got[f], want[f])
