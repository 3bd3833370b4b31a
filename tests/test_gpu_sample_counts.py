"""The matchers at every number of random-search samples around their groups of 2, 3
and 6, at the sizes where each shape is chosen (up to 50,000 updates and above,
both maps), against one lane per pixel: identical fields and costs."""
import sys

import numpy as np
import pytest

from sff_inputs import params_dict

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("maps", ["bins", "desc"])
@pytest.mark.parametrize("H,W,C", [(40, 61, 1), (40, 61, 3), (180, 300, 3), (250, 500, 2), (300, 701, 3)])
def test_sample_counts(H, W, C, maps, monkeypatch):
    import torch
    import paper_1710_10096_amd as sff
    rng = np.random.default_rng(H + W + C)
    base = rng.integers(0, 256, (H, W + 8, C), dtype=np.uint8)
    imgs = torch.from_numpy(np.stack([base[:, k:k + W] for k in (0, 3, 5, 8)])).cuda()
    hyp0 = torch.from_numpy(rng.integers(0, 13, (2, 1, H, W, 4)).astype(np.int16)).cuda()
    seeds = torch.tensor([77], dtype=torch.int64, device="cuda")
    monkeypatch.delenv("SFF_MATCH_SPLIT", raising=False)
    for rs in range(17):
        p = params_dict(H, W, C, levels=1, iters=1, rs_samples=rs, fmax=16, dmax=12)
        feats = sff.sff_wht_features(p, imgs, 0, want_desc=maps == "desc")
        if maps == "desc":
            feats = (feats[0] if isinstance(feats, tuple) else feats).view(1, 4, H, W, -1, 16)
        run = sff.sff_match_level_bins if maps == "bins" else sff.sff_match_level
        print("[case] sample counts", H, W, C, maps, rs, file=sys.stderr, flush=True)
        out = {}
        for ev in ("auto", "lane"):
            monkeypatch.setenv("SFF_MATCH_EVAL", ev)
            hyp, cost = hyp0.clone(), torch.full((2, 1, H, W), -1, dtype=torch.int32, device="cuda")
            run(p, feats, sff.DIR_BOTH, 0, seeds, hyp, cost)
            out[ev] = hyp, cost
        assert all(torch.equal(a, b) for a, b in zip(out["auto"], out["lane"])), rs
