"""The bin matcher's 64-pixel shapes against the per-lane one (itself checked
against the oracle): identical fields and costs for every channel count, with
ragged rows, sample counts that are no multiple of the groups, and the two fields
in one launch sequence or on two streams."""
import sys

import numpy as np
import pytest

from sff_inputs import params_dict

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("split", ["0", "1"])
@pytest.mark.parametrize("C", [1, 2, 3, 4])
@pytest.mark.parametrize("H,W,level,rs", [(37, 95, 0, 6), (5, 259, 0, 5), (70, 131, 1, 7), (1, 1, 0, 1)])
def test_bin_shapes(H, W, level, rs, C, split, monkeypatch):
    import torch
    import paper_1710_10096_amd as sff
    rng = np.random.default_rng(H * 100 + W + C)
    p = params_dict(H, W, C, levels=3, iters=2, rs_samples=rs, fmax=16, dmax=12)
    base = rng.integers(0, 256, (H, W + 8, C), dtype=np.uint8)
    imgs = np.stack([base[:, k:k + W] for k in (0, 3, 5, 8)])
    imgs = np.clip(imgs.astype(np.int64) + rng.integers(-3, 4, imgs.shape), 0, 255).astype(np.uint8)
    bins = sff.sff_wht_features(p, torch.from_numpy(imgs).cuda(), level, want_desc=False)
    n = 2 ** (level + 1)
    coarse = torch.from_numpy(rng.integers(0, 13, (2, 1, (H + n - 1) // n, (W + n - 1) // n, 4)).astype(np.int16)).cuda()
    seeds = torch.tensor([77], dtype=torch.int64, device="cuda")
    monkeypatch.setenv("SFF_MATCH_SPLIT", split)
    out = {}
    for ev in ("lane", "coop-22", "coop-43", "auto"):
        monkeypatch.setenv("SFF_MATCH_EVAL", ev)
        print("[case] bins", H, W, level, rs, C, split, ev, file=sys.stderr, flush=True)
        out[ev] = [t.cpu() for t in sff.sff_match_level_bins(p, bins, sff.DIR_BOTH, level, seeds, hyp_coarse=coarse)]
    for ev in ("coop-22", "coop-43", "auto"):
        assert torch.equal(out[ev][0], out["lane"][0]) and torch.equal(out[ev][1], out["lane"][1]), ev
