"""The record matcher's cooperative shapes against the per-lane one (itself
checked against the oracle elsewhere): identical fields and costs for every
channel count, with ragged rows, sample counts on both sides of the group of
six, and the two fields in one launch sequence or on two streams."""
import sys

import numpy as np
import pytest

from sff_inputs import params_dict

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("split", ["0", "1"])
@pytest.mark.parametrize("C", [1, 2, 3, 4])
@pytest.mark.parametrize("H,W,level,rs,B", [(37, 95, 0, 6, 1), (5, 33, 0, 5, 2), (70, 131, 1, 7, 1), (1, 1, 0, 6, 1)])
def test_record_shapes(H, W, level, rs, B, C, split, monkeypatch):
    import torch
    import paper_1710_10096_amd as sff
    rng = np.random.default_rng(H * 100 + W + C)
    p = params_dict(H, W, C, levels=2, iters=2, rs_samples=rs, fmax=16, dmax=12)
    desc = rng.integers(-4000, 4001, (B, 4, H, W, sff.desc_channels(C), 16)).astype(np.int16)
    desc[:, 1:] = np.roll(desc[:, :1], 2, axis=3) + rng.integers(-300, 301, desc[:, 1:].shape).astype(np.int16)
    n = 2 ** (level + 1)
    coarse = rng.integers(0, 13, (2, B, (H + n - 1) // n, (W + n - 1) // n, 4)).astype(np.int16)
    d, h = torch.from_numpy(desc).cuda(), torch.from_numpy(coarse).cuda()
    seeds = torch.arange(1, B + 1, dtype=torch.int64, device="cuda") * 77
    monkeypatch.setenv("SFF_MATCH_SPLIT", split)
    out = {}
    for ev in ("lane", "coop-46-32", "coop-xts", "auto"):
        monkeypatch.setenv("SFF_MATCH_EVAL", ev)
        print("[case] records", H, W, level, rs, B, C, split, ev, file=sys.stderr, flush=True)
        hyp, cost = sff.sff_match_level(p, d, sff.DIR_BOTH, level, seeds, hyp_coarse=h if level == 0 else None,
                                        **({} if level == 0 else _start(p, B, h.device)))
        torch.cuda.synchronize()
        out[ev] = hyp.cpu(), cost.cpu()
    for ev in ("coop-46-32", "coop-xts", "auto"):
        assert torch.equal(out[ev][0], out["lane"][0]) and torch.equal(out[ev][1], out["lane"][1]), ev


def _start(p, B, device):
    """A zero field at level 1 with costs above every sum: the first candidates replace it."""
    import torch
    Hk, Wk = (p["H"] + 1) // 2, (p["W"] + 1) // 2
    hyp = torch.zeros((2, B, Hk, Wk, 4), dtype=torch.int16, device=device)
    cost = torch.full((2, B, Hk, Wk), -1, dtype=torch.int32, device=device)
    return dict(hyp=hyp, cost=cost)
