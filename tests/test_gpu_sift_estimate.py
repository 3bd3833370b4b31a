"""GPU checks of the matching half-step that compares candidates by estimated
costs (the default) against the per-lane one that sums every candidate exactly
(SFF_SIFT_EVAL=lane), bit for bit, on features chosen against the estimate: ties
(few distinct values, constant maps), values whose squares are subnormal, values
near the largest float, infinities and NaN; and at the edges of its tiles (4
rows, 64 pixels of a colour)."""
import sys

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sff():
    import torch
    import paper_1710_10096_amd as m
    assert torch.cuda.is_available()
    return m


def _features(kind, H, W, rng):
    a = rng.standard_normal((1, 4, H, W, 3)).astype(np.float32)
    if kind == "ties":
        a = rng.integers(0, 3, a.shape).astype(np.float32)
    elif kind == "constant":
        a[:] = 0.25
    elif kind == "tiny":
        a *= np.float32(1e-21) * (10.0 ** rng.integers(0, 4, a.shape)).astype(np.float32)
    elif kind == "huge":
        a *= np.float32(1e19)
    elif kind == "nan":
        a[rng.random(a.shape) < 0.01] = np.nan
        a[rng.random(a.shape) < 0.01] = np.inf
    elif kind == "close":  # sums that differ by less than the estimate can tell
        a = (1.0 + rng.integers(0, 2, a.shape) * 2.0 ** -20).astype(np.float32)
        a[0, 0] = 0.0
    return np.concatenate([a, np.zeros(a.shape[:-1] + (1,), np.float32)], -1)


KINDS = ["normal", "ties", "constant", "tiny", "huge", "nan", "close"]
SIZES = [(1, 1), (5, 127), (4, 128), (9, 131), (37, 261)]


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("size", SIZES, ids=str)
def test_estimated_half_step_same_as_exact(sff, kind, size, monkeypatch):
    import torch
    H, W = size
    print("[case] sift estimate", kind, size, file=sys.stderr, flush=True)
    rng = np.random.default_rng(H * 1000 + W)
    phi = torch.from_numpy(_features(kind, H, W, rng)).cuda()
    p = dict(H=H, W=W, C=3, levels=1, iters=3, rs_r0=8, rs_samples=5, fmax=20, dmax=16, tau=1)
    h0 = np.stack([rng.integers(-20, 21, (2, 1, H, W)), rng.integers(-20, 21, (2, 1, H, W)),
                   rng.integers(0, 17, (2, 1, H, W)), rng.integers(0, 17, (2, 1, H, W))], -1).astype(np.int16)
    seeds = torch.tensor([5], dtype=torch.int64, device="cuda")
    out = {}
    for mode in ("", "lane"):
        monkeypatch.setenv("SFF_SIFT_EVAL", mode)
        h = torch.from_numpy(h0).cuda()
        c = sff.sff_match_sift(p, phi, seeds, h)
        out[mode] = (h, c.view(torch.int32))
    assert torch.equal(out[""][0], out["lane"][0])
    nan = out[""][1].view(torch.float32).isnan() & out["lane"][1].view(torch.float32).isnan()
    assert bool(((out[""][1] == out["lane"][1]) | nan).all())
