"""The grouping of pixels by target centre behind the window cost's gradient, at
the edges of its sort tiles (2048 elements, 64 a step) and search blocks (256
cells), with scattered, identical and crowded centres.  Maps and weights are
small integers and halves, so every sum is exact in FP32 in any order and the
gradient equals the float64 oracle's."""
import sys

import numpy as np
import pytest

from oracle import cost_f32 as ocf

pytestmark = pytest.mark.gpu

# 3 H W elements: one wave step and less, around a search block, around a sort tile, several tiles
SIZES = [(1, 1), (3, 7), (1, 85), (1, 86), (11, 62), (1, 683), (31, 67)]


@pytest.mark.parametrize("kind", ["scattered", "one", "rows"])
@pytest.mark.parametrize("size", SIZES, ids=str)
def test_grouping_is_exact(size, kind):
    import torch
    import paper_1710_10096_amd as sff
    H, W = size
    rng = np.random.default_rng(H * 1000 + W)
    F = rng.integers(-3, 4, (1, 4, H, W, 4)).astype(np.float32)
    hyp = np.zeros((1, H, W, 4), np.int16)
    if kind == "scattered":
        hyp[..., :2] = rng.integers(-W, W + 1, (1, H, W, 2))
        hyp[..., 2:] = rng.integers(0, W + 1, (1, H, W, 2))
    elif kind == "one":      # every centre clamped to one corner
        hyp[..., :2] = 2000
    else:                    # every centre clamped into the first column
        hyp[..., 0] = -2000
        hyp[..., 2] = 2000
    g = rng.choice([0.5, 1.0], (1, H, W)).astype(np.float32)
    print("[case] grouping", kind, size, file=sys.stderr, flush=True)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    for s in (1, -1):
        grad = sff.sff_cost_f32_bwd(dev(F), dev(hyp), s, dev(g)).cpu().numpy()
        G = ocf.window_cost_grad([F[0, m].astype(np.float64) for m in range(4)], hyp[0], s, g[0])
        for m in range(4):
            assert np.abs(G[m]).max() < 2.0 ** 23
            assert np.array_equal(grad[0, m].astype(np.float64), G[m]), (s, m)
