"""The SGM path kernel's splits at their edges, bit-exact against the oracle:
the disparity counts where the lanes per line change, lines that end inside a
wave, lines shorter and longer than the load ring."""
import sys

import numpy as np
import pytest

import oracle
from sff_inputs import params_dict

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,W,D,P2,B", [
    (33, 45, 56, 24, 1), (33, 45, 57, 231, 1), (19, 67, 64, 24, 2), (19, 67, 65, 24, 1), (50, 9, 128, 231, 1),
    (9, 50, 129, 24, 2), (35, 38, 193, 100, 1), (16, 16, 256, 231, 1), (3, 5, 193, 24, 1), (2, 130, 72, 24, 1),
])
def test_sgm_lane_splits(H, W, D, P2, B):
    import torch
    import paper_1710_10096_amd as sff
    rng = np.random.default_rng(H * 1000 + W * 10 + D)
    left = rng.integers(0, 256, (B, H, W, 3), dtype=np.uint8)
    right = np.roll(left, -3, axis=2)
    right[:, :, :: 5] = rng.integers(0, 256, right[:, :, :: 5].shape, dtype=np.uint8)
    p = params_dict(H, W, 3, levels=1, iters=1, dmax=D - 1)
    print("[case] sgm", H, W, D, P2, B, file=sys.stderr, flush=True)
    imgs = torch.from_numpy(np.ascontiguousarray(np.stack([left, right], axis=1))).cuda()
    disp = sff.sff_sgm_disparity(p, imgs[:, 0], imgs[:, 1], 3, P2)
    torch.cuda.synchronize()
    d = disp.cpu().numpy()
    for b in range(B):
        assert np.array_equal(d[b], oracle.sgm(left[b], right[b], D, 3, P2)), b
