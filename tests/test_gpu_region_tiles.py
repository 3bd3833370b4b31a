"""Region filter at the edges of its 16 x 64 tiles, bit-exact against the oracle:
fields whose joins are not transitive (vectors within tau of one neighbour and not
of the next), snakes one pixel wide, and pixel rows and columns on either side of
a tile border."""
import sys

import numpy as np
import pytest

import oracle
from sff_inputs import params_dict

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", ["ramps", "snake", "comb"])
@pytest.mark.parametrize("H,W", [(16, 64), (17, 65), (33, 130), (64, 63), (15, 200)])
def test_region_tile_borders(H, W, kind):
    import torch
    import paper_1710_10096_amd as sff
    rng = np.random.default_rng(H * W)
    y, x = np.indices((H, W))
    hyp = np.zeros((2, H, W, 4), np.int16)
    valid = np.ones((2, H, W), np.uint8)
    if kind == "ramps":
        hyp[..., 0] = rng.integers(0, 4, (2, H, W))
        valid[:] = rng.random((2, H, W)) < 0.93
    elif kind == "snake":  # rows joined at alternating ends
        valid[:] = (y % 2 == 0) | (x == np.where(y % 4 == 1, W - 1, 0))
    else:  # columns hanging from one row, on either side of every border
        valid[:] = (y == 0) | (x % 2 == 0)
        valid[1] = valid[1, ::-1, ::-1]
    hyp[..., 2] = rng.integers(0, 2, (2, H, W))
    print("[case] region", kind, H, W, file=sys.stderr, flush=True)
    p = params_dict(H, W, 1, levels=1, iters=1, tau=1)
    for s_c in (4, H * W):
        keep = sff.sff_region_filter(p, torch.from_numpy(hyp).cuda(), torch.from_numpy(valid).cuda(), s_c).cpu().numpy()
        for b in range(2):
            assert np.array_equal(keep[b], oracle.region_filter(hyp[b], valid[b], 1, s_c)), (s_c, b)
