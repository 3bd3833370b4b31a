"""The record initialisation's packed operands (C <= 2) and column rotation
(grids of a multiple of 8 column tiles) against the bin-plane initialisation,
which takes other kernels to the same fields and costs."""
import sys

import numpy as np
import pytest

from sff_inputs import params_dict

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("leaves", [1, 2, 4])
@pytest.mark.parametrize("C", [1, 2, 3])
@pytest.mark.parametrize("H,W,fmax,B", [(13, 128, 30, 1), (21, 121, 200, 2), (5, 256, 7, 1), (9, 17, 16, 1)])
def test_packed_init(H, W, fmax, B, C, leaves):
    import torch
    import paper_1710_10096_amd as sff
    rng = np.random.default_rng(H + W + C)
    imgs = rng.integers(0, 256, (4 * B, H, W, C), dtype=np.uint8)
    imgs[0::4, :, ::2] = 0  # extreme contrast: coefficients at both ends of their range
    imgs[0::4, :, 1::2] = 255
    p = params_dict(H, W, C, levels=1, iters=1, fmax=fmax, dmax=20)
    print("[case] init", H, W, fmax, B, C, leaves, file=sys.stderr, flush=True)
    flat = torch.from_numpy(imgs).cuda()
    desc = sff.sff_wht_features(p, flat, 0).view(B, 4, H, W, sff.desc_channels(C), 16)
    bins = sff.sff_wht_features(p, flat, 0, want_desc=False)
    a = sff.sff_init_nn(p, desc, sff.DIR_BOTH, leaves=leaves)
    b = sff.sff_init_nn_bins(p, bins, B, sff.DIR_BOTH, leaves=leaves)
    torch.cuda.synchronize()
    assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1])
