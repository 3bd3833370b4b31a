"""The bin-plane initialisation with 2, 4 and 8 query rows per block (by the size of
the grid) against the record initialisation, which takes another kernel to the
same fields and costs; heights that are no multiple of the rows."""
import sys

import numpy as np
import pytest

from sff_inputs import params_dict

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("leaves", [1, 2, 4])
@pytest.mark.parametrize("H,W,C,fmax,B", [(39, 100, 1, 40, 1), (3, 17, 3, 9, 1),      # 2 rows
                                          (97, 161, 3, 50, 1), (45, 70, 4, 70, 3),    # 4 rows
                                          (203, 250, 1, 30, 1), (101, 130, 2, 30, 2)])  # 8 rows
def test_init_rows(H, W, C, fmax, B, leaves):
    import torch
    import paper_1710_10096_amd as sff
    rng = np.random.default_rng(H + W + C)
    imgs = rng.integers(0, 256, (4 * B, H, W, C), dtype=np.uint8)
    imgs[:, H // 2:, : W // 2] = 77  # equal descriptors: ties
    p = params_dict(H, W, C, levels=1, iters=1, fmax=fmax, dmax=20)
    print("[case] init rows", H, W, C, fmax, B, leaves, file=sys.stderr, flush=True)
    flat = torch.from_numpy(imgs).cuda()
    desc = sff.sff_wht_features(p, flat, 0).view(B, 4, H, W, sff.desc_channels(C), 16)
    bins = sff.sff_wht_features(p, flat, 0, want_desc=False)
    a = sff.sff_init_nn(p, desc, sff.DIR_BOTH, leaves=leaves)
    b = sff.sff_init_nn_bins(p, bins, B, sff.DIR_BOTH, leaves=leaves)
    torch.cuda.synchronize()
    assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1])
