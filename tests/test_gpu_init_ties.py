"""Several temporal leaves where many targets tie (a flat region): both
initialisations against the oracle, which keeps the smallest target indices."""
import sys

import numpy as np
import pytest

import oracle
from sff_inputs import params_dict

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("leaves", [1, 2, 4])
@pytest.mark.parametrize("H,W,C", [(45, 70, 4), (40, 33, 1), (30, 50, 3)])
def test_leaves_with_ties(H, W, C, leaves):
    import torch
    import paper_1710_10096_amd as sff
    rng = np.random.default_rng(H + W + C)
    imgs = rng.integers(0, 256, (4, H, W, C), dtype=np.uint8)
    imgs[:, H // 2:, : W // 2] = 77
    p = params_dict(H, W, C, levels=1, iters=1, fmax=70, dmax=20)
    print("[case] ties", H, W, C, leaves, file=sys.stderr, flush=True)
    flat = torch.from_numpy(imgs).cuda()
    desc = sff.sff_wht_features(p, flat, 0).view(1, 4, H, W, sff.desc_channels(C), 16)
    bins = sff.sff_wht_features(p, flat, 0, want_desc=False)
    a = [t.cpu().numpy() for t in sff.sff_init_nn(p, desc, sff.DIR_BOTH, leaves=leaves)]
    b = [t.cpu().numpy() for t in sff.sff_init_nn_bins(p, bins, 1, sff.DIR_BOTH, leaves=leaves)]
    D = [oracle.features(imgs[m], 0) for m in range(4)]
    for di, s in enumerate((1, -1)):
        oh, oc = oracle.init_nn(D, 0, s, 70, 20, leaves=leaves)
        for hyp, cost in (a, b):
            assert np.array_equal(hyp[di, 0], oh), s
            assert np.array_equal(cost[di, 0].view(np.uint32), oc), s
