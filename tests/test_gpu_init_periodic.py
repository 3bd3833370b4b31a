"""GPU check of the initialisation with temporal leaves on a texture that is periodic
in 16 columns and 4 rows, its deviations growing smaller along the scan: the best
candidates of a query all fall to one lane, the candidate lists overflow scan after
scan, and the leaves are taken one by one after a bounded number; against the CPU
oracle, bit for bit."""
import sys

import numpy as np
import pytest

import oracle
from sff_inputs import params_dict

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("leaves", [2, 4])
@pytest.mark.parametrize("noise", [0, 1, 2])
def test_init_on_periodic_texture(noise, leaves):
    import torch
    import paper_1710_10096_amd as sff
    print("[case] init periodic", noise, leaves, file=sys.stderr, flush=True)
    H, W, C, F = 100, 140, 1, 64
    rng = np.random.default_rng(noise)
    a = np.tile(rng.integers(40, 200, (4, 16, C)), (H // 4, W // 16 + 1, 1))[None, :, :W].repeat(4, 0)
    a[1:] += np.linspace(40, 0, H).astype(np.int64)[None, :, None, None]
    imgs = np.clip(a + rng.integers(-noise, noise + 1, a.shape), 0, 255).astype(np.uint8)
    p = params_dict(H, W, C, levels=1, iters=1, fmax=F, dmax=16)
    bins = sff.sff_wht_features(p, torch.from_numpy(imgs).cuda(), 0, want_desc=False)
    hyp, cost = sff.sff_init_nn_bins(p, bins, 1, leaves=leaves)
    D = np.stack([oracle.features(im, 0) for im in imgs])
    for d, s in enumerate((1, -1)):
        oh, oc = oracle.init_nn(D, 0, s, F, 16, leaves=leaves)
        assert np.array_equal(hyp[d, 0].cpu().numpy(), oh)
        assert np.array_equal(cost[d, 0].cpu().numpy().view(np.uint32), oc)
