"""GPU checks of the initialisation with temporal leaves where its candidate lists
are at their limits: images whose distances tie (constant, two grey levels,
periodic), so that lists overflow with equal keys and the leaves are taken one by
one, and grids with fewer candidates than leaves; against the CPU oracle, bit for
bit.  Both dense (n = 1) and coarse (n = 4) grids."""
import sys

import numpy as np
import pytest

import oracle
from sff_inputs import params_dict

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sff():
    import torch
    import paper_1710_10096_amd as m
    assert torch.cuda.is_available()
    return m


def _images(kind, H, W, C, rng):
    a = rng.integers(0, 256, (4, H, W, C))
    if kind == "constant":
        a[:] = 77
    elif kind == "two":
        a = rng.integers(0, 2, (4, H, W, C)) * 255
    elif kind == "periodic":
        t = rng.integers(0, 256, (8, 8, C))
        a = np.broadcast_to(np.tile(t, (H // 8 + 1, W // 8 + 1, 1))[:H, :W], a.shape)
    elif kind == "blocks":  # flat areas: a few distinct patches, many equal ones
        a = np.repeat(np.repeat(rng.integers(0, 3, (4, H // 16 + 1, W // 16 + 1, C)) * 100, 16, 1), 16, 2)[:, :H, :W]
    elif kind == "far":  # bright references, dark targets: keys above 2^24 (C = 4)
        a = rng.integers(0, 4, (4, H, W, C))
        a[0], a[3] = 255 - a[0], 255 - a[3]
    return np.ascontiguousarray(a, np.uint8)


CASES = [("constant", 40, 50, 1, 1), ("constant", 70, 90, 3, 3), ("two", 33, 47, 1, 1), ("periodic", 40, 60, 3, 1),
         ("periodic", 96, 130, 2, 3), ("blocks", 60, 70, 3, 1), ("blocks", 100, 120, 4, 3), ("noise", 1, 2, 1, 1),
         ("noise", 1, 3, 3, 1), ("noise", 5, 9, 3, 3),
         ("far", 24, 40, 4, 1)]


@pytest.mark.parametrize("leaves", [1, 2, 4])
@pytest.mark.parametrize("case", CASES, ids=str)
def test_init_lists(sff, case, leaves):
    import torch
    kind, H, W, C, levels = case
    print("[case] init lists", case, leaves, file=sys.stderr, flush=True)
    imgs = _images(kind, H, W, C, np.random.default_rng(H + W))
    p = params_dict(H, W, C, levels=levels, iters=1, fmax=24, dmax=16)
    dev = torch.from_numpy(imgs).cuda()
    bins = sff.sff_wht_features(p, dev, levels - 1, want_desc=False)
    hyp, cost = sff.sff_init_nn_bins(p, bins, 1, leaves=leaves)
    D = np.stack([oracle.features(im, levels - 1) for im in imgs])
    for d, s in enumerate((1, -1)):
        oh, oc = oracle.init_nn(D, levels - 1, s, 24, 16, leaves=leaves)
        assert np.array_equal(hyp[d, 0].cpu().numpy(), oh)
        assert np.array_equal(cost[d, 0].cpu().numpy().view(np.uint32), oc)
