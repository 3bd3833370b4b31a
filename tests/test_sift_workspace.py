"""The SIFT features' workspace: in proportion to the pixels for small pairs and
batches of them (host only), and a pair's results independent of its batch."""
import ctypes
import sys

import numpy as np
import pytest

from paper_1710_10096_amd import _native
from paper_1710_10096_amd._native import SffParams
from sff_inputs import params_dict


def _bytes(H, W, nimg):
    p = SffParams(**params_dict(H, W, 3, levels=1, iters=1))
    return _native.lib().sff_sift_workspace_bytes(ctypes.byref(p), nimg)


@pytest.mark.parametrize("batch", [1, 16])
@pytest.mark.parametrize("H,W", [(96, 160), (97, 161), (200, 300), (375, 1242)])
def test_workspace_in_proportion(H, W, batch):
    """Per pair: 32 B per cell of the planes, 4 B per descriptor, a partial of 36 * 256 + 128
    doubles per 768 descriptors, and half a megabyte of matrices."""
    bound = 4 * (H + 9) * (W + 9) * 32 + 4 * H * W * (4 + (36 * 256 + 128) * 8 / 768) + 2 ** 19
    assert 0 < _bytes(H, W, 4 * batch) <= batch * bound + 2 ** 18


@pytest.mark.gpu
def test_batch_of_five_same_as_alone():
    import torch
    import paper_1710_10096_amd as sff
    H, W = 45, 83
    rng = np.random.default_rng(5)
    imgs = torch.from_numpy(rng.integers(0, 256, (5, 4, H, W, 3), dtype=np.uint8)).cuda()
    imgs[3, :, :20] = 255  # its spectrum takes the direct solution
    p = params_dict(H, W, 3, levels=1, iters=1)
    print("[case] sift features, batch 5", file=sys.stderr, flush=True)
    out = sff.sff_sift_pca(p, imgs)
    for b in range(5):
        one = sff.sff_sift_pca(p, imgs[b:b + 1].contiguous())
        for k in ("mean", "cov", "eigval", "axes", "phi"):
            assert torch.equal(out[k][b], one[k][0]), (k, b)
