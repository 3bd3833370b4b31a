"""GPU check of the covariance of the dense SIFT descriptors, which is summed from
fixed-point digits on the int8 matrix cores, against float64 products of the
same FP32 descriptors.

An entry is rounded to a multiple of 2^-38 (exact from 2^-15 on) and products of
its digits below 2^-52 are dropped: the mean is within 2^-39 and a product of two
entries (at most 1) within 2^-38 + 2^-44 of the exact one, and so are their means;
the covariance subtracts a product of means within 2^-38.  8e-12 bounds the sum."""
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


def _images(kind, H, W, rng):
    a = rng.integers(0, 256, (4, H, W, 3))
    if kind == "dots":      # isolated pixels: descriptors with few, large entries
        a = np.where(rng.random((4, H, W, 1)) < 0.01, a, 100)
    elif kind == "ramp":    # the same gradient everywhere
        a = np.broadcast_to((np.arange(W) * 2 % 256)[None, None, :, None], a.shape)
    elif kind == "faint":   # one strong edge beside faint texture: small entries
        a = 100 + rng.integers(0, 2, a.shape)
        a[:, :, W // 2:] += 150
    return np.ascontiguousarray(a, np.uint8)


# one descriptor step (128) and less, one more, several blocks with a ragged end, many steps per block
SIZES = [(1, 1), (4, 8), (3, 11), (16, 16), (17, 37), (97, 150), (200, 331)]


@pytest.mark.parametrize("kind", ["noise", "dots", "ramp", "faint"])
@pytest.mark.parametrize("size", SIZES, ids=str)
def test_covariance_of_fixed_point_digits(sff, kind, size):
    import torch
    H, W = size
    print("[case] covariance", kind, size, file=sys.stderr, flush=True)
    imgs = torch.from_numpy(_images(kind, H, W, np.random.default_rng(H * 1000 + W))).cuda()
    p = dict(H=H, W=W, C=3, levels=1, iters=1, rs_r0=8, rs_samples=1, fmax=1, dmax=1, tau=1)
    out = sff.sff_sift_pca(p, torch.stack([imgs, imgs.flip(2)]))
    for b, im in enumerate((imgs, imgs.flip(2).contiguous())):
        f = sff.sff_dense_sift(p, im).double().reshape(-1, 128)
        mean = f.mean(0)
        cov = f.t().contiguous() @ f / f.shape[0] - mean[:, None] * mean[None]
        assert float((out["mean"][b] - mean).abs().max()) <= 2.0 ** -38
        assert float((out["cov"][b] - cov).abs().max()) <= 8e-12
        assert torch.equal(out["cov"][b], out["cov"][b].t())
