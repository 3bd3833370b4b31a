"""GPU check of the covariance's precision: no further from the exact sums of the
same FP32 descriptors than FP64 additions would bring it, for descriptors with
entries that the fixed-point digits do not hold (their products are summed in FP64)
and without.

All terms are at least zero, so a sum is off by at most one rounding (u = 2^-53) of
itself per addition: on the way of a descriptor's product there are the additions of
its block (at most the descriptors summed in FP64), 7 of the digit sums, at most
512 / 8 + 3 over the blocks, and 5 roundings to the covariance."""
import sys
from fractions import Fraction

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

U = 2.0 ** -53
BITS, DIGITS = 58, 8  # entries of these images are multiples of 2^-58 or cut there


def _images(kind, H, W, rng):
    a = rng.integers(0, 256, (4, H, W, 3))
    if kind == "smooth":
        a = sum(np.roll(a, k, 2) for k in range(5)) // 5
    elif kind == "faint":  # faint texture beside a strong edge: most descriptors have small entries
        a = 100 + rng.integers(0, 2, a.shape)
        a[:, :, W // 2:] += 150
    elif kind == "dots":
        a = np.where(rng.random((4, H, W, 1)) < 0.01, a, 100)
    return np.ascontiguousarray(a, np.uint8)


def _exact(f):
    """Sum and Gram matrix of f (float32 [N][128], in [0, 1]) as integers, scaled by 2^BITS and 2^(2 BITS)."""
    F = np.rint(f.astype(np.float64) * 2.0 ** BITS).astype(np.int64)
    total, digits = F.sum(0, dtype=object), []
    for _ in range(DIGITS):
        d = ((F + 128) & 255) - 128
        digits.append(d.astype(np.float64))
        F = (F - d) >> 8
    assert not F.any()
    G = np.zeros((128, 128), object)
    for i in range(DIGITS):
        for j in range(DIGITS):  # exact in float64: below 2^14 per descriptor
            G = G + (digits[i].T @ digits[j]).astype(np.int64).astype(object) * (1 << (8 * (i + j)))
    return total, G


@pytest.mark.parametrize("kind", ["noise", "smooth", "faint", "dots"])
@pytest.mark.parametrize("size", [(8, 8), (3, 11), (17, 37), (61, 90), (96, 160)], ids=str)
def test_covariance_as_exact_as_fp64_sums(kind, size):
    import torch
    import paper_1710_10096_amd as sff
    H, W = size
    print("[case] exact covariance", kind, size, file=sys.stderr, flush=True)
    imgs = torch.from_numpy(_images(kind, H, W, np.random.default_rng(H * 1000 + W))).cuda()
    p = dict(H=H, W=W, C=3, levels=1, iters=1, rs_r0=8, rs_samples=1, fmax=1, dmax=1, tau=1)
    out = sff.sff_sift_pca(p, imgs[None])
    f = sff.sff_dense_sift(p, imgs).cpu().numpy().reshape(-1, 128)
    N = len(f)
    small = int(((f > 0) & (f < 2.0 ** -15)).any(1).sum())
    total, G = _exact(f)
    mean, cov = out["mean"][0].cpu().numpy(), out["cov"][0].cpu().numpy()
    steps = small + 7 + 512 / 8 + 3 + 5
    cut = 2.0 ** -(BITS + 1)
    err_m = max(abs(Fraction(float(m)) - Fraction(int(t), N << BITS)) for m, t in zip(mean, total))
    assert err_m <= steps * U * mean.max() + cut, float(err_m)
    gmax = max(int(g) for g in np.diag(G)) / (N * 2.0 ** (2 * BITS))
    worst = max(abs(Fraction(float(cov[r, c])) -
                    (Fraction(int(G[r, c]), N << (2 * BITS)) - Fraction(int(total[r]) * int(total[c]), N * N << (2 * BITS))))
                for r in range(128) for c in range(128))
    assert worst <= 3 * steps * U * gmax + 2 * cut, (float(worst), gmax, small)
