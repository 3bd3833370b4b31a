"""GPU check of the principal axes on covariances whose spectrum falls steeply
(images that are flat in part, stripes, single dots, a flat image), where a power
of the covariance keeps only the first vector, and on ordinary ones, against
float64 eigenvalues of the same covariance.

The iteration stops at residuals of 1e-12 of the largest eigenvalue and the direct
solution errs by a few ulp of it (an eigenvalue is within its vector's residual of
a true one); 2e-12 of the norm leaves room for evaluating them.  Unit length and
orthogonality hold to 128 roundings."""
import sys

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _images(kind, H, W, rng):
    a = rng.integers(0, 256, (4, H, W, 3))
    if kind.startswith("sky"):  # texture below, a saturated part above
        a[:, :H * int(kind[3:]) // 100] = 255
    elif kind == "stripes":
        s = 128 + 100 * np.sin(np.arange(W) * 0.7)[None, None, :, None]
        a = np.clip(s + rng.integers(-3, 4, a.shape), 0, 255)
    elif kind == "ramp":  # one descriptor everywhere: a covariance of rounding errors
        a = np.broadcast_to((np.arange(W) * 2 % 256)[None, None, :, None], a.shape)
    elif kind == "edge":  # flat but for one edge: a covariance of low rank
        a = np.full_like(a, 90)
        a[:, :, W // 2:] = 200
    elif kind == "dot":
        a = np.full_like(a, 90)
        a[:, H // 2, W // 2] = 200
    elif kind == "flat":
        a = np.full_like(a, 7)
    return np.ascontiguousarray(a, np.uint8)


@pytest.mark.parametrize("kind", ["noise", "sky10", "sky40", "sky90", "stripes", "ramp", "edge", "dot", "flat"])
@pytest.mark.parametrize("size", [(16, 20), (97, 150)], ids=str)
def test_axes_of_any_spectrum(kind, size):
    import torch
    import paper_1710_10096_amd as sff
    H, W = size
    print("[case] axes", kind, size, file=sys.stderr, flush=True)
    rng = np.random.default_rng(H * 1000 + W)
    imgs = torch.from_numpy(np.stack([_images(kind, H, W, rng), _images("noise", H, W, rng)])).cuda()
    p = dict(H=H, W=W, C=3, levels=1, iters=1, rs_r0=8, rs_samples=1, fmax=1, dmax=1, tau=1)
    out = {k: v.cpu().numpy() for k, v in sff.sff_sift_pca(p, imgs).items()}
    for b in range(2):
        cov, axes, eig = out["cov"][b], out["axes"][b], out["eigval"][b]
        lam = np.linalg.eigvalsh(cov)[::-1]
        tol = 2e-12 * np.abs(lam).max()
        assert np.abs(axes @ axes.T - np.eye(3)).max() < 1e-10
        assert np.abs(eig - lam[:3]).max() <= tol, (eig, lam[:3])
        assert np.linalg.norm(axes @ cov - eig[:, None] * axes, axis=1).max() <= tol
        assert all(a[np.argmax(np.abs(a))] > 0 for a in axes)
        f = sff.sff_dense_sift(p, imgs[b]).cpu().numpy().astype(np.float64)
        d = f - out["mean"][b].astype(np.float32)
        # 128 products and sums in FP32 of terms below |axis| |d|, axes rounded to FP32
        assert np.abs(out["phi"][b][..., :3] - d @ axes.T).max() <= 200 * 2.0 ** -24 * np.linalg.norm(d, axis=-1).max() + 1e-30
