"""The weight gradient with infinite activations: exactly the entries whose sum has
the product are infinite, as in a float64 sum of the products that belong to it.
One infinity per input channel, at corners, along borders and across the rows where
a wave's share of a column ends (8 rows at these sizes, per residue of the
dilation); dy has no zeros, so no product is NaN."""
import sys

import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("case", [(1, 40, 65, 32, 1), (1, 40, 65, 3, 1), (2, 21, 33, 32, 2), (1, 37, 30, 32, 16),
                                  (1, 37, 30, 3, 3), (1, 1, 1, 32, 1), (1, 9, 64, 32, 1)], ids=str)
def test_infinite_activations(case):
    import torch
    import paper_1710_10096_amd as sff
    n, H, W, cin, dil = case
    print("[case] weight gradient, infinities", case, file=sys.stderr, flush=True)
    g = torch.Generator().manual_seed(H * 1000 + W + dil)
    for first in range(0, 64, cin):
        x = torch.randn((n, H, W, cin), generator=g).bfloat16()
        dy = torch.randn((n, H, W, 32), generator=g).bfloat16()
        dy[dy == 0] = 1
        for c in range(cin):
            k = first + c
            row = (0, H - 1, 7, 8, 15, 16, 8 * dil - 1, 8 * dil, 9 * dil, H // 2)[k % 10] % H
            col = (0, W - 1, 31, 32, W // 2, max(W - 1 - dil, 0), 33)[k % 7] % W
            x[k % n, row, col, c] = float("inf") if k % 2 else -float("inf")
        dw, db = (t.cpu() for t in sff.sff_conv3x3_bf16_wgrad(x.cuda(), dy.cuda(), dil))
        dz = dy.double().reshape(-1, 32)
        xp = torch.nn.functional.pad(x.double(), (0, 0, dil, dil, dil, dil))
        for ky in range(3):
            for kx in range(3):
                xs = xp[:, ky * dil:ky * dil + H, kx * dil:kx * dil + W].reshape(-1, cin)
                inf = xs.isinf()
                ref = dz.t() @ torch.where(inf, torch.zeros_like(xs), xs)
                # one infinity of a channel at most
                sign = dz.t().sign() @ torch.where(inf, xs.sign(), torch.zeros_like(xs))
                want = torch.where(sign != 0, sign * float("inf"), ref)
                got, fin = dw[:, ky, kx].double(), want.isfinite()
                assert torch.equal(got[~fin], want[~fin]), (first, ky, kx)
                assert got[fin].isfinite().all(), (first, ky, kx)
                mag = dz.abs().t() @ torch.where(inf, torch.zeros_like(xs), xs).abs()
                # sums of fewer than 2000 terms on any path
                assert ((got - want).abs() <= 2000 * 2.0 ** -24 * mag + 1e-12)[fin].all()
        assert db.isfinite().all()
