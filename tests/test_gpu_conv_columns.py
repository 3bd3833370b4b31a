"""GPU checks of the 32-channel convolution by pixel columns at the edges of its
split: columns of 16 pixels, chunks of rows per wave (4 or more), the residues
of the dilation, and masks with every kind of bf16 value.  The im2col kernel
(SFF_CONV_IM2COL=1) issues the same MFMAs on the same values, so the results
agree bit for bit."""
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


CASES = [(1, 1, 1, 1), (1, 4, 16, 1), (1, 5, 17, 1), (2, 3, 15, 2), (1, 9, 64, 3), (1, 33, 65, 5),
         (3, 17, 80, 16), (1, 130, 33, 4), (2, 375, 400, 1)]


@pytest.mark.parametrize("case", CASES, ids=str)
def test_column_kernel_same_as_im2col(sff, case, monkeypatch):
    import torch
    n, H, W, dil = case
    print("[case] conv columns", case, file=sys.stderr, flush=True)
    g = torch.Generator().manual_seed(H * 1000 + W + dil)
    x = torch.randn((n, H, W, 32), generator=g).bfloat16()
    w = (torch.randn((32, 3, 3, 32), generator=g) / 17).bfloat16()
    b = torch.randn(32, generator=g)
    # masks: positive, zero, negative zero, negative, infinities, NaNs, the smallest subnormals
    vals = np.array([0x3F80, 0, 0x8000, 0xBF80, 0x7F80, 0xFF80, 0x7FC0, 0xFFC0, 0x7F81, 0x0001, 0x8001, 0x7F7F],
                    np.uint16).view(np.int16)
    m = torch.from_numpy(vals)[torch.randint(0, len(vals), (n, H, W, 32), generator=g)].view(torch.bfloat16)
    x, w, b, m = x.cuda(), w.cuda(), b.cuda(), m.contiguous().cuda()

    def all_three():
        return (sff.sff_conv3x3_bf16_fwd(x, w, b, dil, True), sff.sff_conv3x3_bf16_fwd(x, w, None, dil, False),
                sff.sff_conv3x3_bf16_dgrad(x, w, dil, m), sff.sff_conv3x3_bf16_dgrad(x, w, dil, None))

    monkeypatch.delenv("SFF_CONV_IM2COL", raising=False)
    got = all_three()
    monkeypatch.setenv("SFF_CONV_IM2COL", "1")
    for a, r in zip(got, all_three()):
        assert torch.equal(a.view(torch.int16), r.view(torch.int16))


WGRAD_CASES = [(1, 1, 1, 3, 1), (1, 8, 32, 32, 1), (1, 9, 33, 32, 1), (2, 7, 31, 3, 2), (1, 40, 65, 32, 9),
               (1, 35, 64, 32, 16), (3, 20, 100, 3, 5), (2, 375, 400, 32, 1), (2, 375, 400, 3, 1), (300, 9, 250, 32, 1)]


@pytest.mark.parametrize("case", WGRAD_CASES, ids=str)
def test_weight_gradient_columns(sff, case):
    """Columns of 32 pixels, chunks of 8 or more rows, residues of the dilation
    and (last case) more columns than waves, against float64 on the same values.
    An FP32 sum of N terms in any order is within N 2^-24 of the sum of their
    magnitudes; the chains here (a wave's rows, its MFMAs of 32 products, 8 waves,
    up to 32 + 8 block partials) are below 2000 terms long."""
    import torch
    n, H, W, cin, dil = case
    print("[case] weight gradient", case, file=sys.stderr, flush=True)
    g = torch.Generator().manual_seed(H * 1000 + W + dil)
    x = torch.randn((n, H, W, cin), generator=g).bfloat16().cuda()
    dy = torch.randn((n, H, W, 32), generator=g).bfloat16().cuda()
    m = torch.randn((n, H, W, 32), generator=g).bfloat16().cuda()
    dw, db = sff.sff_conv3x3_bf16_wgrad(x, dy, dil, m)
    dz = torch.where(m > 0, dy, torch.zeros_like(dy)).double().reshape(-1, 32).t().contiguous()
    xp = torch.nn.functional.pad(x.double(), (0, 0, dil, dil, dil, dil))
    for ky in range(3):
        for kx in range(3):
            xs = xp[:, ky * dil:ky * dil + H, kx * dil:kx * dil + W].reshape(-1, cin)
            ref, mag = dz @ xs, dz.abs() @ xs.abs()
            assert ((dw[:, ky, kx].double() - ref).abs() <= 2000 * 2.0 ** -24 * mag + 1e-12).all()
    assert ((db.double() - dz.sum(1)).abs() <= 2000 * 2.0 ** -24 * dz.abs().sum(1) + 1e-12).all()
