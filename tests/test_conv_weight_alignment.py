"""Weights at an address that is no multiple of 16 bytes: the records call, whose
kernel reads them in 16-byte pieces, refuses them as it refuses such inputs; the
forward takes its element-wise kernel, with the same results."""
import sys

import pytest

from paper_1710_10096_amd import _native
from .test_abi import host_only


@host_only
@pytest.mark.parametrize("off", [2, 4, 8])
def test_records_refuse_unaligned_weights(off):
    L, at = _native.lib(), 1 << 20  # addresses that are never read: refused on the host
    INVALID = 1
    assert L.sff_conv3x3_bf16_records(1, 8, 8, 1, at, at + off, None, 4096.0, at, None) == INVALID
    assert L.sff_conv3x3_bf16_records(1, 8, 8, 1, at + off, at, None, 4096.0, at, None) == INVALID


@pytest.mark.gpu
@pytest.mark.parametrize("off", [1, 4])
def test_forward_takes_unaligned_weights(off):
    import torch
    import paper_1710_10096_amd as sff
    print("[case] unaligned weights", off, file=sys.stderr, flush=True)
    g = torch.Generator().manual_seed(off)
    x = torch.randn((2, 19, 37, 32), generator=g).bfloat16().cuda()
    w = (torch.randn(32 * 9 * 32, generator=g) / 17).bfloat16().cuda()
    moved = torch.zeros(w.numel() + 8, dtype=torch.bfloat16, device="cuda")
    moved[off:off + w.numel()] = w
    moved = moved[off:off + w.numel()].view(32, 3, 3, 32)
    w = w.view(32, 3, 3, 32)
    assert moved.data_ptr() % 16 and w.data_ptr() % 16 == 0
    assert torch.equal(sff.sff_conv3x3_bf16_fwd(x, moved, None, 2, True), sff.sff_conv3x3_bf16_fwd(x, w, None, 2, True))
    assert torch.equal(sff.sff_conv3x3_bf16_dgrad(x, moved, 2, None), sff.sff_conv3x3_bf16_dgrad(x, w, 2, None))
    with pytest.raises(Exception):
        sff.sff_conv3x3_bf16_records(x, moved, None, 2)
