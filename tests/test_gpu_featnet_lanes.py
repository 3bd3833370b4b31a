"""GPU checks of the learned-feature helpers at the edges of their split over
lanes: triples not a multiple of a block's, and gradient buffers whose length or
address does not allow 16-byte accesses."""
import sys

import numpy as np
import pytest

from oracle import featnet as ofn

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sff():
    import torch
    import paper_1710_10096_amd as m
    assert torch.cuda.is_available()
    return m


@pytest.mark.parametrize("n,off", [(1, 0), (7, 0), (8, 0), (2049, 0), (4096, 1), (4099, 4), (32, 3)])
def test_take_grad_lengths_and_alignment(sff, n, off):
    import torch
    print("[case] take_grad", n, off, file=sys.stderr, flush=True)
    g = torch.randn(n + 8, generator=torch.Generator().manual_seed(n)).cuda()
    before = g.clone()
    out = torch.full((n + 8,), 7.0, dtype=torch.bfloat16, device="cuda")
    sff.sff_take_grad_bf16(g[off:off + n], out[off:off + n])
    ref = before.bfloat16()
    assert torch.equal(out[off:off + n], ref[off:off + n])
    assert not g[off:off + n].any()
    keep = torch.ones(n + 8, dtype=torch.bool)
    keep[off:off + n] = False
    assert torch.equal(g[keep.cuda()], before[keep.cuda()]) and bool((out[keep.cuda()] == 7.0).all())


@pytest.mark.parametrize("T", [1, 31, 32, 33, 257])
def test_triplet_counts(sff, T):
    """Loss and gradient of T triples over distinct pixels; FP32 sums of 32 terms
    after two normalisations, so 1e-5 of the largest value."""
    import torch
    print("[case] triplet", T, file=sys.stderr, flush=True)
    rng = np.random.default_rng(T)
    f = ofn.bf16_round(rng.standard_normal((3 * T, 32)))
    trip = rng.permutation(3 * T).reshape(T, 3).astype(np.int32)
    ft = torch.from_numpy(f.astype(np.float32)).to(torch.bfloat16).cuda()
    grad = torch.zeros((3 * T, 32), dtype=torch.float32, device="cuda")
    loss = sff.sff_triplet_loss(ft, torch.from_numpy(trip).cuda(), 0.5, grad, weight=0.5)
    x = torch.from_numpy(f).requires_grad_(True)
    a, p, n = (x / x.norm(dim=1, keepdim=True))[torch.from_numpy(trip.astype(np.int64)).t().contiguous()]
    ref = torch.clamp(0.5 + ((a - p) ** 2).sum(1) - ((a - n) ** 2).sum(1), min=0)
    (0.5 * ref.sum()).backward()
    assert np.abs(loss.cpu().numpy() - ref.detach().numpy()).max() <= 1e-5
    assert np.abs(grad.cpu().numpy() - x.grad.numpy()).max() <= 1e-5 * max(float(x.grad.abs().max()), 1e-3)
