"""The network's forward pass and its records on both sides of the sizes where they
change between one launch and layer by layer: the same bits."""
import sys

import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dil", [1, 2])
@pytest.mark.parametrize("n,H,W", [(1, 3, 5), (3, 97, 161), (1, 300, 501), (2, 399, 540), (1, 601, 719)])
def test_routes_agree(n, H, W, dil):
    import torch
    import paper_1710_10096_amd as sff
    from paper_1710_10096_amd.featnet import FeatNet
    print("[case] network routes", n, H, W, dil, file=sys.stderr, flush=True)
    net = FeatNet(seed=3, device="cuda")
    g = torch.Generator().manual_seed(H)
    x = torch.randn((n, H, W, 3), generator=g).bfloat16().cuda()
    wb = net.weights_bf16()
    want, acts = net.forward(x, dil, keep=True, wb=wb)
    assert torch.equal(net.forward(x, dil, wb=wb), want)
    desc = torch.empty((n, H, W, 2, 16), dtype=torch.int16, device="cuda")
    assert torch.equal(net.records(x, dil, 4096.0, desc, wb=wb), sff.sff_quantise_features(want, 4096.0))
