"""The network's last layer written as descriptor records: the same int16 values as
the layer and sff_quantise_features one after the other, at ragged sizes, every
dilation the matcher uses, all-zero and very small and large features."""
import sys

import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("gain", [1.0, 0.0, 1e-15, 1e12])
@pytest.mark.parametrize("n,H,W,dil", [(1, 1, 1, 1), (2, 7, 17, 1), (4, 33, 65, 2), (1, 70, 130, 4), (1, 5, 16, 8)])
def test_layer_records(n, H, W, dil, gain):
    import torch
    import paper_1710_10096_amd as sff
    print("[case] records", n, H, W, dil, gain, file=sys.stderr, flush=True)
    g = torch.Generator(device="cuda").manual_seed(H * W + dil)
    x = torch.relu(torch.randn((n, H, W, 32), generator=g, device="cuda")).to(torch.bfloat16)
    w = (gain * 0.1 * torch.randn((32, 3, 3, 32), generator=g, device="cuda")).to(torch.bfloat16)
    b = gain * torch.randn((32,), generator=g, device="cuda")
    f = sff.sff_conv3x3_bf16_fwd(x, w, b, dil, relu=False)
    want = sff.sff_quantise_features(f, 4096.0)
    got = sff.sff_conv3x3_bf16_records(x, w, b, dil, 4096.0)
    torch.cuda.synchronize()
    assert torch.equal(got, want)
