"""The network's forward pass in one call against the same layers called one
by one: the output and everything kept for the backward pass must be the same
bits."""
import pytest
import torch

from paper_2211_03160_amd import nn

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("chans,shape", [((32,), (3, 5, 7)), ((32, 64), (8, 34, 34)), ((16, 48), (1, 2, 6)),
                                         ((32, 64, 128), (2, 12, 20)), ((16, 16, 32, 32), (1, 8, 24))])
def test_forward_is_its_layers(chans, shape):
    net = nn.UNet(cin=16, cout=16, chans=chans, seed=4)
    g = torch.Generator(device="cuda")
    g.manual_seed(1)
    for lay in net.layers:
        lay["b"].copy_(0.1 * torch.randn(lay["co"], generator=g, device="cuda"))
    x = nn.to_bf16(torch.randn(*shape, 16, generator=g, device="cuda"))
    y, tape = net.forward(x)
    want, h, k, skips, levels = [], x, 0, [], len(chans)
    for lvl in list(range(levels)) + list(range(levels - 2, -1, -1)):
        if k >= 2 * levels:
            h = nn.upsample2_concat(h, skips[lvl])
        elif lvl:
            h = nn.avgpool2(h)
        for _ in range(2):
            lay = net.layers[k]
            out = nn.conv3x3(h, lay["wbf"], lay["b"], lay["co"], True)
            want.append((h, k, out))
            h, k = out, k + 1
        skips.append(h)
    lay = net.layers[k]
    assert torch.equal(y, nn.conv3x3(h, lay["wbf"], lay["b"], lay["co"], False))
    assert tape[-1][1] == k and tape[-1][2] is None and torch.equal(tape[-1][0], h) and len(tape) == k + 1
    for (h0, k0, y0), (h1, k1, y1) in zip(want, tape):
        assert k0 == k1 and torch.equal(h0, h1) and torch.equal(y0, y1)


def test_forward_refuses_odd_sizes():
    net = nn.UNet(cin=16, cout=16, chans=(32, 64), seed=4)
    with pytest.raises(nn._lbm.LBMError):
        net.forward(nn.empty_bf16(1, 5, 6, 16))
