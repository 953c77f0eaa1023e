"""The convolution that stages both operands in LDS (input channels a multiple
of 32) against the FP64 reference, at the edges of its blocks and of the rule
that chooses them: pixel counts one off whole blocks, images one pixel wide or
high, fewer pixels than a block, several images per block, channel counts of
every block shape, and operands too large for the LDS (the direct kernel).

Tolerance: the output is one BF16 rounding (2^-8 relative) of an FP32 sum of
exact products, whose accumulated rounding is below 1e-5 of the sum of
|terms|."""
import numpy as np
import pytest

from oracle import nn_ref as R
from tests.test_gpu_nn import BF, _bf, _dev_bf16, _host, _w_gpu_to_ref

pytestmark = pytest.mark.gpu

SHAPES = [(1, 5, 3, 32, 32), (2, 7, 1, 32, 32), (2, 1, 40, 64, 64), (5, 3, 7, 96, 32), (1, 8, 8, 128, 128),
          (1, 13, 5, 160, 32), (3, 17, 17, 256, 64), (2, 9, 11, 32, 16), (1, 33, 70, 96, 48), (1, 9, 9, 320, 48),
          (1, 4, 5, 864, 32), (9, 121, 121, 32, 32), (4, 131, 127, 64, 32), (4, 91, 93, 128, 64)]


@pytest.mark.parametrize("n,h,w,ci,co", SHAPES)
def test_conv3x3_lds_blocks(n, h, w, ci, co):
    import torch
    from paper_2211_03160_amd import nn
    rng = np.random.default_rng(n + h + w + ci + co)
    x = _bf(rng.standard_normal((n, h, w, ci)))
    wt = _bf(rng.standard_normal((9, co, ci)) * 0.2)
    b = rng.standard_normal(co).astype(np.float32)
    xd, wd, bd = _dev_bf16(x), _dev_bf16(wt), torch.from_numpy(b).cuda()
    plain = R.conv3x3(x, _w_gpu_to_ref(wt))
    scale = R.conv3x3(np.abs(x), np.abs(_w_gpu_to_ref(wt))) + np.abs(b)
    for bias, relu in ((bd, True), (None, False)):
        ref = plain + b if bias is not None else plain
        ref = R.relu(ref) if relu else ref
        err = np.abs(_host(nn.conv3x3(xd, wd, bias, co, relu)) - ref)
        assert np.all(err <= BF * np.abs(ref) + 1e-5 * scale), err.max()


# channel tiles of 32 and 64 on either side, ragged ones, pixel tiles one off
# their 8 x 16 (16 x 16 with 32 channels), one chunk, a chunk per tile and more
@pytest.mark.parametrize("chunks", [1, 2, 5, 400])
@pytest.mark.parametrize("n,h,w,ci,co", [(2, 17, 15, 32, 32), (1, 16, 17, 16, 48), (3, 15, 9, 64, 32),
                                         (2, 5, 24, 32, 64), (1, 33, 8, 80, 80), (2, 9, 7, 128, 96), (1, 1, 1, 16, 16)])
def test_conv3x3_wgrad_tiles(n, h, w, ci, co, chunks):
    """FP32 sums of exact BF16 products: within 1e-5 of the sum of |terms|."""
    import torch
    from paper_2211_03160_amd import nn
    rng = np.random.default_rng(ci + co + chunks)
    x = _bf(rng.standard_normal((n, h, w, ci)))
    dz = _bf(rng.standard_normal((n, h, w, co)))
    xd, dzd = _dev_bf16(x), _dev_bf16(dz)
    zero = np.zeros((3, 3, ci, co))
    _, ref, bref = R.conv3x3_backward(x, zero, dz)
    _, scale, bscale = R.conv3x3_backward(np.abs(x), zero, np.abs(dz))
    partial = torch.full((chunks * 9 * co * ci,), float("nan"), device="cuda")
    for with_bias in (True, False):
        dw = torch.full((9, co, ci), float("nan"), device="cuda")
        db = torch.full((co,), float("nan"), device="cuda")
        nn._check(nn.lib().lbm_nn_conv3x3_wgrad(nn._p(xd), nn._p(dzd), n, h, w, ci, co, nn._p(partial), chunks,
                                                nn._p(dw), nn._p(db) if with_bias else None, nn._s()))
        got = dw.cpu().numpy().astype(np.float64).reshape(3, 3, co, ci).transpose(0, 1, 3, 2)
        assert np.all(np.abs(got - ref) <= 1e-5 * scale + 1e-6)
        if with_bias:
            assert np.all(np.abs(db.cpu().numpy() - bref) <= 1e-5 * bscale + 1e-6)


@pytest.mark.parametrize("n,h,w,c,cs", [(1, 1, 1, 8, 8), (2, 5, 3, 16, 24), (3, 17, 33, 64, 32), (1, 2, 300, 72, 8)])
def test_joins_equal_their_parts(n, h, w, c, cs):
    """The one-pass joins against the single layers they combine, bit for bit,
    and those against numpy (exact but for the stated roundings)."""
    import torch
    from paper_2211_03160_amd import nn
    rng = np.random.default_rng(c + cs)
    x, dlow = (_bf(rng.standard_normal((n, h, w, c))) for _ in range(2))
    skip, big = (_bf(rng.standard_normal((n, 2 * h, 2 * w, k))) for k in (cs, c + cs))
    xd, skd, bigd, dlowd = _dev_bf16(x), _dev_bf16(skip), _dev_bf16(big), _dev_bf16(dlow)
    # upsample beside skip
    y = nn.upsample2_concat(xd, skd)
    assert torch.equal(y, nn.concat(nn.upsample2(xd), skd))
    assert np.array_equal(_host(y), np.concatenate([R.upsample2(x), skip], -1))
    # its gradient in front of the ReLU
    part = nn.empty_bf16(n, 2 * h, 2 * w, c)
    nn.copy_channels(bigd, 0, part, 0, c)
    assert np.array_equal(_host(part), big[..., :c])
    assert torch.equal(nn.upsample2_concat_backward(bigd, xd), nn.relu_backward(xd, nn.upsample2_backward(part)))
    # pooling gradient plus the last channels of the concatenation's
    yhigh = _dev_bf16(_bf(rng.standard_normal((n, 2 * h, 2 * w, c))))
    want = nn.avgpool2_backward(dlowd)
    assert np.array_equal(_host(want), R.avgpool2_backward(dlow))  # a quarter of a BF16 value is exact
    nn.copy_channels(bigd, cs, want, 0, c, accumulate=True)
    assert torch.equal(nn.avgpool2_backward_add(dlowd, bigd, yhigh), nn.relu_backward(yhigh, want))
    assert np.array_equal(_host(nn.avgpool2(bigd)), _bf(R.avgpool2(big)))


def test_layers_without_16_byte_access():
    """Channel counts that are no multiple of 8 and tensors off 16-byte
    addresses take the element kernels: the same values."""
    import torch
    from paper_2211_03160_amd import nn
    rng = np.random.default_rng(1)
    x = _bf(rng.standard_normal((2, 4, 6, 12)))
    xd = _dev_bf16(x)
    up = nn.upsample2(xd)
    assert np.array_equal(_host(up), R.upsample2(x))
    assert np.array_equal(_host(nn.avgpool2(xd)), _bf(R.avgpool2(x)))
    assert np.array_equal(_host(nn.avgpool2_backward(xd)), R.avgpool2_backward(x))
    assert np.allclose(_host(nn.upsample2_backward(xd)), R.upsample2_backward(x), rtol=BF, atol=0)
    flat = torch.zeros(1 + x.size, dtype=torch.int16, device="cuda")
    flat[1:] = xd.flatten()
    off = flat[1:]  # two bytes off
    dy = _dev_bf16(rng.standard_normal(x.size))
    assert torch.equal(nn.relu_backward(off, dy), nn.relu_backward(xd.flatten(), dy))
    with pytest.raises(Exception, match="bad arguments"):
        nn.upsample2_concat(xd, up)
    with pytest.raises(Exception, match="bad arguments"):
        nn.upsample2_concat_backward(up, xd)


@pytest.mark.parametrize("ci,co", [(32, 64), (48, 32), (16, 16)])
def test_masked_convolution_and_flips(ci, co):
    """The masked data gradient equals the convolution followed by the ReLU's
    gradient, and flipped weights of many layers equal those of each."""
    import torch
    from paper_2211_03160_amd import nn
    rng = np.random.default_rng(ci)
    dz = _dev_bf16(rng.standard_normal((2, 9, 11, ci)))
    mask = _dev_bf16(rng.standard_normal((2, 9, 11, co)))
    wt = _dev_bf16(rng.standard_normal((9, co, ci)) * 0.2)
    assert torch.equal(nn.conv3x3_masked(dz, wt, mask, co),
                       nn.relu_backward(mask, nn.conv3x3(dz, wt, None, co, False)))
    layers = [(_dev_bf16(rng.standard_normal((9, o, i))), i, o) for i, o in [(16, 48), (ci, co), (96, 32)] * 13]
    for (w, i, o), wf in zip(layers, nn.conv3x3_flip_many(layers)):
        assert torch.equal(wf, w.flip(0).transpose(1, 2).contiguous())
        assert torch.equal(wf, nn.conv3x3_flip(w, i, o))
