"""Values, alignments and shapes at the edges of what the network kernels take:
infinities beside padding, tensors off 16-byte addresses, images of a few
pixels, and sizes beyond one launch's grid.  Tolerances are those of the
kernels' FP32 sums of exact BF16 products: 1e-5 of the sum of |terms|, and one
BF16 rounding (2^-8 relative) where the output is BF16."""
import numpy as np
import pytest

from oracle import nn_ref as R
from tests.test_gpu_nn import BF, _bf, _dev_bf16, _host, _w_gpu_to_ref

pytestmark = pytest.mark.gpu


def _wgrad(x, dz, co, chunks=3):
    import torch
    from paper_2211_03160_amd import nn
    n, h, w, ci = x.shape
    dw, db = torch.empty((9, co, ci), device="cuda"), torch.empty((co,), device="cuda")
    partial = torch.full((chunks * 9 * co * ci,), float("nan"), device="cuda")
    nn._check(nn.lib().lbm_nn_conv3x3_wgrad(nn._p(x), nn._p(dz), n, h, w, ci, co, nn._p(partial), chunks, nn._p(dw),
                                            nn._p(db), nn._s()))
    return dw.cpu().numpy().astype(np.float64).reshape(3, 3, co, ci).transpose(0, 1, 3, 2), db.cpu().numpy()


# the last row and column of images off whole 8 x 16 (16 x 16) pixel tiles,
# and of whole ones
@pytest.mark.parametrize("n,h,w,ci,co", [(1, 5, 7, 16, 16), (2, 17, 9, 32, 64), (2, 16, 8, 64, 64), (3, 3, 10, 64, 16)])
def test_wgrad_infinite_activation_reaches_only_its_taps(n, h, w, ci, co):
    rng = np.random.default_rng(h * w)
    x = _bf(rng.standard_normal((n, h, w, ci)))
    dz = _bf(1.0 + rng.random((n, h, w, co)))  # positive: an infinity never meets its negative
    zero = np.zeros((3, 3, ci, co))
    for i, j in ((h - 1, w - 1), (0, w - 1), (h - 1, 0), (0, 0), (h - 1, w // 2), (h // 2, w - 1)):
        for b in {0, n - 1}:
            xi = x.copy()
            xi[b, i, j, ci // 2] = np.inf
            _, ref, _ = R.conv3x3_backward(xi, zero, dz)
            _, scale, _ = R.conv3x3_backward(np.abs(x), zero, np.abs(dz))
            got, _ = _wgrad(_dev_bf16(xi), _dev_bf16(dz), co)
            far = np.isinf(ref)
            assert far.any() and not far.all() and not np.isnan(ref).any()
            assert np.array_equal(got[far], ref[far]), (b, i, j)
            assert np.all(np.abs(got[~far] - ref[~far]) <= 1e-5 * scale[~far] + 1e-6), (b, i, j)


@pytest.mark.parametrize("ci,co", [(32, 32), (64, 48), (16, 32)])
@pytest.mark.parametrize("skew", [1, 2, 4])
def test_convolution_output_and_mask_off_8_byte_addresses(ci, co, skew):
    """An output and a mask that only a value's own size aligns: the bits of
    the aligned call, and no value beside the output."""
    import torch
    from paper_2211_03160_amd import nn
    rng = np.random.default_rng(ci + skew)
    n, h, w = 2, 9, 11
    x, wt = _dev_bf16(rng.standard_normal((n, h, w, ci))), _dev_bf16(rng.standard_normal((9, co, ci)) * 0.2)
    b = torch.from_numpy(rng.standard_normal(co).astype(np.float32)).cuda()
    mask = _dev_bf16(rng.standard_normal((n, h, w, co)))
    size = mask.numel()

    def off(t=None):
        flat = torch.full((size + 8,), 0x7abc, dtype=torch.int16, device="cuda")
        if t is not None:
            flat[skew:skew + size] = t.flatten()
        return flat, flat[skew:skew + size].view(n, h, w, co)

    flat, y = off()
    nn._check(nn.lib().lbm_nn_conv3x3(nn._p(x), n, h, w, ci, nn._p(wt), nn._p(b), co, 1, nn._p(y), nn._s()))
    assert torch.equal(y, nn.conv3x3(x, wt, b, co, True))
    assert (flat[:skew] == 0x7abc).all() and (flat[skew + size:] == 0x7abc).all()
    _, m = off(mask)
    want = nn.conv3x3_masked(x, wt, mask, co)
    assert torch.equal(nn.conv3x3_masked(x, wt, m, co), want)
    flat, y = off()
    nn._check(nn.lib().lbm_nn_conv3x3_masked(nn._p(x), n, h, w, ci, nn._p(wt), nn._p(m), co, nn._p(y), nn._s()))
    assert torch.equal(y, want)
    assert (flat[:skew] == 0x7abc).all() and (flat[skew + size:] == 0x7abc).all()


# narrow images (many rows per block), rows of odd lengths, one channel group,
# image rows longer than 65535 blocks of 256 groups (the concatenation), and
# more rows than one launch can hold blocks for
@pytest.mark.parametrize("n,h,w,c,cs", [(7, 50, 1, 8, 8), (1, 1, 129, 24, 16), (300, 1, 1, 40, 8), (5, 13, 17, 8, 48),
                                        (1, 1, 65600, 512, 512), ((1 << 23) + 5, 1, 1, 8, 8)])
def test_row_passes_of_any_shape(n, h, w, c, cs):
    """Copies and sums of four BF16 values: the same bits as torch."""
    import torch
    from paper_2211_03160_amd import nn
    g = torch.Generator(device="cuda")
    g.manual_seed(n + w)
    val = lambda *s: (torch.randint(-64, 65, s, generator=g, device="cuda").to(torch.bfloat16) / 16)  # noqa: E731
    raw = lambda t: t.contiguous().view(torch.int16)  # noqa: E731
    up = lambda t: t[:, :, None, :, None].expand(n, h, 2, w, 2, t.shape[-1]).reshape(n, 2 * h, 2 * w, -1)  # noqa: E731
    quad = lambda t: t.reshape(n, h, 2, w, 2, t.shape[-1])  # noqa: E731
    x, skip = val(n, h, w, c), val(n, 2 * h, 2 * w, cs)
    cat = torch.cat([up(x), skip], -1)
    assert torch.equal(nn.upsample2(raw(x)), raw(up(x)))
    assert torch.equal(nn.upsample2_concat(raw(x), raw(skip)), raw(cat))
    q = quad(cat)
    four = lambda t: ((t[:, :, 0, :, 0].float() + t[:, :, 0, :, 1].float())  # noqa: E731
                      + t[:, :, 1, :, 0].float()) + t[:, :, 1, :, 1].float()
    assert torch.equal(nn.avgpool2(raw(cat)), raw((0.25 * four(q)).to(torch.bfloat16)))
    s = four(q[..., :c]).to(torch.bfloat16)
    assert torch.equal(nn.upsample2_concat_backward(raw(cat), raw(x)), raw(torch.where(x > 0, s, 0)))
    assert torch.equal(nn.upsample2_backward(raw(skip)), raw(four(quad(skip)).to(torch.bfloat16)))
    y = val(n, 2 * h, 2 * w, cs)
    dlow = val(n, h, w, cs)
    part = (0.25 * up(dlow).float()).to(torch.bfloat16)
    assert torch.equal(nn.avgpool2_backward(raw(dlow)), raw(part))
    add = (part.float() + cat[..., c:].float()).to(torch.bfloat16)
    assert torch.equal(nn.avgpool2_backward_add(raw(dlow), raw(cat), raw(y)), raw(torch.where(y > 0, add, 0)))


# images lower than a tile of 16 rows, one row off it, and tall ones; narrow
# and one off 8 and 16 columns; tiles that hold many images and parts of two
@pytest.mark.parametrize("n,h,w", [(70, 1, 1), (16, 2, 2), (33, 1, 9), (9, 3, 5), (5, 15, 9), (4, 16, 17), (3, 31, 7)])
@pytest.mark.parametrize("ci,co", [(16, 16), (64, 32), (32, 80), (128, 64)])
def test_wgrad_of_many_small_images(n, h, w, ci, co):
    rng = np.random.default_rng(n * h + w + ci)
    x, dz = _bf(rng.standard_normal((n, h, w, ci))), _bf(rng.standard_normal((n, h, w, co)))
    zero = np.zeros((3, 3, ci, co))
    _, ref, bref = R.conv3x3_backward(x, zero, dz)
    _, scale, bscale = R.conv3x3_backward(np.abs(x), zero, np.abs(dz))
    for chunks in (1, 2, 3, 5, 6, 50):
        got, bias = _wgrad(_dev_bf16(x), _dev_bf16(dz), co, chunks)
        assert np.all(np.abs(got - ref) <= 1e-5 * scale + 1e-6)
        assert np.all(np.abs(bias - bref) <= 1e-5 * bscale + 1e-6)


def test_more_weights_than_a_launch_holds_blocks_for():
    """Flips and chunk sums whose pieces exceed 65536 blocks, each block then
    taking several: exact against torch (one pixel, whose products and sums are
    exact in FP32 with these values)."""
    import torch
    from paper_2211_03160_amd import nn
    g = torch.Generator(device="cuda")
    g.manual_seed(3)
    val = lambda *s: torch.randint(-8, 9, s, generator=g, device="cuda").to(torch.bfloat16)  # noqa: E731
    raw = lambda t: t.contiguous().view(torch.int16)  # noqa: E731
    ci, co = 2752, 2784  # 9 x 86 x 87 squares of 32 x 32
    layers = [(raw(val(9, o, i)), i, o) for i, o in ((16, 32), (ci, co), (48, 16))]
    for (w, i, o), wf in zip(layers, nn.conv3x3_flip_many(layers)):
        assert torch.equal(wf, w.flip(0).transpose(1, 2).contiguous())
    n = 9 * 256 * ci  # 99072 blocks of 64 sums
    for m, chunks in ((3, 2), (16 * 5, 7)):  # one chunk, and six: images of 16 x 1 pixels fill a tile each
        x, dz = val(m, 16, 1, ci), val(m, 16, 1, 256)
        x[:, 1:] = 0  # of which one holds values
        dz[:, 1:] = 0
        partial = torch.full((chunks * n,), float("nan"), device="cuda")
        dw, db = torch.full((9, 256, ci), float("nan"), device="cuda"), torch.full((256,), float("nan"), device="cuda")
        nn._check(nn.lib().lbm_nn_conv3x3_wgrad(nn._p(raw(x)), nn._p(raw(dz)), m, 16, 1, ci, 256, nn._p(partial), chunks,
                                                nn._p(dw), nn._p(db), nn._s()))
        want = torch.zeros(9, 256, ci, device="cuda")
        want[4] = dz[:, 0, 0].float().t().contiguous() @ x[:, 0, 0].float()
        assert torch.equal(dw, want) and torch.equal(db, dz.float().sum((0, 1, 2)))


def test_bias_gradient_keeps_its_precision():
    """Mean relative error of the bias gradient over 16 x 136 x 136 pixels: the
    FP32 trees of an earlier kernel reached 7.8e-8 with these inputs."""
    import torch
    from paper_2211_03160_amd import nn
    n, h, w, ci, co, err = 16, 136, 136, 32, 32, []
    for seed in range(12):
        g = torch.Generator(device="cuda")
        g.manual_seed(seed)
        x = torch.relu(torch.randn(n, h, w, ci, generator=g, device="cuda")).to(torch.bfloat16)
        dz = (torch.randn(n, h, w, co, generator=g, device="cuda") * 0.01).to(torch.bfloat16)
        dw, db = torch.empty(9, co, ci, device="cuda"), torch.empty(co, device="cuda")
        nn.conv3x3_wgrad(x.view(torch.int16), dz.view(torch.int16), co, dw, db)
        ref = dz.double().sum((0, 1, 2))
        err.append(float((db.double() - ref).norm() / ref.norm()))
    assert np.mean(err) < 7.8e-8, np.mean(err)
