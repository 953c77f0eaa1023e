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
