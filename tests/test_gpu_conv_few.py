"""FP32 convolutions of few channels (csrc/kernels/conv3x3_f32.hip: up to eight,
by the FP32 instruction, four channels a step): at and past the edges of its
tiles, steps and channels, several images; at most one rounding a product, so
9 C 2^-24 of the sum of |products| (2^-23 where the pair of an instruction is
rounded on its own as well)."""

import numpy as np
import pytest

import test_gpu_kernels as G
from oracle import kernels as OK
from test_gpu_split_range import _operands, _us

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("c", [1, 2, 4, 5, 8, 9])
@pytest.mark.parametrize("n,h,w", [(1, 1, 1), (1, 8, 16), (2, 9, 17), (3, 5, 33), (1, 130, 140)])
def test_few_channels(n, c, h, w):
    r = np.random.default_rng(c + h)
    X = r.standard_normal((n, c, h, w)).astype(np.float32)
    W = r.standard_normal((c, c, 3, 3)).astype(np.float32)
    err = np.abs(G.run_conv(X, W) - OK.conv3x3_f64(X, W))
    assert np.all(err <= 9 * c * 2.0 ** -23 * OK.conv3x3_abs_f64(X, W))
    I = r.integers(-8, 9, X.shape).astype(np.float32), r.integers(-8, 9, W.shape).astype(np.float32)
    assert np.array_equal(G.run_conv(*I), OK.conv3x3_f64(*I).astype(np.float32))


# a chunk of 16 channels took as long for four as for nine (7.2 us against 10.5
# since, at 336^2)
def test_few_channels_take_less_time():
    us = {}
    for c in (4, 9):
        shape = (1, c, 336, 336)
        us[c] = _us("conv3x3", shape, *_operands("conv3x3", shape))
    assert us[4] < 0.85 * us[9], us
