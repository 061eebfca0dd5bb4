"""The two forms of 64 x 8x16 of the FP32 convolution (csrc/kernels/conv3x3_f32.hip:
nine taps with one buffer of the patch, tap rows), 32 x 16x16 and 32 x 8x16 by tap
rows, at the edges of tiles, channels and chunks: one chunk, two, several, odd and even
numbers of them, the last one whole or not.  Integer-valued inputs: every
partial sum is exact, so the results match the oracle bit for bit."""

import numpy as np
import pytest
import torch

import test_gpu_kernels as G
from oracle import kernels as OK
from paper_2509_12207_amd import capi

pytestmark = pytest.mark.gpu


# variant 0 up to 256 workgroups (nine taps) and past them (tap rows), variant 1,
# variant 2 past 256 workgroups
@pytest.mark.parametrize("variant,n,c,h,w", [
    (0, 1, 16, 9, 17), (0, 1, 32, 8, 16), (0, 2, 33, 7, 31), (0, 1, 64, 120, 130),
    (0, 3, 65, 25, 47), (0, 1, 130, 40, 50), (0, 1, 47, 200, 201), (0, 300, 17, 3, 5),
    (1, 1, 16, 17, 15), (1, 1, 32, 16, 16), (1, 2, 33, 40, 31), (1, 1, 48, 5, 70),
    (1, 3, 20, 33, 33), (2, 300, 17, 3, 5), (2, 1, 48, 100, 305), (2, 1, 32, 264, 260)])
def test_forms(variant, n, c, h, w):
    r = np.random.default_rng(c + h + w)
    X = r.integers(-8, 9, (n, c, h, w)).astype(np.float32)
    W = r.integers(-8, 9, (c, c, 3, 3)).astype(np.float32)
    x, wt, y = G.dev(X), G.dev(W), torch.full((n, c, h, w), float("nan"), device=G.DEV)
    capi.kernel_launch_variant({"op": "conv3x3", "shape": (n, c, h, w), "in": (0, 1), "out": (2,)},
                               [t.data_ptr() for t in (x, wt, y)], variant)
    torch.cuda.synchronize()
    assert np.array_equal(y.cpu().numpy(), OK.conv3x3_f64(X, W).astype(np.float32))
