"""Every tile of the low-precision contractions (csrc/kernels/gemm_lowp.hip), at
and around its edges and with K steps that its K slices do not divide, on
integer-valued operands: every partial sum is a small integer, exact in any
order, so the results match the oracle bit for bit."""

import numpy as np
import pytest

import test_gpu_kernels as G
from oracle import kernels as OK

pytestmark = pytest.mark.gpu

BF16 = np.array([0x0000, 0x3F80, 0xBF80, 0x4000, 0xC000], np.uint16)   # 0, +-1, +-2
FP8 = np.array([0x00, 0x38, 0xB8, 0x40, 0xC0], np.uint8)

# 256x256; 128x128; 64x64; the same with two K slices; 32x64 with two; 32x32
# with eight
SHAPES = [(3073, 3080, 64), (1500, 1665, 96), (1000, 1100, 32), (1000, 900, 1056), (65, 500, 96),
          (31, 64, 32), (100, 130, 2080), (97, 33, 2048)]


@pytest.mark.parametrize("M,N,K", SHAPES)
def test_gemm_bf16_tiles(M, N, K):
    r = np.random.default_rng(M + N + K)
    A, B = BF16[r.integers(0, 5, (M, K))], BF16[r.integers(0, 5, (N, K))]
    assert np.array_equal(G.run_gemm_bf16(A, B), OK.gemm_bf16_f64(A, B).astype(np.float32))


# K a multiple of 64 and, for each tile, one that ends inside a 64-byte slice
@pytest.mark.parametrize("M,N,K", [(m, n, 2 * k + d) for m, n, k in SHAPES for d in (0, 16)])
def test_gemm_fp8_tiles(M, N, K):
    r = np.random.default_rng(M + N + K)
    A, B = FP8[r.integers(0, 5, (M, K))], FP8[r.integers(0, 5, (N, K))]
    assert np.array_equal(G.run_gemm_fp8(A, B), OK.gemm_fp8_f64(A, B).astype(np.float32))


# 128x128; 64x64; the same with two and four K slices; 32x32 with eight
@pytest.mark.parametrize("C,H,W", [(96, 150, 150), (64, 190, 191), (64, 100, 101), (160, 60, 50),
                                   (96, 17, 19), (32, 1, 3)])
def test_conv3x3_bf16_tiles(C, H, W):
    r = np.random.default_rng(C + H + W)
    X, Wt = BF16[r.integers(0, 5, (H, W, C))], BF16[r.integers(0, 5, (C, 3, 3, C))]
    assert np.array_equal(G.run_conv_bf16(X, Wt),
                          OK.conv3x3_bf16_f64(X, Wt).astype(np.float32))


# stages loaded in pairs, odd and even numbers of them, fewer than the ring
# holds and more: 256x256; 128x128; 64x64
PAIRS = [(3600, 3500, 32), (3590, 3585, 160), (2300, 2310, 96), (2177, 2305, 64), (1000, 900, 288)]


@pytest.mark.parametrize("M,N,K", PAIRS)
def test_gemm_bf16_stage_pairs(M, N, K):
    test_gemm_bf16_tiles(M, N, K)


@pytest.mark.parametrize("M,N,K", [(m, n, 2 * k + d) for m, n, k in PAIRS for d in (0, 16)])
def test_gemm_fp8_stage_pairs(M, N, K):
    test_gemm_fp8_tiles(M, N, K)


# 256x256 with an odd number of steps
@pytest.mark.parametrize("C,H,W", [(224, 193, 192)])
def test_conv3x3_bf16_stage_pairs(C, H, W):
    test_conv3x3_bf16_tiles(C, H, W)


# 64 channels of 16x16 pixels, 32 of 8x16, by groups of 64 channels and of 32:
# channels that the tile does not divide, tiles cut in both directions, one
# group and several
@pytest.mark.parametrize("C,H,W", [(64, 310, 321), (128, 225, 230), (160, 180, 200), (64, 9, 33),
                                   (128, 8, 16), (32, 17, 15), (96, 7, 50), (224, 31, 1),
                                   (32, 340, 333)])
def test_conv3x3_bf16_patches(C, H, W):
    test_conv3x3_bf16_tiles(C, H, W)
