"""The FP32 contractions on the BF16 matrix cores: every value split into
three bfloat16 pieces, six of nine products (csrc/kernels/split.hpp).

Accuracy: the matrix instruction rounds its accumulator once per 16 products
(at most one unit in the last place, 2^-23, of a partial sum that the sum of
|products| bounds), the five small products have an accumulator of their own
(below 2^-7 of that), and the products left out are below 2^-24 of the sum:
(K / 16 + 8) * 2^-23 of the sum of |products| covers all of it.

Values without a split (infinities, NaN, values that round to infinity in
bfloat16, values below about 2^-109) are computed by the FP32 instruction and
come out as before."""

import numpy as np
import pytest

import test_gpu_kernels as G
from oracle import kernels as OK

pytestmark = pytest.mark.gpu


def bound(K):
    return (K / 16 + 8) * 2.0 ** -23


# each tile with its K splits, at and around their edges: 128x128; 64x64 split
# two and four ways; 32x32 split four and eight ways; rows longer than 2^22
@pytest.mark.parametrize("M,N,K", [(1500, 1700, 33), (1537, 1665, 16), (700, 1100, 65),
                                   (1000, 1000, 1030), (65, 33, 64), (31, 32, 63),
                                   (200, 130, 600), (1, 5, 129), (3, (1 << 22) + 1, 5),
                                   (2, 3, (1 << 22) + 5)])
def test_gemm_error(M, N, K):
    r = np.random.default_rng(M + 3 * N + 5 * K)
    A = r.standard_normal((M, K)).astype(np.float32)
    B = r.standard_normal((K, N)).astype(np.float32)
    C = G.run_gemm(A, B)
    ref, scale = OK.gemm_f64(A, B), OK.gemm_abs_f64(A, B)
    assert np.all(np.abs(C - ref) <= bound(K) * scale), np.max(np.abs(C - ref) / scale)


def same_kind(got, ref):
    """Infinities and NaN where the exact result has them."""
    with np.errstate(over="ignore"):
        want = ref.astype(np.float32)
    assert np.array_equal(np.isnan(got), np.isnan(want))
    inf = np.isinf(want)
    assert np.array_equal(got[inf], want[inf]) and not np.isinf(got[~inf]).any()
    return np.isfinite(want)


@pytest.mark.parametrize("M,N,K", [(70, 90, 40), (1500, 1700, 20), (700, 1100, 48)])
def test_gemm_values_without_a_split(M, N, K):
    r = np.random.default_rng(M)
    A = r.uniform(0.5, 1, (M, K)).astype(np.float32)
    B = r.uniform(-1, 1, (K, N)).astype(np.float32)
    A[3, 5], A[9, 0], A[17, K - 1] = np.inf, -np.inf, np.nan
    A[21, 7], B[7, :] = 3.4e38, np.float32(2.0 ** -40)   # rounds to infinity in bfloat16
    B[2, N - 1] = np.inf
    with np.errstate(invalid="ignore"):
        ref = A.astype(np.float64) @ B.astype(np.float64)
        scale = np.abs(A).astype(np.float64) @ np.abs(B).astype(np.float64)
    C = G.run_gemm(A, B)
    ok = same_kind(C, ref)
    assert np.all(np.abs(C - ref)[ok] <= K * 2.0 ** -23 * scale[ok])


@pytest.mark.parametrize("lo", [-112, -126, -140])
def test_gemm_tiny_values(lo):
    M, N, K = 100, 70, 50
    r = np.random.default_rng(-lo)
    A = (r.uniform(1, 2, (M, K)) * 2.0 ** lo).astype(np.float32)
    B = (r.uniform(1, 2, (K, N)) * 2.0 ** 100).astype(np.float32)
    A[::2] = 0.0
    C = G.run_gemm(A, B)
    ref, scale = OK.gemm_f64(A, B), OK.gemm_abs_f64(A, B)
    assert np.all(np.abs(C - ref) <= K * 2.0 ** -23 * scale)


# ------------------------------------------------------------- convolution
# 64 x 8x16 by tap rows and at once, 32 x 16x16, 32 x 8x16, 32 x 4x16 and
# 32 x 2x16; one chunk of channels, with two buffers and with one
CONV = [(1, 64, 250, 250), (1, 130, 70, 90), (1, 30, 250, 260), (1, 40, 100, 140), (1, 40, 60, 80),
        (1, 100, 33, 47), (3, 17, 5, 16), (2, 16, 40, 50), (1, 3, 13, 21), (1, 7, 200, 199)]


@pytest.mark.parametrize("n,c,h,w", CONV)
def test_conv_error(n, c, h, w):
    r = np.random.default_rng(n + 3 * c + 5 * h + 7 * w)
    X = r.standard_normal((n, c, h, w)).astype(np.float32)
    W = r.standard_normal((c, c, 3, 3)).astype(np.float32)
    Y = G.run_conv(X, W)
    ref, scale = OK.conv3x3_f64(X, W), OK.conv3x3_abs_f64(X, W)
    # every chunk of 16 channels is one matrix instruction a tap
    K = 9 * ((c + 15) // 16) * 16
    assert np.all(np.abs(Y - ref) <= bound(K) * scale), np.max(np.abs(Y - ref) / scale)


def conv_abs(X, W):
    """Sum of |products| of a zero-padded convolution, zero where one is not finite."""
    return OK.conv3x3_abs_f64(np.nan_to_num(X, posinf=0, neginf=0),
                              np.nan_to_num(W, posinf=0, neginf=0))


@pytest.mark.parametrize("n,c,h,w", [CONV[0], CONV[1], CONV[4], CONV[7]])
def test_conv_values_without_a_split(n, c, h, w):
    r = np.random.default_rng(c)
    X = r.uniform(0.5, 1, (n, c, h, w)).astype(np.float32)
    W = r.uniform(-1, 1, (c, c, 3, 3)).astype(np.float32)
    X[0, 2, 3, 4], X[0, 5, h - 3, w - 2], X[0, c - 1, 20, 9] = np.inf, -np.inf, np.nan
    with np.errstate(invalid="ignore"):
        ref = OK.conv3x3_f64(X, W)
    Y = G.run_conv(X, W)
    ok = same_kind(Y, ref)
    assert np.all(np.abs(Y - ref)[ok] <= 9 * c * 2.0 ** -23 * conv_abs(X, W)[ok])


@pytest.mark.parametrize("n,c,h,w", [CONV[4], CONV[7]])
def test_conv_tiny_values(n, c, h, w):
    r = np.random.default_rng(c + 1)
    X = (r.uniform(1, 2, (n, c, h, w)) * 2.0 ** -125).astype(np.float32)
    W = (r.uniform(1, 2, (c, c, 3, 3)) * 2.0 ** 90).astype(np.float32)
    Y = G.run_conv(X, W)
    ref, scale = OK.conv3x3_f64(X, W), OK.conv3x3_abs_f64(X, W)
    assert np.all(np.abs(Y - ref) <= 9 * c * 2.0 ** -23 * scale)


# 256 x 128 tiles: odd and even numbers of steps of 16, one to five, the first
# of them whole or not; edges of both sides
@pytest.mark.parametrize("M,N,K", [(3900, 1930, 1), (3900, 1930, 16), (4096, 2048, 17),
                                   (3900, 1930, 33), (4095, 2047, 48), (3900, 1930, 64),
                                   (3900, 1930, 65)])
def test_gemm_error_wide_tiles(M, N, K):
    test_gemm_error(M, N, K)


def test_gemm_values_without_a_split_wide_tiles():
    test_gemm_values_without_a_split(3900, 1930, 40)


# 128 x 128 tiles with K in two slices of 16: K a multiple of their step and
# not, one slice short of its last step, edges of both sides
@pytest.mark.parametrize("M,N,K", [(1500, 1700, 1000), (1537, 1665, 1024), (1530, 1690, 1037),
                                   (700, 2800, 1010)])
def test_gemm_error_two_slices(M, N, K):
    test_gemm_error(M, N, K)


def test_gemm_values_without_a_split_two_slices():
    test_gemm_values_without_a_split(1500, 1700, 1005)
