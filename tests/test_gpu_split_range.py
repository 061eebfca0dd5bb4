"""The FP32 contractions over the whole range of FP32 values.

Values are scaled before they are split into bfloat16 pieces
(csrc/kernels/split.hpp), so that values of every magnitude have a split,
subnormal ones too, with pieces that are subnormal bfloat16 values: the bound
of the split (test_gpu_split.py) holds throughout, and a tile that holds tiny
values takes the time of any other."""

import numpy as np
import pytest
import torch

import test_gpu_kernels as G
from oracle import kernels as OK
from paper_2509_12207_amd import capi
from test_gpu_split import bound

pytestmark = pytest.mark.gpu

# 32x32 and 64x64 tiles with K slices; 128x128 with two
GEMM = [(100, 70, 50), (700, 1100, 65), (1500, 1700, 1005)]
CONV = [(1, 40, 60, 80), (2, 16, 40, 50), (1, 64, 70, 90)]


def values(r, shape, e, bits):
    """Random multiples of 2^e in magnitude: of 1 <= v < 2 with `bits` bits
    after the point (FP32 rounds what is below 2^-149)."""
    v = (1.0 + r.integers(0, 1 << bits, shape) / (1 << bits)) * r.choice([-1.0, 1.0], shape)
    return np.ldexp(v, e).astype(np.float32)


# the whole significand where the third piece becomes subnormal, where it has
# no place below it and where the values themselves are subnormal; short
# significands whose first or second piece is subnormal
CASES = [(23, e) for e in (-101, -103, -105, -107, -109, -110, -112, -118, -126, -135)]
CASES += [(1, e) for e in (-120, -127, -131, -148)] + [(11, e) for e in (-110, -120, -126)]


@pytest.mark.parametrize("bits,e", CASES)
@pytest.mark.parametrize("M,N,K", GEMM)
def test_gemm_small_magnitudes(M, N, K, bits, e):
    r = np.random.default_rng(M - e)
    A, B = values(r, (M, K), e, bits), values(r, (K, N), 100, 23)
    C = G.run_gemm(A, B)
    ref, scale = OK.gemm_f64(A, B), OK.gemm_abs_f64(A, B)
    assert np.all(np.abs(C - ref) <= bound(K) * scale), np.max(np.abs(C - ref) / scale)


@pytest.mark.parametrize("bits,e", CASES)
@pytest.mark.parametrize("n,c,h,w", CONV)
def test_conv_small_magnitudes(n, c, h, w, bits, e):
    r = np.random.default_rng(c - e)
    X, W = values(r, (n, c, h, w), e, bits), values(r, (c, c, 3, 3), 90, 23)
    Y = G.run_conv(X, W)
    ref, scale = OK.conv3x3_f64(X, W), OK.conv3x3_abs_f64(X, W)
    K = 9 * ((c + 15) // 16) * 16
    assert np.all(np.abs(Y - ref) <= bound(K) * scale), np.max(np.abs(Y - ref) / scale)


# sums past 2^96, values past 2^112 and sums that overflow only when scaled or on
# the way: by the FP32 instruction, at most one rounding a product and a sum (the
# sums of |products| stay below 2^128, so none overflows)
@pytest.mark.parametrize("ea,eb", [(40, 50), (56, 60), (115, -100), (126, -60)])
@pytest.mark.parametrize("M,N,K", GEMM[:2])
def test_gemm_large_magnitudes(M, N, K, ea, eb):
    r = np.random.default_rng(M + ea)
    A, B = values(r, (M, K), ea, 23), values(r, (K, N), eb, 23)
    C = G.run_gemm(A, B)
    ref, scale = OK.gemm_f64(A, B), OK.gemm_abs_f64(A, B)
    assert np.all(np.abs(C - ref) <= K * 2.0 ** -23 * scale), np.max(np.abs(C - ref) / scale)


@pytest.mark.parametrize("ea,eb", [(56, 60), (115, -100)])
@pytest.mark.parametrize("n,c,h,w", CONV)
def test_conv_large_magnitudes(n, c, h, w, ea, eb):
    r = np.random.default_rng(c + ea)
    X, W = values(r, (n, c, h, w), ea, 23), values(r, (c, c, 3, 3), eb, 23)
    Y = G.run_conv(X, W)
    ref, scale = OK.conv3x3_f64(X, W), OK.conv3x3_abs_f64(X, W)
    assert np.all(np.abs(Y - ref) <= 9 * c * 2.0 ** -23 * scale), np.max(np.abs(Y - ref) / scale)


def _us(op, shape, a, b, out):
    desc = capi.kernel_struct({"op": op, "shape": shape, "in": (0, 1), "out": (2,)})
    ptrs = capi.pointer_array([t.data_ptr() for t in (a, b, out)])
    best = float("inf")
    for _ in range(5):
        s, e = (torch.cuda.Event(enable_timing=True) for _ in range(2))
        s.record()
        for _ in range(20):
            assert capi.lib().ug_kernel_launch(desc, ptrs, 3,
                                               torch.cuda.current_stream().cuda_stream) == capi.OK
        e.record()
        e.synchronize()
        best = min(best, s.elapsed_time(e) * 50.0)
    return best


def _operands(op, shape):
    g = torch.Generator(device=G.DEV).manual_seed(3)
    u = lambda *s: torch.rand(*s, generator=g, device=G.DEV) * 2 - 1
    if op == "gemm":
        M, N, K = shape
        return u(M, K), u(K, N), torch.empty(M, N, device=G.DEV)
    n, c, h, w = shape
    return u(n, c, h, w), u(c, c, 3, 3), torch.empty(n, c, h, w, device=G.DEV)


TIMED = [("gemm", (1003, 2050, 1021)), ("conv3x3", (1, 128, 128, 128))]


def _poisoned(op, a, value):
    """`value` in the operands of every tile."""
    b = a.clone()
    if op == "gemm":
        b[::32, 3] = value
    else:
        b[0, 1, ::8, ::16] = value
    return b


# a tile that holds such a value took 3.4 to 5.7 times as long when it was
# computed again; its time is now that of any other (half as much again is
# far above the spread of the measurement)
@pytest.mark.parametrize("op,shape", TIMED)
def test_tiny_values_take_no_time(op, shape):
    a, b, out = _operands(op, shape)
    plain = _us(op, shape, a, b, out)
    tiny = _us(op, shape, _poisoned(op, a, 1.2345678e-34), b, out)
    assert tiny < 1.5 * plain, (tiny, plain)


# one NaN in every tile: the tiles are computed again by the FP32 instruction,
# staged through LDS (2.5 and 3.2 times as long in all; 5.8 and 5.7 times where
# each lane read its operands from memory)
@pytest.mark.parametrize("op,shape", TIMED)
def test_values_without_a_split_are_staged(op, shape):
    a, b, out = _operands(op, shape)
    plain = _us(op, shape, a, b, out)
    again = _us(op, shape, _poisoned(op, a, float("nan")), b, out)
    assert again < 4.5 * plain, (again, plain)
