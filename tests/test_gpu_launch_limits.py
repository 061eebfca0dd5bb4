"""Shapes whose grids would have more threads than one holds, run: products of
one column, or one row, of 2^29 to 2^30 and images of one pixel in millions.
Small whole numbers, so every result is exact; compared on the device."""

import pytest
import torch

import test_gpu_kernels as G

pytestmark = pytest.mark.gpu


def _ints(n, seed):
    g = torch.Generator(device=G.DEV).manual_seed(seed)
    return torch.randint(-8, 9, (n,), generator=g, device=G.DEV, dtype=torch.int8).float()


# one product a value, and three (the split's tiles have more threads)
@pytest.mark.parametrize("M,N,K", [((1 << 30) + 77, 1, 1), (1, (1 << 30) + 77, 1),
                                   ((1 << 29) + 77, 1, 3), (1, (1 << 29) + 77, 3)])
def test_gemm_of_one_column_or_row(M, N, K):
    n = max(M, N)
    long = _ints(n * K, 1)
    few = torch.tensor([3.0, -2.0, 5.0], device=G.DEV)[:K].contiguous()
    c = torch.full((n,), float("nan"), device=G.DEV)
    a, b = (long, few) if N == 1 else (few, long)
    G.launch({"op": "gemm", "shape": (M, N, K), "in": (0, 1), "out": (2,)}, [a, b, c])
    terms = long.view(n, K).unbind(1) if N == 1 else long.view(K, n).unbind(0)
    want = sum(t * f.item() for t, f in zip(terms, few))
    assert torch.equal(c, want)


def test_fp8_of_one_column():
    M, K = (1 << 30) + 77, 16
    a = torch.zeros(M, K, dtype=torch.uint8, device=G.DEV)
    codes = torch.tensor([0x00, 0x38, 0xB8, 0x40], dtype=torch.uint8, device=G.DEV)   # 0 1 -1 2
    pick = torch.arange(M, device=G.DEV, dtype=torch.int32) % 4
    a[:, 5] = codes[pick]
    b = torch.full((1, K), 0x40, dtype=torch.uint8, device=G.DEV)                     # 2
    c = torch.full((M,), float("nan"), device=G.DEV)
    G.launch({"op": "gemm_fp8", "shape": (M, 1, K), "in": (0, 1), "out": (2,)}, [a, b, c])
    assert torch.equal(c, torch.tensor([0.0, 2.0, -2.0, 4.0], device=G.DEV)[pick])


def test_conv_of_pixels_in_millions():
    n, c = 9_000_001, 17
    x = _ints(n * c, 2).reshape(n, c)
    w = _ints(c * c * 9, 3).reshape(c, c, 3, 3)
    y = torch.full((n, c), float("nan"), device=G.DEV)
    G.launch({"op": "conv3x3", "shape": (n, c, 1, 1), "in": (0, 1), "out": (2,)}, [x, w, y])
    # one pixel meets the middle tap only
    want = torch.zeros_like(y)
    for k in range(c):
        want += x[:, k:k + 1] * w[:, k, 1, 1]
    assert torch.equal(y, want)
