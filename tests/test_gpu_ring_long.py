"""FP8 products with rows near the longest (K below 2^31), whole 64-byte slices
and not: the number of steps must not pass through 2^31.  A few nonzero codes,
the row's ends among them, so the result is a small integer."""

import pytest
import torch

import test_gpu_kernels as G

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K", [(1 << 31) - 16, (1 << 31) - 64])
def test_longest_rows(K):
    a = torch.zeros(1, K, dtype=torch.uint8, device=G.DEV)
    b = torch.zeros(1, K, dtype=torch.uint8, device=G.DEV)
    at = torch.tensor([0, 15, 64, 1 << 30, K - 65, K - 33, K - 16, K - 1], device=G.DEV)
    a[0, at] = 0x38   # 1
    b[0, at] = torch.tensor([0x38, 0x40, 0x48, 0x38, 0x40, 0xB8, 0x48, 0x40], dtype=torch.uint8,
                            device=G.DEV)   # 1 2 4 1 2 -1 4 2
    c = torch.full((1, 1), float("nan"), device=G.DEV)
    G.launch({"op": "gemm_fp8", "shape": (1, 1, K), "in": (0, 1), "out": (2,)}, [a, b, c])
    assert c.item() == 15.0
