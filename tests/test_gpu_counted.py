"""The completion counter of every kernel that carries one (each instance that
the launchers' plans name): it ends at exactly the wavefront count that the
launch reports, and a counted launch stores what an uncounted one does."""

import pytest
import torch

import test_gpu_fused as F
import test_gpu_kernels as G
from paper_2509_12207_amd import capi
from test_launch_limits import plan

pytestmark = pytest.mark.gpu

CASES = {
    # 256x128; 128x128 with two K slices and with one; 64x64 with four and two;
    # 32x32 with eight and four; rows longer than 2^22; sums of two products
    "gemm": [(4096, 2048, 64), (1500, 1700, 1005), (1500, 1700, 65), (1024, 1024, 1024),
             (1024, 1024, 300), (96, 160, 2048), (96, 160, 264), (3, (1 << 22) + 1, 5),
             (2, 3, (1 << 22) + 5), (100, 130, 2)],
    # few channels; one chunk, one buffer and two; 32 x 2x16, 4x16, 8x16 and, by tap
    # rows, 8x16 and 16x16; 64 x 8x16 of nine taps and by tap rows
    "conv3x3": [(1, 8, 20, 20), (1, 16, 336, 336), (1, 16, 64, 64), (1, 32, 20, 16), (1, 64, 84, 84),
                (1, 64, 128, 128), (1, 20, 264, 264), (1, 32, 256, 256), (1, 128, 128, 128), (1, 64, 200, 200)],
    # 256x256 with stages in pairs and single, 128x128 likewise, 32x32 with eight
    # K slices, 32x64 with two, 64x64 with two and in pairs
    "gemm_bf16": [(3600, 3500, 32), (3073, 3080, 64), (2300, 2310, 96), (1500, 1665, 96),
                  (97, 33, 2048), (65, 500, 96), (1000, 900, 1056), (1000, 1100, 32)],
    # 64 channels of 16x16 pixels and 32 of 8x16, by groups of 64 channels and of 32
    "conv3x3_bf16": [(1, 64, 310, 321), (1, 160, 192, 208), (1, 64, 24, 40), (1, 96, 7, 50)],
}


def test_the_cases_are_different_kernels():
    for op, shapes in CASES.items():
        assert len({plan(op, s).func for s in shapes}) == len(shapes), op


@pytest.mark.parametrize("op,shape", [(op, s) for op, shapes in CASES.items() for s in shapes])
def test_counts_every_wavefront(op, shape):
    F.test_launch_signal_counts_every_wavefront(op, shape, -1)


# by the short sums' kernel and the split's
@pytest.mark.parametrize("M,K", [((1 << 30) + 77, 1), ((1 << 29) + 77, 3)])
def test_counts_the_idle_workgroups_of_a_two_sided_grid(M, K):
    a, b = torch.ones(M, K, device=G.DEV), torch.full((K,), 2.0, device=G.DEV)
    c, cnt = torch.zeros(M, device=G.DEV), torch.zeros(1, dtype=torch.int32, device=G.DEV)
    torch.cuda.synchronize()
    waves = capi.kernel_launch_signal({"op": "gemm", "shape": (M, 1, K), "in": (0, 1), "out": (2,)},
                                      [t.data_ptr() for t in (a, b, c)], cnt.data_ptr(), 0)
    torch.cuda.synchronize()
    assert plan("gemm", (M, 1, K)).grid.y > 1 and cnt.item() == waves
    assert (c == 2 * K).all()
