"""Row sums of many short rows (csrc/kernels/pointwise.hip: past 8192 rows sixteen
lanes a row up to 128 floats, 32 up to 512), at the edges of lanes, rows per
workgroup and alignments."""

import numpy as np
import pytest
import torch

import test_gpu_kernels as G
from oracle import kernels as OK
from paper_2509_12207_amd import capi
from test_gpu_rows import PAD, shifted, untouched

pytestmark = pytest.mark.gpu


# a lane adds at most 16 values and a tail one, five shuffles follow: 22
# roundings of 2^-24 of the sum of |values| at most
@pytest.mark.parametrize("L", [1, 3, 4, 5, 63, 64, 66, 127, 128, 129, 131, 256, 257, 510, 512, 513])
@pytest.mark.parametrize("R", [9, 8192, 8193, 8208, 8999])
@pytest.mark.parametrize("off", [0, 1, 2, 3])
def test_short_rows(L, R, off):
    Z = np.random.default_rng(L + R + off).uniform(-1, 1, (R, L)).astype(np.float32)
    z, pz = shifted(Z, off)
    r, pr = shifted(np.full(R, np.nan, np.float32), 0)
    capi.kernel_launch({"op": "rowsum", "shape": (R, L), "in": (0,), "out": (1,)}, [pz, pr])
    s, a = OK.rowsum_f64(Z)
    got = r.cpu().numpy()[PAD: PAD + R]
    assert np.all(np.abs(got - s) <= 22 * 2.0 ** -24 * a)
    assert untouched(r, 0, R)


# the same bytes in rows a quarter as long and four times as many take about as
# long (3.1 us; twice as long with a wave a row)
def test_many_short_rows_take_no_longer():
    us = {}
    for R, L in ((47144, 57), (11786, 228)):
        z, r = torch.rand(R, L, device=G.DEV), torch.empty(R, device=G.DEV)
        desc = capi.kernel_struct({"op": "rowsum", "shape": (R, L), "in": (0,), "out": (1,)})
        ptrs = capi.pointer_array([z.data_ptr(), r.data_ptr()])
        best = float("inf")
        for _ in range(5):
            s, e = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            s.record()
            for _ in range(100):
                assert capi.lib().ug_kernel_launch(desc, ptrs, 2,
                                                   torch.cuda.current_stream().cuda_stream) == capi.OK
            e.record()
            e.synchronize()
            best = min(best, s.elapsed_time(e) * 10.0)
        us[L] = best
    assert us[57] < 1.6 * us[228], us
