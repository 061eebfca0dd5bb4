"""Products too short for the split of the FP32 GEMM (fewer than three terms:
what it leaves out is more than the roundings it saves): one product is
correctly rounded, two err by at most one rounding of the first and one of the
sum, 2^-24 of the sum of |products| each."""

import numpy as np
import pytest

import test_gpu_kernels as G
from oracle import kernels as OK

pytestmark = pytest.mark.gpu


# one tile of 64x64 cut in both directions, several, many
@pytest.mark.parametrize("M,N", [(100, 70), (700, 1100), (1537, 1665), (3900, 1930)])
def test_short_sums(M, N):
    r = np.random.default_rng(M)
    A = r.standard_normal((M, 2)).astype(np.float32)
    B = r.standard_normal((2, N)).astype(np.float32)
    assert np.array_equal(G.run_gemm(A[:, :1], B[:1]), A[:, :1] * B[:1])
    err = np.abs(G.run_gemm(A, B) - OK.gemm_f64(A, B))
    assert np.all(err <= 2.0 ** -23 * OK.gemm_abs_f64(A, B))
