"""The height maximum of the direct voxel scatter is kept as the float itself
(integer atomics, signed for values without the sign bit and unsigned for the
others): cells of every mix of signs, zeros and infinities, in every order,
match the oracle bit for bit."""

import itertools

import numpy as np
import pytest

import test_gpu_kernels as G
from oracle import kernels as OK

pytestmark = pytest.mark.gpu

VALUES = [-np.inf, -3.5, -1e-40, -0.0, 0.0, 1e-40, 2.5, np.inf]


@pytest.mark.parametrize("k", [1, 2, 3])
def test_zmax_of_every_mix(k):
    mixes = list(itertools.product(VALUES, repeat=k))
    n = len(mixes) * k
    P = np.zeros((n, 4), np.float32)
    for c, mix in enumerate(mixes):
        for j, z in enumerate(mix):
            # point j of cell c, the cells' points spread over the cloud
            P[j * len(mixes) + c] = (c % 512 / 5.0 - 51.1, c // 512 / 5.0 - 51.1, z, 0.5)
    got = G.run_voxel(P)
    want = OK.voxel_scatter(P)
    for g, w in zip(got, want):
        assert np.array_equal(np.asarray(g).view(np.uint32), np.asarray(w).view(np.uint32))
