"""The direct voxel scatter of clouds with many points a cell (zmax as an ordered
key, decoded by a last launch): cells of every mix of signs, zeros and
infinities, cells without a point, points outside, at both ends of the rule's
range, bit for bit against the oracle."""

import numpy as np
import pytest

import test_gpu_kernels as G
from oracle import kernels as OK

pytestmark = pytest.mark.gpu


# one cell; fewer than 64; past and just short of 12 points a cell; just short of
# 24 Ki points; as many as the listed path takes, in a grid too small for it
@pytest.mark.parametrize("n,nx,ny", [(24 << 10, 1, 1), (24 << 10, 5, 7), (30_000, 50, 50),
                                     (30_000, 50, 51), ((24 << 10) - 1, 9, 9), (200_001, 63, 64)])
@pytest.mark.parametrize("kind", ["normal", "values"])
def test_dense_cells(n, nx, ny, kind):
    r = np.random.default_rng(n + nx)
    P = np.stack([r.uniform(-1, nx + 1, n), r.uniform(-1, ny + 1, n), r.normal(0, 3, n),
                  r.uniform(0, 1, n)], 1).astype(np.float32)
    P[(P[:, 0] >= 0) & (P[:, 0] < 1), 1] += 2 * ny   # the first column stays empty
    if kind == "values":
        v = np.array([-np.inf, -3.5, -1e-40, -0.0, 0.0, 1e-40, 2.5, np.inf], np.float32)
        # a cell takes values from the first k only, so that the maximum is any of them
        cell = np.floor(P[:, 0]).astype(int) + nx * np.floor(P[:, 1]).astype(int)
        P[:, 2] = v[(r.random(n) * (1 + cell % len(v))).astype(int)]
    for _ in range(2):
        G._same(G.run_voxel(P, nx, ny, (0.0, 0.0, 1.0)),
                OK.voxel_scatter(P, nx, ny, np.float32(0), np.float32(0), np.float32(1)))
