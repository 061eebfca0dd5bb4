"""The binned voxel scatter on grids whose cells fill their tiles in every way
(csrc/kernels/voxel.hip: blocks of 64 cells dealt to the tiles in turn): one
tile, fewer tiles than rounds of blocks, a last block and a last round that are
cut short, the largest grid; every cell hit, bit for bit against the oracle."""

import numpy as np
import pytest

import test_gpu_kernels as G
from oracle import kernels as OK

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny", [(1, 1), (63, 65), (64, 64), (4097, 1), (5, 2000), (333, 777),
                                   (2048, 2048)])
def test_binned_cells_of_any_grid(nx, ny):
    n = (1 << 20) + 77
    r = np.random.default_rng(nx * ny)
    P = np.concatenate([r.uniform(-1, nx + 1, (n, 1)), r.uniform(-1, ny + 1, (n, 1)),
                        r.normal(0, 3, (n, 1)), r.uniform(0, 1, (n, 1))], 1).astype(np.float32)
    G._same(G.run_voxel(P, nx, ny, (0.0, 0.0, 1.0)),
            OK.voxel_scatter(P, nx, ny, np.float32(0), np.float32(0), np.float32(1)))
