"""The voxel scatter of 56 Ki to 1 Mi points (csrc/kernels/voxel.hip, listed
path) against the oracle, bit for bit: point counts at the ends of the range,
of its two chunk sizes and of a last chunk; grids at both of its limits and
just outside; clouds of one cell, of none, and with zeros, infinities and NaN."""

import numpy as np
import pytest

import test_gpu_kernels as G
from oracle import kernels as OK

pytestmark = pytest.mark.gpu

LO = 56 << 10


def check(P, nx, ny, fp):
    for _ in range(2):
        G._same(G.run_voxel(P, nx, ny, fp),
                OK.voxel_scatter(P, nx, ny, *(np.float32(f) for f in fp)))


@pytest.mark.parametrize("n", [LO - 1, LO, LO + 511, 256 << 10, (256 << 10) + 1, 700_003,
                               (1 << 20) - 1])
def test_point_counts(n):
    check(G._cloud(n, n), 512, 512, (-51.2, -51.2, 5.0))


@pytest.mark.parametrize("nx,ny", [(63, 64), (37, 109), (300, 100), (1, 16385), (1023, 777),
                                   (1024, 1024), (1025, 1024)])
def test_grids(nx, ny):
    n = LO + 1000
    r = np.random.default_rng(nx * ny)
    P = np.concatenate([r.uniform(-1, nx + 1, (n, 1)), r.uniform(-1, ny + 1, (n, 1)),
                        r.normal(0, 3, (n, 1)), r.uniform(0, 1, (n, 1))], 1).astype(np.float32)
    check(P, nx, ny, (0.0, 0.0, 1.0))


@pytest.mark.parametrize("kind", ["one cell", "none", "one tile a chunk", "values"])
def test_clouds(kind):
    n = LO + 300
    P = G._cloud(5, n)
    if kind == "one cell":
        P[:, :2] = 0.05
    elif kind == "none":
        P[:, 0] = 1000.0
    elif kind == "one tile a chunk":   # the points of 512 in a row in one block of cells
        P[:, 0] = -51.1 + (np.arange(n) // 512 % 8) * 12.8
        P[:, 1] = -51.1 + (np.arange(n) // 512 % 500) / 5.0
    else:
        v = np.array([-np.inf, -3.5, -1e-40, -0.0, 0.0, 1e-40, 2.5, np.inf], np.float32)
        P[:, 2] = v[np.random.default_rng(1).integers(0, len(v), n)]
        P[::7, 0] = np.nan
        P[::11, 1] = np.inf
    check(P, 512, 512, (-51.2, -51.2, 5.0))
