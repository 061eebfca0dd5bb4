"""Row softmax and row sum at the edges of their variants (lanes per row,
float4 per lane) and at every alignment of the rows: rows that start 0 to 3
floats past a 16-byte boundary have up to three floats before their first and
after their last whole float4.  Nothing outside the output is written."""

import numpy as np
import pytest
import torch

import test_gpu_kernels as G
from oracle import kernels as OK
from paper_2509_12207_amd import capi

pytestmark = pytest.mark.gpu
PAD = 16


def shifted(A, off):
    """A on the device, starting `off` floats past a 16-byte boundary."""
    buf = torch.full((A.size + 2 * PAD,), 7.0, device=G.DEV)
    buf[PAD + off: PAD + off + A.size] = torch.from_numpy(A.reshape(-1)).to(G.DEV)
    return buf, buf.data_ptr() + 4 * (PAD + off)


def untouched(buf, off, n):
    host = buf.cpu().numpy()
    return (host[: PAD + off] == 7.0).all() and (host[PAD + off + n:] == 7.0).all()


EDGES = [1, 2, 3, 5, 255, 257, 1023, 1026, 2047, 2049, 4095, 4098, 8191, 8193, 16383, 16385]


# 1e-5 relative: the criterion of the softmax tests, above the exponential's
# error (x - max rounded at |x - max| <= 16: 2^-20) and the sum's.  Alignments
# of X and Y that differ take the path in three passes.
@pytest.mark.parametrize("L", EDGES)
@pytest.mark.parametrize("ox,oy", [(0, 0), (1, 1), (3, 3), (2, 1)])
def test_softmax_lengths_and_alignments(L, ox, oy):
    R = 7
    X = np.random.default_rng(L + ox).uniform(-8, 8, (R, L)).astype(np.float32)
    x, px = shifted(X, ox)
    y, py = shifted(np.full((R, L), np.nan, np.float32), oy)
    capi.kernel_launch({"op": "softmax", "shape": (R, L), "in": (0,), "out": (1,)}, [px, py])
    got = y.cpu().numpy()[PAD + oy: PAD + oy + R * L].reshape(R, L)
    ref = OK.softmax_f64(X)
    assert np.all(np.abs(got - ref) <= 1e-5 * ref)
    assert untouched(y, oy, R * L)
    # in place
    capi.kernel_launch({"op": "softmax", "shape": (R, L), "in": (0,), "out": (0,)}, [px])
    again = x.cpu().numpy()[PAD + ox: PAD + ox + R * L].reshape(R, L)
    assert np.all(np.abs(again - ref) <= 1e-5 * ref)
    assert untouched(x, ox, R * L)


@pytest.mark.parametrize("L", [5, 1026, 8191])
def test_softmax_masked_rows(L):
    X = np.random.default_rng(L).uniform(-8, 8, (5, L)).astype(np.float32)
    X[0, 1:] = -np.inf                        # one value left
    X[1, ::2] = np.finfo(np.float32).min      # the type's lowest value as a mask
    X[2, :] = -np.inf                         # nothing left
    X[3, L // 2] = np.nan
    x, px = shifted(X, 0)
    y, py = shifted(X, 0)
    capi.kernel_launch({"op": "softmax", "shape": (5, L), "in": (0,), "out": (1,)}, [px, py])
    got = y.cpu().numpy()[PAD: PAD + 5 * L].reshape(5, L)
    assert np.isnan(got[2:4]).all()
    ok = [0, 1, 4]
    ref = OK.softmax_f64(np.where(np.isinf(X[ok]), np.float32(-1e30), X[ok]))
    assert np.all(np.abs(got[ok] - ref) <= 1e-5 * ref)


# the sum of |values| times FP32's unit per addition along the longest chain
@pytest.mark.parametrize("R,L", [(7, n) for n in EDGES] + [(5, 511), (5, 513), (1030, 8199),
                                                          (3, 65537), (1, 200003)])
@pytest.mark.parametrize("off", [0, 1, 2, 3])
def test_rowsum_lengths_and_alignments(R, L, off):
    Z = np.random.default_rng(L + off).uniform(-1, 1, (R, L)).astype(np.float32)
    z, pz = shifted(Z, off)
    r, pr = shifted(np.full(R, np.nan, np.float32), 0)
    capi.kernel_launch({"op": "rowsum", "shape": (R, L), "in": (0,), "out": (1,)}, [pz, pr])
    s, a = OK.rowsum_f64(Z)
    got = r.cpu().numpy()[PAD: PAD + R]
    assert np.all(np.abs(got - s) <= (L / 64 + 16) * 2.0 ** -24 * a)
    assert untouched(r, 0, R)
