"""A tail executor asked for more workers than there are compute units runs
one workgroup a CU at most, the dispatcher included: contractions start beside
it whatever their tile, and the tails that wait for them finish long before the
executor would leave."""

import time

import numpy as np
import pytest
import torch

import test_gpu_kernels as G
from oracle import kernels as OK
from paper_2509_12207_amd import capi

pytestmark = pytest.mark.gpu


def _wait(q, item, seconds):
    end = time.monotonic() + seconds
    q.kick()
    while not q.finished(*item):
        assert time.monotonic() < end, "tail not finished"
        time.sleep(0.001)


def _stream_beside_executor():
    """A stream whose hardware queue is not the running executor's."""
    word = torch.zeros(16, device=G.DEV)
    streams = [torch.cuda.Stream() for _ in range(8)]
    done = []
    for s in streams:
        with torch.cuda.stream(s):
            word.zero_()
            done.append(torch.cuda.Event())
            done[-1].record()
    time.sleep(0.2)
    return next(s for s, e in zip(streams, done) if e.query())


def test_workers_are_bounded_by_the_cus():
    # 16384 rows of 4 KiB: rows / workers a tile, 16 at 1024 workers
    R, N = 16384, 1024
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    x, b = torch.rand(R, N, device=G.DEV), torch.zeros(N, device=G.DEV)
    torch.cuda.synchronize()
    q = capi.TailQueue(workers=1024, log_cap=8192)
    _wait(q, q.publish(x.data_ptr(), x.data_ptr(), b.data_ptr(), R, N, 0, key=1), 20)
    tiles = len(q.log())
    q.close()
    rows = (-(-R // (cus - 1)) + 3) // 4 * 4
    assert tiles == -(-R // rows)


# 64 x 8x16 of nine taps and by tap rows, 32 x 16x16; FP32 GEMM of 256x128, of
# 128x128 with two K slices, of 64x64 with four
@pytest.mark.parametrize("op,shape", [
    ("conv3x3", (1, 128, 128, 128)), ("conv3x3", (1, 64, 200, 200)), ("conv3x3", (1, 32, 256, 256)),
    ("gemm", (4096, 2048, 64)), ("gemm", (1500, 1700, 1004)), ("gemm", (1024, 1024, 1024))])
def test_contractions_start_beside_a_full_executor(op, shape):
    r = np.random.default_rng(shape[1])
    if op == "gemm":
        M, N, K = shape
        A, B = (r.integers(-8, 9, s).astype(np.float32) for s in ((M, K), (K, N)))
        ref, rows, cols, axis = OK.gemm_f64(A, B), M, N, 0
    else:
        A = r.integers(-8, 9, shape).astype(np.float32)
        B = r.integers(-8, 9, (shape[1], shape[1], 3, 3)).astype(np.float32)
        ref, rows, cols, axis = OK.conv3x3_f64(A, B), shape[1], shape[2] * shape[3], 1
    a, b, out = G.dev(A), G.dev(B), torch.empty(rows, cols, device=G.DEV)
    bias = torch.zeros(cols if axis == 0 else rows, device=G.DEV)
    cnt = torch.zeros(1, dtype=torch.int32, device=G.DEV)
    k = {"op": op, "shape": shape, "in": (0, 1), "out": (2,)}
    ptrs = [a.data_ptr(), b.data_ptr(), out.data_ptr()]
    waves = capi.kernel_launch_signal(k, ptrs, cnt.data_ptr(), 0)
    torch.cuda.synchronize()
    cnt.zero_()
    torch.cuda.synchronize()
    # the executor waits for the item's counter, for 20 s without progress
    q = capi.TailQueue(workers=1024, idle_ns=20_000_000_000)
    item = q.publish(out.data_ptr(), out.data_ptr(), bias.data_ptr(), rows, cols, axis, key=1,
                     counter=cnt.data_ptr(), target=waves)
    q.kick()
    s = _stream_beside_executor()
    capi.kernel_launch_signal(k, ptrs, cnt.data_ptr(), s.cuda_stream)
    _wait(q, item, 5)
    s.synchronize()
    q.close()
    assert np.array_equal(out.cpu().numpy(), np.maximum(ref, 0).astype(np.float32).reshape(rows, cols))
