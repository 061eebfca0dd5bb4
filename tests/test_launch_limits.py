"""A kernel's grid holds at most 2^32 - 1 threads a side (the dispatch packet's
limit).  Shapes that the validation accepts and 288 GB hold get a grid within
it: narrow products of 2^29 rows and more, small images in millions, long rows
in millions (the launchers' own plans, no GPU needed)."""

import ctypes as C

import pytest

from paper_2509_12207_amd import capi


class Dim3(C.Structure):
    _fields_ = [("x", C.c_uint32), ("y", C.c_uint32), ("z", C.c_uint32)]


class Plan(C.Structure):   # ops.hpp, OpPlan
    _fields_ = [("func", C.c_void_p), ("grid", Dim3), ("block", Dim3), ("lds", C.c_size_t)]


def plan(op, shape):
    f = capi.lib()._ZN2ug11plan_kernelERK9ug_kerneli   # ug::plan_kernel
    f.restype, f.argtypes = Plan, [C.POINTER(capi.Kernel), C.c_int]
    n_in = 1 if op == "softmax" else 2
    return f(C.byref(capi.kernel_struct({"op": op, "shape": shape, "in": tuple(range(n_in)),
                                         "out": (n_in,)})), -1)


@pytest.mark.parametrize("op,shape", [
    ("gemm", (680431841, 8, 10)), ("gemm", (3, 1284745033, 2)), ("gemm", ((1 << 31) - 1, 1, 1)),
    ("gemm", (1, (1 << 31) - 1, 1)), ("gemm", ((1 << 31) - 1, 1, 4)),
    ("gemm", (1, (1 << 31) - 1, 4)), ("gemm", (1 << 28, 60, 32)),
    ("gemm_fp8", (2, 1703227788, 32)), ("gemm_fp8", (1611767944, 4, 32)),
    ("gemm_fp8", (1565754663, 1, 16)), ("gemm_bf16", ((1 << 30) - 1, 4, 32)),
    ("conv3x3", (15871663, 30, 2, 2)), ("conv3x3", (5376279, 22, 1, 25)),
    ("conv3x3", (186313, 32, 3, 818)), ("conv3x3", (38502, 30, 7, 3059)),
    ("softmax", (5748708, 12035)), ("softmax", (12495477, 4908)), ("softmax", (4576275, 8675))])
def test_grids_are_within_the_limit(op, shape):
    p = plan(op, shape)
    for grid, block in ((p.grid.x, p.block.x), (p.grid.y, p.block.y), (p.grid.z, p.block.z)):
        assert 0 < grid * block < 1 << 32, (grid, block)
