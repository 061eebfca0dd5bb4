"""What a compute unit has to hold of each kernel beside a worker of the tail
executor (csrc/kernels/fused.hpp), from the built kernels' own metadata.

The executor may hold a worker on every CU for as long as it has work, and a
tail waits there for the contraction whose output it takes: a contraction that
does not start beside a worker would wait for the executor to leave."""

import struct

import msgpack
import pytest

from paper_2509_12207_amd import build

LDS_BYTES, SIMDS, VGPRS, GRANULE = 160 * 1024, 4, 512, 8


def _code_objects(path):
    """The gfx950 code objects bundled in a shared library."""
    data = open(path, "rb").read()
    magic = b"__CLANG_OFFLOAD_BUNDLE__"
    at = data.find(magic)
    while at >= 0:
        n, = struct.unpack_from("<Q", data, at + len(magic))
        pos = at + len(magic) + 8
        for _ in range(n):
            off, size, length = struct.unpack_from("<QQQ", data, pos)
            name = data[pos + 24: pos + 24 + length].decode()
            pos += 24 + length
            if "gfx950" in name and size:
                yield data[at + off: at + off + size]
        at = data.find(magic, at + 1)


def _kernels(elf):
    """The kernels' metadata (the note of type 32 named AMDGPU)."""
    shoff, = struct.unpack_from("<Q", elf, 0x28)
    entry, count = struct.unpack_from("<HH", elf, 0x3A)
    for i in range(count):
        kind, = struct.unpack_from("<I", elf, shoff + i * entry + 4)
        if kind != 7:   # a note section
            continue
        off, size = struct.unpack_from("<QQ", elf, shoff + i * entry + 0x18)
        name_len, desc_len, note = struct.unpack_from("<III", elf, off)
        if note == 32:
            start = off + 12 + (name_len + 3) // 4 * 4
            yield from msgpack.unpackb(elf[start: start + desc_len])["amdhsa.kernels"]


def _all_kernels():
    return [k for elf in _code_objects(build.OUT) for k in _kernels(elf)]


def _needs(k):
    """LDS bytes and registers a SIMD of one workgroup."""
    waves = (k[".max_flat_workgroup_size"] + 63) // 64
    regs = (k[".vgpr_count"] + GRANULE - 1) // GRANULE * GRANULE
    return k[".group_segment_fixed_size"], (waves + SIMDS - 1) // SIMDS * regs


@pytest.fixture(scope="module")
def kernels():
    found = _all_kernels()
    assert len(found) > 50
    return found


def test_kernels_fit_beside_a_tail_worker(kernels):
    worker, = [k for k in kernels if "tail_executor" in k[".name"]]
    lds, regs = _needs(worker)
    tight = {k[".name"]: _needs(k) for k in kernels
             if k is not worker and (_needs(k)[0] + lds > LDS_BYTES or _needs(k)[1] + regs > VGPRS)}
    assert not tight, tight


def test_no_kernel_spills_vector_registers(kernels):
    spilled = {k[".name"]: k[".vgpr_spill_count"] for k in kernels
               if k[".vgpr_spill_count"] and "tail_executor" not in k[".name"]}
    assert not spilled, spilled
