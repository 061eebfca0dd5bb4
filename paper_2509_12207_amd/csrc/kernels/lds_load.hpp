// Loads from global memory straight into LDS, and BF16 operands read from it
// (kernels with a ring of stages in LDS: gemm_lowp.hip, conv3x3_bf16.hip).
//
// The loads are issued from inline assembly so that the compiler, which
// cannot tell them apart from the LDS being read, does not wait for every
// load in flight before each LDS read; their completion is waited for
// explicitly (vmcnt) before a barrier.
#pragma once

#include <hip/hip_runtime.h>

#include "tile_map.hpp"

namespace ug {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
__device__ __forceinline__ bf16x8 as_bf16x8(int4 v) { return __builtin_bit_cast(bf16x8, v); }

// s_waitcnt vmcnt(N): all but this wave's N most recent loads have arrived
template <int N>
__device__ __forceinline__ void wait_loads() {
  asm volatile("s_waitcnt vmcnt(%0)" ::"i"(N) : "memory");
}

// One 16-byte direct-to-LDS load: lane l writes LDS bytes [lds + 16 l, +16).
// M0 holds the wave's LDS base; one wait state between writing M0 and the
// load that reads it.  M0 has no other use in these kernels.
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
__device__ __forceinline__ void load16_lds(const unsigned char* g, unsigned lds) {
  asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" ::"v"(g), "s"(lds)
               : "memory", "m0");
}
#pragma clang diagnostic pop

// 64 zero bytes: a source for what lies outside of an operand
__device__ __attribute__((aligned(64))) unsigned char kZeroSlice[64];

}  // namespace
}  // namespace ug
