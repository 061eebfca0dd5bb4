// Low-precision GEMMs on the matrix cores of gfx950, FP32 result:
//   FP8:  C[M,N] = A[M,K] B[K,N], A and B in OCP FP8 E4M3 (one byte each);
//   BF16: the same with A and B in bfloat16 (two bytes each).
//
// Operands are K-contiguous: A row-major [M, K], B given transposed as
// Bt [N, K] (row n holds column n of B).  M and N are arbitrary (rows past
// M or N are read from the matrix's first row or zero-filled, and never
// stored).  Workgroups are remapped so each XCD computes a contiguous band
// of output tiles.
//
// Instructions (both wave64, accumulator layout of the other 32x32
// instructions, mfma32_row):
// * v_mfma_scale_f32_32x32x64_f8f6f4, both scale exponents 127 (x1):
//   D[32x32] += A[32x64] B[64x32], 131072 FLOP.  Lane l feeds row (A) or
//   column (B) l % 32 with 32 bytes of K: bytes 32 (l / 32) .. +31 of the
//   64-byte K slice.
// * v_mfma_f32_32x32x16_bf16: D[32x32] += A[32x16] B[16x32], 32768 FLOP.
//   Lane l feeds row / column l % 32 with 8 values of K: k = 8 (l / 32) ..
//   +7.  A 64-byte K slice (32 values) takes two of them: lane l reads 16-
//   byte chunk l / 32 for the first and chunk 2 + l / 32 for the second.
//
// One kernel, gemm_ring<type, RAGGED, WM, WN, TM, TN, KS, NST>: a
// workgroup of WM x WN x KS waves computes a (WM*TM*32) x (WN*TN*32) tile,
// each wave TM x TN products of 32 x 32 over every KS-th 64-byte K slice
// (a step).  Global memory goes straight to LDS (global_load_lds_dwordx4)
// into a ring of NST stages per K slice, NST - 1 stages ahead of the matrix
// cores; the fragments of step s+1 are read from LDS while step s runs.  One
// barrier a step.  LDS rows are 64 bytes with the four 16-byte chunks of row
// r XOR-permuted by (r / 4) % 4: a 16-byte read by sixteen consecutive rows
// then touches all 64 LDS banks once.  The direct-to-LDS loads are issued
// from inline assembly so that the compiler, which cannot tell them apart
// from the ring slots being read, does not wait for every load in flight
// before each LDS read; their completion is waited for explicitly (vmcnt)
// before each barrier.  K slices are summed through LDS in a fixed order.
// RAGGED (FP8 rows that are not a multiple of 64 bytes): the chunks past the
// row's end are read from a zero slice.
// PAIR: two stages are loaded together, the two halves of a row's 128-byte
// line by neighbouring loads.  A stage alone fetches half a line, and by the
// next one the rest has left the first-level cache: twice the traffic from
// the second level, which is what bounds large products.  The lead is two
// stages instead of three.
//
// What bounds it, and the tiles: 256 x 256 is bound by the rate at which
// panels stream into LDS (about 9 TB/s over the chip) and needs about 144
// tiles to fill it; anything smaller left most CUs idle, and a short product
// is a chain of steps whose latency (barrier, LDS, loads) K slices divide.
// us per launch, 256 x 256 only -> now: BF16 4096^3 122 -> 117, 2048^3 47 -> 24,
// 1280x1792x768 22 -> 9.2, 1024^3 25 -> 6.5, 512^3 16 -> 4.1, 256x256x2048
// 42 -> 5.9; FP8 2048x8192x8192 122 -> 113 (on one set of operands again and
// again; 122 where they change from launch to launch), 2048^3 27 -> 14, 1024^3
// 15 -> 4.9.
#include "lds_load.hpp"
#include "mfma.hpp"
#include "ops.hpp"
#include "signal.hpp"
#include "submit.hpp"
#include "tile_map.hpp"

namespace ug {
namespace {

typedef int i32x8 __attribute__((ext_vector_type(8)));

// ------------------------------------------------------------ ring kernel
constexpr int RK = 64;                       // bytes of K per step
enum RingType { kRingFp8 = 0, kRingBf16 = 1 };

__device__ __forceinline__ int ring_swz(int row) { return (row >> 2) & 3; }

// The two 16-byte chunks of a 64-byte K slice that lane group g (= lane /
// 32) feeds to the matrix cores.
template <int T>
__device__ __forceinline__ int ring_chunk(int g, int h) {
  return T == kRingFp8 ? 2 * g + h : g + 2 * h;
}

// Geometry of a ring workgroup: WM x WN x KS waves, each with TM x TN tiles
// of 32 x 32 and every KS-th K step; each K slice has a ring of NST stages.
template <int WM, int WN, int TM, int TN, int KS, int NST>
struct Ring {
  static constexpr int BM = WM * TM * 32, BN = WN * TN * 32;
  static constexpr int WAVES = WM * WN;                  // of one K slice
  static constexpr int NT = 64 * WAVES * KS;
  static constexpr int STAGE = (BM + BN) * RK;           // bytes per stage
  static constexpr int BLOCKS = STAGE / 1024;            // one load of a wave each
  static constexpr int CPT = BLOCKS / WAVES;             // loads per wave and stage
  static constexpr int LDS = KS * NST * STAGE;
  static_assert(BLOCKS % WAVES == 0, "even split of the loads");
  static_assert((NST - 1) * CPT < 64, "the wait counts fit vmcnt");
  static_assert(KS == 1 || LDS >= (KS - 1) * WAVES * TM * TN * 4096, "reduction fits in LDS");
};

// Operands: A and Bt as bytes, `kb` bytes per row (a multiple of 64; of 16 if
// RAGGED).
template <int T, bool RAGGED, int WM, int WN, int TM, int TN, int KS, int NST,
          bool PAIR>
__global__ __launch_bounds__(64 * WM * WN * KS, 1) void gemm_ring(
    const unsigned char* __restrict__ A, const unsigned char* __restrict__ Bt,
    float* __restrict__ C, int M, int N, int kb, unsigned* sig) {
  using R = Ring<WM, WN, TM, TN, KS, NST>;
  constexpr int BM = R::BM, BN = R::BN, CPT = R::CPT;
  __shared__ __attribute__((aligned(1024))) unsigned char ring[R::LDS];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wid = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int ks = wid / R::WAVES, wave = wid % R::WAVES;
  const int wm = wave / WN, wn = wave % WN;
  unsigned char* lds = ring + ks * NST * R::STAGE;
  const int tiles_m = (M - 1) / BM + 1, tiles_n = (N - 1) / BN + 1;
  int tm, tn;
  tile_of(blockIdx.x, tiles_m, tiles_n, &tm, &tn);
  const int m0 = tm * BM, n0 = tn * BN;
  const int steps = kb / RK + (RAGGED && kb % RK != 0);
  const int mine = (steps + KS - 1) / KS;   // steps of a K slice (the last may be missing)

  // A stage is BM + BN rows (of A, then of Bt) of 64 bytes; load i of wave w
  // fills the 1 KiB block w * CPT + i, lane l the chunk q = 64 (w CPT + i) + l:
  // row q / 4, stored chunk q % 4, which holds K chunk (q % 4) ^
  // ring_swz(row).  Rows past M or N read the matrix's first row (never
  // stored).
  const unsigned char* src[CPT];
  int kcs[CPT];
  unsigned at[CPT];
#pragma unroll
  for (int i = 0; i < CPT; ++i) {
    at[i] = (wave * CPT + i) * 1024;
    const int q = (wave * CPT + i) * 64 + lane;
    const int row = q >> 2, kc = (q & 3) ^ ring_swz(row);
    const bool isa = row < BM;
    const int grow = isa ? m0 + row : n0 + (row - BM);
    const bool ok = grow < (isa ? M : N);
    const unsigned char* X = isa ? A : Bt;
    src[i] = (ok ? X + (int64_t)grow * kb : X) + 16 * kc;
    kcs[i] = kc;
  }
  // Stages past the end re-load the last K slice into their own slot, which
  // is never read again: every step issues the same number of loads, so the
  // wait counts are constants.
  auto load = [&](int step, int i) {
    const int k0 = min(step * KS + ks, steps - 1) * RK;
    const unsigned to = (unsigned)(uintptr_t)(lds + step % NST * R::STAGE) + at[i];
    const unsigned char* g = src[i] + k0;
    if (RAGGED && k0 + 16 * kcs[i] >= kb) g = kZeroSlice + 16 * kcs[i];
    load16_lds(g, __builtin_amdgcn_readfirstlane(to));
  };
  auto issue = [&](int step) {
#pragma unroll
    for (int i = 0; i < CPT; ++i) load(step, i);
  };
  // two stages, block by block: the two halves of a row's 128 bytes together
  auto issue2 = [&](int step) {
#pragma unroll
    for (int i = 0; i < CPT; ++i) {
      load(step, i);
      load(step + 1, i);
    }
  };

  f32x16 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] = zero16();

  // fragment of the 32 rows from `row0`: this lane's row, its two K chunks
  // (row0 is a multiple of 32, so row0 + r32 has the swizzle of r32)
  const int g = lane >> 5, r32 = lane & 31;
  const int c0 = 16 * (ring_chunk<T>(g, 0) ^ ring_swz(r32));
  const int c1 = 16 * (ring_chunk<T>(g, 1) ^ ring_swz(r32));
  auto frag = [&](const unsigned char* base, int row0) {
    const unsigned char* r = base + (row0 + r32) * RK;
    const int4 x = *reinterpret_cast<const int4*>(r + c0);
    const int4 y = *reinterpret_cast<const int4*>(r + c1);
    i32x8 v;
    v[0] = x.x; v[1] = x.y; v[2] = x.z; v[3] = x.w;
    v[4] = y.x; v[5] = y.y; v[6] = y.z; v[7] = y.w;
    return v;
  };
  auto read = [&](int step, i32x8 (&a)[TM], i32x8 (&b)[TN]) {
    const unsigned char* base = lds + (step % NST) * R::STAGE;
#pragma unroll
    for (int i = 0; i < TM; ++i) a[i] = frag(base, (wm * TM + i) * 32);
#pragma unroll
    for (int j = 0; j < TN; ++j) b[j] = frag(base, BM + (wn * TN + j) * 32);
  };
  auto multiply_row = [&](int i, const i32x8 (&a)[TM], const i32x8 (&b)[TN]) {
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        if constexpr (T == kRingFp8) {
          acc[i][j] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a[i], b[j], acc[i][j], 0, 0,
                                                                      0, 127, 0, 127);
        } else {
#pragma unroll
          for (int h = 0; h < 2; ++h) {
            const int4 x = {a[i][4 * h], a[i][4 * h + 1], a[i][4 * h + 2], a[i][4 * h + 3]};
            const int4 y = {b[j][4 * h], b[j][4 * h + 1], b[j][4 * h + 2], b[j][4 * h + 3]};
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(x), as_bf16x8(y),
                                                                acc[i][j], 0, 0, 0);
          }
        }
      }
  };
  auto multiply = [&](const i32x8 (&a)[TM], const i32x8 (&b)[TN]) {
#pragma unroll
    for (int i = 0; i < TM; ++i) multiply_row(i, a, b);
  };
  // Step s: wait until stage s+1 is in LDS for every wave (this wave's loads
  // but the NST - 2 latest stages, then the barrier) and this wave's reads of
  // stage s are done; refill the slot of stage s (its fragments are in
  // registers) with stage s+NST; read stage s+1 (past the end: stale bytes,
  // never used); multiply stage s.
  auto step = [&](int s, const i32x8 (&ca)[TM], const i32x8 (&cb)[TN], i32x8 (&na)[TM],
                  i32x8 (&nb)[TN]) {
    wait_loads<(NST - 2) * CPT>();
    __builtin_amdgcn_s_waitcnt(kWaitLdsOnly);
    asm volatile("s_barrier" ::: "memory");
    issue(s + NST);
    read(s + 1, na, nb);
    if (KS == 1 || s * KS + ks < steps) multiply(ca, cb);
  };

  i32x8 a0[TM], b0[TN], a1[TM], b1[TN];
  if constexpr (PAIR) {
    static_assert(NST == 4 && KS == 1, "two pairs of stages, one K slice");
    issue2(0);
    issue2(2);
    wait_loads<2 * CPT>();
    asm volatile("s_barrier" ::: "memory");
    read(0, a0, b0);
    // row by row, so that one set of A's fragments is enough: a row's is read
    // again for the next step once its products are issued (256 x 256: 214
    // registers, 240 with two sets; 216 fit beside a wave of the tail executor)
    auto half = [&](int next, const i32x8 (&b)[TN], i32x8 (&bn)[TN]) {
      const unsigned char* base = lds + (next % NST) * R::STAGE;
#pragma unroll
      for (int j = 0; j < TN; ++j) bn[j] = frag(base, BM + (wn * TN + j) * 32);
#pragma unroll
      for (int i = 0; i < TM; ++i) {
        multiply_row(i, a0, b);
        __builtin_amdgcn_sched_barrier(0);
        a0[i] = frag(base, (wm * TM + i) * 32);
      }
    };
    for (int s = 0; s < mine; s += 2) {
      half(s + 1, b0, b1);
      // stages s, s + 1 are in registers in every wave, s + 2 and s + 3 in LDS
      wait_loads<0>();
      __builtin_amdgcn_s_waitcnt(kWaitLdsOnly);
      asm volatile("s_barrier" ::: "memory");
      issue2(s + 4);
      if (s + 1 < mine) half(s + 2, b1, b0);
    }
  } else {
    for (int s = 0; s < NST; ++s) issue(s);
    wait_loads<(NST - 1) * CPT>();
    asm volatile("s_barrier" ::: "memory");
    read(0, a0, b0);
    for (int s = 0; s < mine; s += 2) {
      step(s, a0, b0, a1, b1);
      if (s + 1 < mine) step(s + 1, a1, b1, a0, b0);
    }
  }
  // no load may still be writing LDS when the workgroup ends
  wait_loads<0>();

  if (KS > 1) {
    // K slices 1..KS-1 hand their sums to slice 0 through LDS, added in order
    constexpr int PER = TM * TN * 16 * 64;   // floats per wave
    float* red = reinterpret_cast<float*>(ring);
    __syncthreads();
    if (ks > 0) {
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
          for (int r = 0; r < 16; ++r)
            red[((ks - 1) * R::WAVES + wave) * PER + ((i * TN + j) * 16 + r) * 64 + lane] =
                acc[i][j][r];
    }
    __syncthreads();
    if (ks > 0) {   // handed over: meet slice 0 at the counter's barrier, then leave
      group_done(sig);
      return;
    }
#pragma unroll
    for (int s = 1; s < KS; ++s)
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
          for (int r = 0; r < 16; ++r)
            acc[i][j][r] += red[((s - 1) * R::WAVES + wave) * PER + ((i * TN + j) * 16 + r) * 64 + lane];
  }

#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const int col = n0 + (wn * TN + j) * 32 + r32;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int row = m0 + (wm * TM + i) * 32 + mfma32_row(r, lane);
        if (row < M && col < N) C[(int64_t)row * N + col] = acc[i][j][r];
      }
    }
  group_done(sig);
}

struct Launch {
  const void* func;
  int bm, bn, nt;
};
template <int T, bool RAGGED, int WM, int WN, int TM, int TN, int KS, int NST,
          bool PAIR = false>
Launch ring() {
  using R = Ring<WM, WN, TM, TN, KS, NST>;
  return {reinterpret_cast<const void*>(
              &gemm_ring<T, RAGGED, WM, WN, TM, TN, KS, NST, PAIR>),
          R::BM, R::BN, R::NT};
}

int64_t tiles(int64_t M, int64_t N, int bm, int bn) { return ((M + bm - 1) / bm) * ((N + bn - 1) / bn); }

// The tile by the number of workgroups it gives (us at either side of a line):
// * 256 x 256 from 144 workgroups on (BF16 2560x4096x1024, 160: 30.5 against
//   32.2 for 128 x 128; 2304x3072x768, 108: 23.9 against 19.7), unless the
//   edges would be mostly padding;
// * 128 x 128 where 64 x 64 would take more than two rounds of 256 CUs
//   (1280x1792x768, 560 / 140 workgroups: 9.2 against 11.4; 1024x2048x1024,
//   512 / 128: 10.9 against 10.0), with the same exception;
// * 32 x 32 with eight K slices for few workgroups and a long K (512x512x2048
//   6.4 against 7.1 for 32 x 64, 512^3 4.6 against 4.1);
// * 32 x 64 with two K slices up to 128 workgroups of 64 x 64 (512x1024x512
//   4.2 against 4.7; 768x1024x512, 192: 5.2 against 4.9);
// * 64 x 64, with two K slices where one round of CUs holds them all and K is
//   long (1024^3 6.5 against 7.0; K = 512: equal).
// Stages in pairs where workgroups enough hide the shorter lead (us single ->
// pairs): 256 x 256 from 192 workgroups (4096^3 121.5 -> 118, FP8
// 2048x8192x8192 122 -> 113; 3072x3072x2048, 144: 47.8 -> 50.1), 128 x 128 from
// two a CU (2304x3072x768 19.5 -> 17.9, FP8 2048x4096x4096 44 -> 37.8; 2048^3,
// 256: 23.3 -> 26.6), 64 x 64 always (1024x2048x1024 9.5 -> 8.5).
template <int T, bool RAGGED>
Launch pick_ring(int64_t M, int64_t N, int64_t kb) {
  const int64_t steps = (kb + RK - 1) / RK;
  const int64_t t256 = tiles(M, N, 256, 256), t128 = tiles(M, N, 128, 128);
  const int64_t t64 = tiles(M, N, 64, 64), t32 = tiles(M, N, 32, 32);
  // (past the most threads a grid holds, the tile with the fewest for its size:
  // a narrow product of 2^30 rows or more)
  if ((t256 >= 144 && 3 * t256 <= t128) || 256 * t64 > kMaxGridThreads)
    return t256 >= 192 ? ring<T, RAGGED, 2, 4, 4, 2, 1, 4, true>()
                       : ring<T, RAGGED, 2, 4, 4, 2, 1, 4>();
  if (t64 > 512 && 3 * t128 <= t64)
    return t128 > 256 ? ring<T, RAGGED, 2, 4, 2, 1, 1, 4, true>()
                      : ring<T, RAGGED, 2, 4, 2, 1, 1, 4>();
  if (t32 <= 256 && steps >= 64) return ring<T, RAGGED, 1, 1, 1, 1, 8, 4>();
  if (t64 <= 128) return ring<T, RAGGED, 1, 2, 1, 1, 2, 4>();
  if (t64 <= 256 && steps >= 32) return ring<T, RAGGED, 2, 2, 1, 1, 2, 4>();
  return ring<T, RAGGED, 2, 2, 1, 1, 1, 4, true>();
}

OpPlan ring_plan(const Launch& l, int64_t M, int64_t N) {
  OpPlan p;
  p.func = l.func;
  p.grid = dim3((unsigned)(((M + l.bm - 1) / l.bm) * ((N + l.bn - 1) / l.bn)));
  p.block = dim3(l.nt);
  return p;
}

hipError_t ring_launch(const OpPlan& p, const void* A, const void* Bt, float* C, int64_t M,
                       int64_t N, int64_t kb, unsigned* sig, hipStream_t s) {
  int m = (int)M, n = (int)N, k = (int)kb;
  void* args[] = {&A, &Bt, &C, &m, &n, &k, &sig};
  return submit(p, args, s);
}

}  // namespace

OpPlan gemm_fp8_plan(int64_t M, int64_t N, int64_t K) {
  return ring_plan(K % RK == 0 ? pick_ring<kRingFp8, false>(M, N, K)
                               : pick_ring<kRingFp8, true>(M, N, K), M, N);
}

hipError_t gemm_fp8_launch(const unsigned char* A, const unsigned char* Bt, float* C, int64_t M,
                           int64_t N, int64_t K, hipStream_t s) {
  return ring_launch(gemm_fp8_plan(M, N, K), A, Bt, C, M, N, K, nullptr, s);
}

OpPlan gemm_bf16_plan(int64_t M, int64_t N, int64_t K) {
  return ring_plan(pick_ring<kRingBf16, false>(M, N, 2 * K), M, N);
}

hipError_t gemm_bf16_launch(const uint16_t* A, const uint16_t* Bt, float* C, int64_t M,
                            int64_t N, int64_t K, hipStream_t s, unsigned* sig) {
  return ring_launch(gemm_bf16_plan(M, N, K), A, Bt, C, M, N, 2 * K, sig, s);
}

}  // namespace ug
