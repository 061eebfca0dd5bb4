// C[M,N] = A[M,K] B[K,N], row-major FP32, on gfx950.
//
// Every value is split into three bfloat16 pieces as it is staged, and the
// products are formed by the BF16 matrix instruction (split.hpp: the error
// against fp64 is 0.28-0.48 of the FP32 instruction's from K = 32 on, the matrix
// cycles 2.67 times fewer).  K = 1 and 2 and tiles that hold a value without a
// split are computed by the FP32 instruction (exact_tile); one NaN in every
// tile, us: 4096^3 2056, 1003x2050x1021 135, 1024^3 47, 256^3 10.5.
//
// One kernel template <WM, WN, TM, TN, KS, BK, U, PF>: the workgroup tile is
// (WM*TM*32) x (WN*TN*32); its waves form a WM x WN x KS grid; each wave owns
// TM x TN tiles of 32 x 32 and one of KS slices (BK values) of every K step;
// operands are staged in units of U K values.
//   big   <2,4,2,1,1,16,4>: 128 x 128 tiles, eight waves of 64 x 32,
//         <2,2,2,2,2,16,4>: the same in waves of 64 x 64, K split two ways, or
//         <4,2,2,2,1,16,4>: 256 x 128 tiles, eight waves of 64 x 64;
//   mid   <2,2,1,1,2,16,4> or, where K is long and no CU has more than one
//         tile, <2,2,1,1,4,16,4>: 64 x 64, K split two or four ways;
//   small <1,1,1,1,4,16,8> or <1,1,1,1,8,16,4>: 32 x 32, K split four or
//         eight ways.
// K slices are summed through LDS in a fixed order (results do not depend on
// scheduling).
//
// What bounds it: at 4096^3 the matrix cores; six BF16 instructions per 16
// products sustain 1.3 PFLOP/s there, more than the library's 8192^3 BF16
// product (1.12) on the same card.  Smaller products are bound by the latency
// of a step (global load, split, LDS, barrier) in the few waves a CU has,
// hence eight waves for 128 x 128 (two such workgroups make four waves a
// SIMD at 126 registers; four waves of 64 x 64 took 695 us at 4096^3 against
// 670) and the K splits.  One tile of 256 x 128 loads and splits a quarter
// less than two of 128 x 128 (4096^3: 661 -> 640 us).
// (Figures side by side are of one session; sessions differ by up to 5 % at
// 4096^3, where the clock gives way, and by 1 to 3 % below.)
// us per launch, launched in a row, FP32 instruction before -> now:
//   4096^3 1109 -> 631, 2048^3 164 -> 92, 1280x2048x1024 65 -> 42,
//   1003x2050x1021 98 -> 41.5, 1024^3 33 -> 18.1, 768x1280x256 11.0 -> 7.4,
//   512^3 8.8 -> 7.3, 256x256x2048 26 -> 16.6, 256^3 5.8 -> 5.7.
//
// The pipeline of a step: while the products of the m pieces run, the next
// step's values (in registers, loaded a step ahead) are split and written to
// the other LDS buffer, six and a half vector instructions per value
// interleaved with the matrix instructions; after the step's only barrier the
// next fragments are read under the remaining products.  The barrier waits for
// LDS only (__syncthreads would also drain the global loads).
//
// Workgroups are dispatched round-robin over the 8 XCDs; the linear id is
// remapped so each XCD works on a contiguous band of output tiles (sharing A
// and B panels in its own L2), walked in groups of 8 tile-rows.
#include "mfma.hpp"
#include "ops.hpp"
#include "signal.hpp"
#include "split.hpp"
#include "submit.hpp"
#include "tile_map.hpp"

namespace ug {
namespace {

template <int WM, int WN, int TM, int TN, int KS, int BK, int U>
struct GemmCfg {
  static constexpr int NT = 64 * WM * WN * KS;         // threads
  static constexpr int BM = WM * TM * 32, BN = WN * TN * 32;
  static constexpr int BKT = BK * KS;                  // K values per step
  static constexpr int ROWS = BM + BN;                 // LDS rows: A's, then B's
  static constexpr int ROWB = 2 * BK;                  // bytes per LDS row and piece
  static constexpr int PIECE = ROWS * ROWB;            // bytes
  static constexpr int STAGE = KS * 3 * PIECE;
  static constexpr int UPR = BKT / U;                  // units per row and step
  static constexpr int AU = BM * UPR / NT, BU = BN * UPR / NT;   // units per thread
  static constexpr int LDS = 2 * STAGE;                // bytes
  static constexpr int RAW = BKT + 1;                  // floats per row of unsplit values
  static_assert(BK == 16, "one matrix instruction per row");
  static_assert(BM * UPR % NT == 0 && BN * UPR % NT == 0, "even split of the units");
  static_assert(LDS >= 4 * ROWS * RAW, "unsplit values fit in LDS");
  static_assert(KS == 1 || LDS >= (KS - 1) * 4096 * TM * TN * WM * WN, "reduction fits in LDS");
};

// The two 16-byte chunks of a row are permuted so that a read of one chunk by
// sixteen consecutive rows touches all 64 LDS banks once.
__device__ __forceinline__ int swz(int row) { return (row >> 3) & 1; }

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef __amdgpu_buffer_rsrc_t rsrc_t;
__device__ __forceinline__ rsrc_t make_rsrc(const void* p) {   // raw, unbounded
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, -1, 0x00027000);
}
__device__ __forceinline__ float buffer_load4(rsrc_t r, uint32_t off, uint32_t soff) {
  return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, off, soff, 0));
}
__device__ __forceinline__ u32x4 buffer_load16(rsrc_t r, uint32_t off, uint32_t soff) {
  return __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(r, off, soff, 0));
}

// Issue order of what precedes: N times a matrix instruction, then V vector
// instructions in its shadow.
template <int N, int V>
__device__ __forceinline__ void interleave() {
#pragma unroll
  for (int i = 0; i < N; ++i) {
    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
    __builtin_amdgcn_sched_group_barrier(0x002, V, 0);
  }
  __builtin_amdgcn_sched_barrier(0);
}

// Stores a wave's tile, its first row m0 and column n0.
template <int TM, int TN>
__device__ __forceinline__ void store_tile(const f32x16 (&acc)[TM][TN], float* __restrict__ C, int M,
                                           int N, int m0, int n0) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const int n = n0 + 32 * j + (lane & 31);
      if (n >= N) continue;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int m = m0 + 32 * i + mfma32_row(r, lane);
        if (m < M) C[(size_t)m * N + n] = acc[i][j][r];
      }
    }
}

// A workgroup's tile with the FP32 instruction, on the values as they are
// (inputs without a split, and sums too short for one): the same K slices, one
// buffer of FP32 rows a step, the next step's values in registers.  The
// thread's index is hidden from the compiler, which would otherwise keep what
// it has in common with the kernel's in registers throughout.
template <int WM, int WN, int TM, int TN, int KS, int BK, int U>
__device__ __forceinline__ void exact_tile(f32x16 (&acc)[TM][TN], float* raw,
                                           const float* __restrict__ A,
                                           const float* __restrict__ B, int M, int N, int K, int m0,
                                           int n0) {
  using G = GemmCfg<WM, WN, TM, TN, KS, BK, U>;
  constexpr int BM = G::BM, BN = G::BN, BKT = G::BKT, NT = G::NT, UPR = G::UPR;
  int tid = threadIdx.x;
  asm("" : "+v"(tid));
  const int half = tid >> 5 & 1, col = tid & 31, wave = tid >> 6;
  const int ks = wave / (WM * WN), wm = wave % (WM * WN) / WN, wn = wave % WN;
  float ra[G::AU][U], rb[G::BU][U];
  auto load = [&](int64_t k0) {
#pragma unroll
    for (int i = 0; i < G::AU; ++i) {
      const int u = tid + NT * i, m = min(m0 + u / UPR, M - 1);
#pragma unroll
      for (int j = 0; j < U; ++j) {
        const int64_t k = k0 + U * (u % UPR) + j;
        ra[i][j] = k < K ? A[(size_t)m * K + k] : 0.f;
      }
    }
#pragma unroll
    for (int i = 0; i < G::BU; ++i) {
      const int u = tid + NT * i, n = min(n0 + u % BN, N - 1);
#pragma unroll
      for (int j = 0; j < U; ++j) {
        const int64_t k = k0 + U * (u / BN) + j;
        rb[i][j] = k < K ? B[(size_t)k * N + n] : 0.f;
      }
    }
  };
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] = zero16();
  const float* x = raw + (wm * TM * 32 + col) * G::RAW + ks * BK + half;
  const float* y = raw + (BM + wn * TN * 32 + col) * G::RAW + ks * BK + half;
  load(0);
#pragma clang loop unroll(disable)
  for (int64_t k0 = 0; k0 < K; k0 += BKT) {
#pragma unroll
    for (int i = 0; i < G::AU; ++i)
#pragma unroll
      for (int j = 0; j < U; ++j) {
        const int u = tid + NT * i;
        raw[u / UPR * G::RAW + U * (u % UPR) + j] = ra[i][j];
      }
#pragma unroll
    for (int i = 0; i < G::BU; ++i)
#pragma unroll
      for (int j = 0; j < U; ++j) {
        const int u = tid + NT * i;
        raw[(BM + u % BN) * G::RAW + U * (u / BN) + j] = rb[i][j];
      }
    __syncthreads();
    if (k0 + BKT < K) load(k0 + BKT);
#pragma unroll
    for (int k = 0; k < BK; k += 2)
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
          acc[i][j] = mfma_32x32x2(x[i * 32 * G::RAW + k], y[j * 32 * G::RAW + k], acc[i][j]);
    __syncthreads();   // read, and at the end free for the sums of the K slices
  }
}

// Sums of too few products for the split: exact_tile alone.
template <int WM, int WN, int TM, int TN, int BK, int U>
__global__ __launch_bounds__(64 * WM * WN) void gemm_f32_short(const float* __restrict__ A,
                                                               const float* __restrict__ B,
                                                               float* __restrict__ C, int M, int N,
                                                               int K, unsigned* sig) {
  using G = GemmCfg<WM, WN, TM, TN, 1, BK, U>;
  __shared__ float raw[G::ROWS * G::RAW];
  const int tiles_m = (M - 1) / G::BM + 1, tiles_n = (N - 1) / G::BN + 1;
  const int wg = blockIdx.y * gridDim.x + blockIdx.x;   // (two sides where one is too long)
  if (wg < tiles_m * tiles_n) {
    int tm, tn;
    tile_of(wg, tiles_m, tiles_n, &tm, &tn);
    f32x16 acc[TM][TN];
    exact_tile<WM, WN, TM, TN, 1, BK, U>(acc, raw, A, B, M, N, K, tm * G::BM, tn * G::BN);
    const int wave = threadIdx.x >> 6;
    store_tile<TM, TN>(acc, C, M, N, tm * G::BM + wave / WN * TM * 32, tn * G::BN + wave % WN * TN * 32);
  }
  group_done(sig);
}

// Registers: a workgroup fits on a SIMD beside a wave of the tail executor
// (80 of 512), that is two waves a SIMD take 216 each at most (the attribute
// counts half of the unified registers), four 104.
template <int WM, int WN, int TM, int TN, int KS, int BK, int U, int PF, bool WIDE>
__attribute__((amdgpu_num_vgpr(108))) __global__
__launch_bounds__(64 * WM * WN * KS, (TM * TN < 4 && WM * WN * KS >= 8 ? 4 : 2)) void gemm_f32_kernel(
    const float* __restrict__ A, const float* __restrict__ B, float* __restrict__ C, int M, int N,
    int K, unsigned* sig) {
  using G = GemmCfg<WM, WN, TM, TN, KS, BK, U>;
  constexpr int BM = G::BM, BN = G::BN, BKT = G::BKT, NT = G::NT, UPR = G::UPR;
  __shared__ __attribute__((aligned(1024))) unsigned char lds[G::LDS];
  __shared__ int redo;

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int ks = wave / (WM * WN);
  const int wm = (wave % (WM * WN)) / WN, wn = wave % WN;
  const int tiles_m = (M - 1) / BM + 1, tiles_n = (N - 1) / BN + 1;
  int wg = blockIdx.x;
  if constexpr (WIDE) {   // (a grid of two sides where one would be too long)
    wg += blockIdx.y * gridDim.x;
    if (wg >= tiles_m * tiles_n) {
      group_done(sig);
      return;
    }
  }
  int tm, tn;
  tile_of(wg, tiles_m, tiles_n, &tm, &tn);
  const int m0 = tm * BM, n0 = tn * BN;
  if (tid == 0) redo = 0;

  // Staging units: eight K values of a row of A (contiguous in memory) or of
  // a column of B (eight rows, consecutive threads on consecutive columns).
  // Rows past M or N repeat the last one (their results are not stored).
  // Loads are buffer loads: a resource that starts at the tile's first row or
  // column and moves along K by scalar arithmetic, an offset per thread that
  // stays, and a scalar offset per K row of B (no vector address arithmetic;
  // A is read 16 bytes at a time at any alignment of its rows).  WIDE: K or N
  // too large for 32-bit offsets, plain loads.
  uint32_t pa[G::AU], pb[G::BU];  // byte offsets
  int ra_row[G::AU], rb_col[G::BU];
  int ka[G::AU], kb[G::BU];       // first K value of the unit in a step
  int oa[G::AU], ob[G::BU];       // its LDS place (piece 0)
  const auto place = [](int r, int q) {
    const int k = q * U % BK;   // in the row
    return q * U / BK * 3 * G::PIECE + r * G::ROWB + 16 * ((k / 8) ^ swz(r)) + 2 * (k % 8);
  };
#pragma unroll
  for (int i = 0; i < G::AU; ++i) {
    const int u = tid + NT * i, r = u / UPR, q = u % UPR;
    ka[i] = U * q;
    ra_row[i] = min(m0 + r, M - 1);
    pa[i] = ((uint32_t)(ra_row[i] - m0) * (uint32_t)K + U * q) * 4;
    oa[i] = place(r, q);
  }
#pragma unroll
  for (int i = 0; i < G::BU; ++i) {
    const int u = tid + NT * i, r = u % BN, q = u / BN;
    kb[i] = U * q;
    rb_col[i] = min(n0 + r, N - 1);
    pb[i] = ((uint32_t)(rb_col[i] - n0) + (uint32_t)(U * q) * (uint32_t)N) * 4;
    ob[i] = place(BM + r, q);
  }
  const float* a0 = A + (size_t)m0 * K;
  const float* b0 = B + n0;

  // PF sets of registers: each is filled PF steps before it is staged
  float ra[PF][G::AU][U], rb[PF][G::BU][U];
  auto load_a = [&](int k0, float (&ra)[G::AU][U]) {
    const rsrc_t rs = make_rsrc(a0 + k0);
#pragma unroll
    for (int i = 0; i < G::AU; ++i)
#pragma unroll
      for (int j = 0; j < U; j += 4) {
        if constexpr (!WIDE) {
          const u32x4 v = buffer_load16(rs, pa[i] + 4 * j, 0);
#pragma unroll
          for (int t = 0; t < 4; ++t) ra[i][j + t] = __uint_as_float(v[t]);
        } else {
#pragma unroll
          for (int t = 0; t < 4; ++t)
            ra[i][j + t] = A[(size_t)ra_row[i] * K + k0 + ka[i] + j + t];
        }
      }
  };
  auto load_b = [&](int k0, float (&rb)[G::BU][U]) {
    const rsrc_t rs = make_rsrc(b0 + (size_t)k0 * N);
#pragma unroll
    for (int i = 0; i < G::BU; ++i)
#pragma unroll
      for (int j = 0; j < U; ++j)
        rb[i][j] = WIDE ? B[(size_t)(k0 + kb[i] + j) * N + rb_col[i]]
                        : buffer_load4(rs, pb[i], j * N * 4);
  };
  // the first step: its K values from `kn` on are zero
  auto load_first = [&](int kn, float (&ra)[G::AU][U], float (&rb)[G::BU][U]) {
#pragma unroll
    for (int i = 0; i < G::AU; ++i)
#pragma unroll
      for (int j = 0; j < U; ++j) {
        const int k = ka[i] + j;
        const float v = A[(size_t)ra_row[i] * K + min(k, kn - 1)];
        ra[i][j] = k < kn ? v : 0.f;
      }
#pragma unroll
    for (int i = 0; i < G::BU; ++i)
#pragma unroll
      for (int j = 0; j < U; ++j) {
        const int k = kb[i] + j;
        const float v = B[(size_t)min(k, kn - 1) * N + rb_col[i]];
        rb[i][j] = k < kn ? v : 0.f;
      }
  };
  auto put = [&](const float (&x)[U], unsigned char* at) {
    uint32_t p[3][U / 2];
#pragma unroll
    for (int j = 0; j < U / 2; ++j)
      split2(x[2 * j], x[2 * j + 1], &p[0][j], &p[1][j], &p[2][j]);
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      if constexpr (U == 8)
        *reinterpret_cast<uint4*>(at + j * G::PIECE) = make_uint4(p[j][0], p[j][1], p[j][2], p[j][3]);
      else
        *reinterpret_cast<uint2*>(at + j * G::PIECE) = make_uint2(p[j][0], p[j][1]);
    }
  };
  auto store_a = [&](const float (&ra)[G::AU][U]) {
#pragma unroll
    for (int i = 0; i < G::AU; ++i) put(ra[i], lds + oa[i]);
  };
  auto store_b = [&](const float (&rb)[G::BU][U]) {
#pragma unroll
    for (int i = 0; i < G::BU; ++i) put(rb[i], lds + ob[i]);
  };

  const int half = lane >> 5, col = lane & 31;
  constexpr int KH = BK / 16;   // matrix instructions per row and product
  uint4 a[3][KH][TM], b[3][KH][TN];   // this wave's fragments, by piece
  // (their rows start at a multiple of 32, so they have row col's permutation)
  int fa[KH], fb[KH];
#pragma unroll
  for (int h = 0; h < KH; ++h) {
    const int c = ks * 3 * G::PIECE + 16 * ((2 * h + half) ^ swz(col));
    fa[h] = c + (wm * TM * 32 + col) * G::ROWB;
    fb[h] = c + (BM + wn * TN * 32 + col) * G::ROWB;
  }
  auto frag = [&](int p) {
#pragma unroll
    for (int h = 0; h < KH; ++h) {
#pragma unroll
      for (int i = 0; i < TM; ++i)
        a[p][h][i] = *reinterpret_cast<const uint4*>(lds + fa[h] + p * G::PIECE +
                                                     i * 32 * G::ROWB);
#pragma unroll
      for (int j = 0; j < TN; ++j)
        b[p][h][j] = *reinterpret_cast<const uint4*>(lds + fb[h] + p * G::PIECE +
                                                     j * 32 * G::ROWB);
    }
  };
  // to the other buffer
  int stage = G::STAGE;
  auto flip = [&]() {
#pragma unroll
    for (int i = 0; i < G::AU; ++i) oa[i] += stage;
#pragma unroll
    for (int i = 0; i < G::BU; ++i) ob[i] += stage;
#pragma unroll
    for (int h = 0; h < KH; ++h) {
      fa[h] += stage;
      fb[h] += stage;
    }
    stage = -stage;
  };
  f32x16 ah[TM][TN], as[TM][TN];   // sums of hh, of the other five products
  auto mul = [&](int p, int q, f32x16 (&d)[TM][TN]) {
#pragma unroll
    for (int h = 0; h < KH; ++h)
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) d[i][j] = mfma_bf16(a[p][h][i], b[q][h][j], d[i][j]);
  };

  // The first step takes what K leaves over from whole ones.  Step kt: the
  // next step's values are split and written to the other buffer among the
  // products of m, and its fragments are read after the barrier, each piece
  // once this step's products of it are done.
  const int nk = (K - 1) / BKT + 1;
  const int first = K - (nk - 1) * BKT;
  if (TM * TN == 1 && first == BKT) {   // (the big tile has no registers for a branch)
    load_a(0, ra[0]);
    load_b(0, rb[0]);
  } else {
    load_first(first, ra[0], rb[0]);
  }
  store_a(ra[0]);
  store_b(rb[0]);
  // K value where step i starts; past the end the last one again, never used
  auto at = [&](int i) { return first + (min(i, nk - 1) - 1) * BKT; };
  if (nk > 1) {
#pragma unroll
    for (int i = 0; i < PF; ++i) {
      load_a(at(i + 1), ra[i]);
      load_b(at(i + 1), rb[i]);
    }
  }
  lds_barrier();
  frag(1);
  frag(2);
  frag(0);
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) ah[i][j] = as[i][j] = zero16();
  __builtin_amdgcn_s_waitcnt(kWaitLdsOnly);
  auto step = [&](int kt, float (&ra)[G::AU][U], float (&rb)[G::BU][U]) {
    flip();
    const int k2 = at(kt + 1 + PF);
    mul(1, 1, as);
    store_a(ra);
    load_a(k2, ra);
    interleave<KH * TM * TN, (13 * U / 2 * G::AU + KH * TM * TN - 1) / (KH * TM * TN)>();
    mul(1, 0, as);
    store_b(rb);
    load_b(k2, rb);
    interleave<KH * TM * TN, (13 * U / 2 * G::BU + KH * TM * TN - 1) / (KH * TM * TN)>();
    mul(0, 1, as);
    __builtin_amdgcn_sched_barrier(0);
    lds_barrier();
    frag(1);
    __builtin_amdgcn_sched_barrier(0);
    mul(2, 0, as);
    mul(0, 2, as);
    __builtin_amdgcn_sched_barrier(0);
    frag(2);
    __builtin_amdgcn_sched_barrier(0);
    mul(0, 0, ah);
    frag(0);
    __builtin_amdgcn_sched_barrier(0);
  };
#pragma clang loop unroll(disable)
  for (int kt = 0; kt + 1 < nk;) {
#pragma unroll
    for (int i = 0; i < PF; ++i) {
      step(kt, ra[i], rb[i]);
      if (++kt + 1 >= nk) break;
    }
  }
  mul(1, 1, as);
  mul(1, 0, as);
  mul(0, 1, as);
  mul(2, 0, as);
  mul(0, 2, as);
  mul(0, 0, ah);

  bool bad = false;
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      ah[i][j] += as[i][j];
      bad = bad || !finite16(ah[i][j]);
      ah[i][j] *= kSplitUnscale;
    }
  if (bad) redo = 1;
  __syncthreads();   // also: every read of the stages is done
  if (redo)
    exact_tile<WM, WN, TM, TN, KS, BK, U>(ah, reinterpret_cast<float*>(lds), A, B, M, N, K, m0, n0);

  if (KS > 1) {
    // K slices 1..KS-1 hand their partial sums to slice 0 through LDS; slice
    // 0 adds them in slice order.
    constexpr int PER = TM * TN * 16 * 64;   // floats per wave
    float* red0 = reinterpret_cast<float*>(lds);
    if (ks > 0) {
      float* red = red0 + (ks - 1) * PER * (WM * WN) + (wave % (WM * WN)) * PER;
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
          for (int r = 0; r < 16; ++r) red[((i * TN + j) * 16 + r) * 64 + lane] = ah[i][j][r];
    }
    __syncthreads();
    if (ks > 0) {   // handed over: meet slice 0 at the counter's barrier, then leave
      group_done(sig);
      return;
    }
#pragma unroll
    for (int s = 1; s < KS; ++s) {
      const float* red = red0 + (s - 1) * PER * (WM * WN) + (wave % (WM * WN)) * PER;
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
          for (int r = 0; r < 16; ++r) ah[i][j][r] += red[((i * TN + j) * 16 + r) * 64 + lane];
    }
  }

  store_tile<TM, TN>(ah, C, M, N, m0 + wm * TM * 32, n0 + wn * TN * 32);
  group_done(sig);
}

int64_t rounds(int64_t tiles) { return (tiles + 255) / 256; }   // of one tile per CU

enum Shape { kBig = 0, kMid = 1, kSmall = 2 };

int64_t tiles(int64_t M, int64_t N, int bm, int bn) { return ((M + bm - 1) / bm) * ((N + bn - 1) / bn); }

// Two 64 x 64 workgroups share a CU, and up to 512 of them finish together;
// past that 128 x 128 is faster (1280x2048x1024, 640 / 160 tiles: 42 against
// 44 us; 1024x2048x1024, 512 / 128: 41 against 32), unless the matrix's edge
// would leave a quarter of its work as padding.  64 x 64 needs about 128
// tiles to beat 32 x 32 (768x768x512, 144 / 576 tiles: 11.2 against 13.9 us;
// 512x768x512, 96 / 384: 10.3 against 9.5).
Shape pick(int64_t M, int64_t N) {
  const int64_t t64 = tiles(M, N, 64, 64);
  if (t64 > 512 && 3 * tiles(M, N, 128, 128) <= t64) return kBig;
  return t64 >= 128 ? kMid : kSmall;
}

// The variant asked for, else the tuning table's, else the rule above.
Shape choose(int64_t M, int64_t N, int64_t K, int variant) {
  if (variant < 0) {
    const int64_t key[4] = {M, N, K, 0};
    variant = tune_get(UG_OP_GEMM_F32, key);
  }
  return variant >= 0 && variant < 3 ? static_cast<Shape>(variant) : pick(M, N);
}

OpPlan plan_of(const void* func, int threads, int64_t tiles) {
  OpPlan p;
  p.func = func;
  p.block = dim3(threads);
  const int64_t sides = tiles * threads / kMaxGridThreads + 1;
  p.grid = dim3((unsigned)((tiles + sides - 1) / sides), (unsigned)sides);
  return p;
}
template <int WM, int WN, int TM, int TN, int KS, int BK, int U, int PF, bool WIDE>
OpPlan plan_at(int64_t M, int64_t N) {
  return plan_of(reinterpret_cast<const void*>(&gemm_f32_kernel<WM, WN, TM, TN, KS, BK, U, PF, WIDE>),
                 64 * WM * WN * KS, tiles(M, N, WM * TM * 32, WN * TN * 32));
}
// PFW: sets of registers of the WIDE instance
template <int WM, int WN, int TM, int TN, int KS, int BK, int U, int PF, int PFW = PF>
OpPlan plan(int64_t M, int64_t N, bool wide) {
  return wide ? plan_at<WM, WN, TM, TN, KS, BK, U, PFW, true>(M, N)
              : plan_at<WM, WN, TM, TN, KS, BK, U, PF, false>(M, N);
}

}  // namespace

OpPlan gemm_f32_plan(int64_t M, int64_t N, int64_t K, bool, int variant) {
  // 32-bit offsets within a step's panels: up to 256 rows of K values, 16 of N.
  // Long columns: the grid may have a second side.
  const bool wide = K >= (1 << 22) || N >= (1 << 22) || M >= (1 << 28);
  if (K < kSplitMinTerms)
    return plan_of(reinterpret_cast<const void*>(&gemm_f32_short<2, 2, 1, 1, 16, 4>), 256,
                   tiles(M, N, 64, 64));
  switch (choose(M, N, K, variant)) {
    case kBig:
      // one 256 x 128 tile in the place of a CU's two of 128 x 128, where
      // they fill the CUs and leave no more of the last round idle (4096^3,
      // 512 / 1024 tiles: 640 against 661 us; 2048x4096x2048, 256 / 512: 166
      // against 173; 3000x3001x1000, 288 / 576: 148 against 118)
      if (tiles(M, N, 256, 128) >= 256 &&
          2 * rounds(tiles(M, N, 256, 128)) <= rounds(tiles(M, N, 128, 128)))
        return plan<4, 2, 2, 2, 1, 16, 4, 1>(M, N, wide);
      // one tile a CU at most and K long: waves of 64 x 64, a third fewer LDS
      // reads a product, and K in two slices so that there are eight of them
      // (one slice / two, us: 1536x1792 K = 512 26.2 / 26.6, 704 31.6 / 31.7, 768
      // 33.9 / 33.7, 960 40.9 / 40.0; 2048^2 K = 704 35.7 / 36.1, 768 39.2 / 39.2, 960
      // 46.9 / 46.6; 2048^3 90.6 / 87.0)
      return K >= 768 && tiles(M, N, 128, 128) <= 256
                 ? plan<2, 2, 2, 2, 2, 16, 4, 1>(M, N, wide)
                 : plan<2, 4, 2, 1, 1, 16, 4, 1>(M, N, wide);
    case kMid:
      // one tile a CU at most: eight more waves pay once K is long
      // (4096x256x4096 71 -> 62 us, 1024^3 18.8 -> 18.3, K = 256 7.2 -> 7.6); with
      // plain loads' addresses a third set of registers would not fit beside a
      // tail-executor worker
      return K >= 1024 && tiles(M, N, 64, 64) <= 256 ? plan<2, 2, 1, 1, 4, 16, 4, 3, 2>(M, N, wide)
                                                     : plan<2, 2, 1, 1, 2, 16, 4, 4>(M, N, wide);
    default:
      // the same for 32 x 32 (256x256x2048 19.7 -> 16.3 us, 512^3 7.6 -> 7.1;
      // with 512 tiles 9.6 -> 12.6)
      return K >= 512 && tiles(M, N, 32, 32) <= 256 ? plan<1, 1, 1, 1, 8, 16, 4, 3>(M, N, wide)
                                                    : plan<1, 1, 1, 1, 4, 16, 8, 3>(M, N, wide);
  }
}

hipError_t gemm_f32_launch(const float* A, const float* B, float* C, int64_t M, int64_t N,
                           int64_t K, hipStream_t s, unsigned* sig, int variant) {
  const OpPlan p = gemm_f32_plan(M, N, K, true, variant);
  int m = (int)M, n = (int)N, k = (int)K;
  void* args[] = {&A, &B, &C, &m, &n, &k, &sig};
  return submit(p, args, s);
}

}  // namespace ug
