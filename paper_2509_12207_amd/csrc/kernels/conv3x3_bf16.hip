// BF16 3x3 convolution (stride 1, zero padding) on the matrix cores of gfx950:
// X [H, W, C] and W [C, 3, 3, C] in bfloat16, Y [C, H, W] in FP32.
//
// A workgroup computes BM output channels of a TH x TW tile of pixels.  Per
// group of CG input channels the tile's pixels and their border are put in
// LDS once (a patch) and read nine times, shifted by the tap; the weights
// come in stages of TS taps, in a ring of NST.  Both go from memory straight
// to LDS.  Each of the WM x WN waves forms TM x TN products of 32 channels
// by 32 pixels with v_mfma_f32_32x32x16_bf16 (lane l feeds row / column l % 32
// with the 16 bytes k = 8 (l / 32) .. +7).
//
// LDS rows (a pixel, or a weight row of one tap) are CG values; their 16-byte
// chunks are XOR-permuted, by the row for weights and by the column for
// pixels, so that a fragment's read of one chunk of 32 weight rows, or of 16
// pixels of two rows of the tile, whatever the tap, touches every LDS bank
// equally (permuted by the pixel's place in the patch, whose rows are 18
// apart, two lanes of sixteen met in a bank: 2 to 6 % slower).  Groups are 64
// channels, whole 128-byte lines, unless C is not a multiple of 64.
//
// What bounds it: read tap by tap, as the product of a matrix that holds
// every pixel nine times, the convolution was bound by the rate at which
// stages reach LDS; with patches a large one is bound by the matrix cores
// (C = 256, 256^2: 1.15 PFLOP/s), a mid one by LDS reads (a wave reads 16 bytes
// for every product row and column it has), a small one by the latency of its
// 27 stages a 64 channels.  us per launch, tap by tap -> now: C = 256, 256^2
// 88 -> 67.4, 128^2 38 -> 22.7, 64^2 17 -> 9.0, 32^2 8.5 -> 8.6; C = 128, 256^2
// 30 -> 21.6, 128^2 17.4 -> 8.1, 64^2 11.4 -> 5.8; C = 64, 336^2 25 -> 14.3, 128^2
// 8.6 -> 4.7; C = 96, 160^2 17.7 -> 8.9; C = 32, 336^2 17 -> 7.1, 64^2 5.6 -> 3.7.
// (A second patch buffer, filled during the group before: 1 to 15 % slower,
// for the workgroups a CU that it takes.)
#include "lds_load.hpp"
#include "mfma.hpp"
#include "ops.hpp"
#include "signal.hpp"
#include "submit.hpp"

namespace ug {
namespace {

template <int WM, int WN, int TM, int TN, int TH, int TW, int CG, int TS, int NST>
struct Patch {
  static constexpr int BM = WM * TM * 32, WAVES = WM * WN, NT = 64 * WAVES;
  static constexpr int ROWB = 2 * CG, CH = CG / 8;             // bytes, chunks of an LDS row
  static constexpr int PW = CG == 64 ? TW + 2 : TW + 4;        // the patch's pixels, two unused
  static constexpr int PP = (TH + 2) * PW;                     //   where a row has to be 4 n
  static constexpr int PB = (PP * ROWB + 1023) / 1024;         // its 1 KiB blocks, a wave's load each
  static constexpr int PPT = (PB + WAVES - 1) / WAVES;         // loads per wave
  static constexpr int STAGE = TS * BM * ROWB, WB = STAGE / 1024, WPT = (WB + WAVES - 1) / WAVES;
  static constexpr int LDS = PB * 1024 + NST * STAGE;
  static_assert(TH * TW == WN * TN * 32 && (32 % TW == 0 || TW % 32 == 0), "pixels of the waves");
  static_assert(STAGE % 1024 == 0 && 9 % TS == 0 && NST >= 2, "whole stages");
  static_assert((NST - 1) * WPT < 64, "the wait counts fit vmcnt");
};

// permutation of the chunks of weight row `row`, of a pixel in column `row` of
// the patch
template <int CG>
__device__ __forceinline__ int patch_swz(int row) {
  return CG == 64 ? (row >> 1) & 7 : (row >> 2) & 3;
}

template <int WM, int WN, int TM, int TN, int TH, int TW, int CG, int TS, int NST>
__global__ __launch_bounds__(64 * WM * WN, 2) void conv3x3_bf16_kernel(
    const unsigned char* __restrict__ Wt, const unsigned char* __restrict__ X,
    float* __restrict__ Y, int C, int H, int W, unsigned* sig) {
  using P = Patch<WM, WN, TM, TN, TH, TW, CG, TS, NST>;
  __shared__ __attribute__((aligned(1024))) unsigned char lds[P::LDS];
  unsigned char* ring = lds + P::PB * 1024;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave / WN, wn = wave % WN;
  // each XCD takes a contiguous band of pixel tiles, all channels of a tile
  // in a row
  const int tiles_x = (W + TW - 1) / TW, tiles_c = gridDim.y;
  const int total = gridDim.x * gridDim.y, wg = blockIdx.y * gridDim.x + blockIdx.x;
  const int xcd = wg % kXcds;
  const int id = xcd * (total / kXcds) + min(xcd, total % kXcds) + wg / kXcds;
  const int tile = id / tiles_c;
  const int m0 = (id - tile * tiles_c) * P::BM;
  const int ty = tile / tiles_x;
  const int y0 = ty * TH, x0 = (tile - ty * tiles_x) * TW;
  const int groups = C / CG, steps = 9 / TS * groups;

  // Load i of a wave fills 1 KiB block wave * WPT + i of a stage, lane l its
  // chunk l.  Blocks past the last repeat it, so that every wave has the same
  // number of loads in flight; channels past C repeat the last (not stored).
  const unsigned char* src[P::WPT];
  unsigned to[P::WPT];
#pragma unroll
  for (int i = 0; i < P::WPT; ++i) {
    const int b = min(wave * P::WPT + i, P::WB - 1);
    const int q = (b * 64 + lane) / P::CH, tap = q / P::BM, row = q % P::BM;
    src[i] = Wt + ((size_t)min(m0 + row, C - 1) * 9 + tap) * 2 * C +
             16 * (lane % P::CH ^ patch_swz<CG>(row));
    to[i] = (unsigned)(uintptr_t)ring + b * 1024;
  }
  // stage `step`; past the end the last one again, into a slot not read any more
  auto load_weights = [&](int step) {
    const int sc = min(step, steps - 1);
    const int g = (int)((unsigned)sc / (9u / TS)), tap = TS * (sc - 9 / TS * g);
    const size_t off = (size_t)tap * 2 * C + (size_t)g * P::ROWB;
#pragma unroll
    for (int i = 0; i < P::WPT; ++i)
      load16_lds(src[i] + off, __builtin_amdgcn_readfirstlane(to[i] + step % NST * P::STAGE));
  };
  auto load_patch = [&](int g) {
#pragma unroll
    for (int i = 0; i < P::PPT; ++i) {
      const int b = min(i * P::WAVES + wave, P::PB - 1);
      const int p = (b * 64 + lane) / P::CH, py = p / P::PW;
      const int px = p - py * P::PW, y = y0 + py - 1, x = x0 + px - 1;
      const bool in = p < P::PP && (unsigned)y < (unsigned)H && (unsigned)x < (unsigned)W;
      const unsigned char* from =
          in ? X + (((size_t)y * W + x) * C + (size_t)g * CG) * 2 +
                   16 * (lane % P::CH ^ patch_swz<CG>(px))
             : kZeroSlice;
      load16_lds(from, __builtin_amdgcn_readfirstlane((unsigned)(uintptr_t)lds + b * 1024));
    }
  };

  f32x16 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] = zero16();
  const int half = lane >> 5, col = lane & 31;
  int pix[TN];   // this lane's pixels, at tap (0, 0) in the patch
#pragma unroll
  for (int j = 0; j < TN; ++j) {
    const int n = (wn * TN + j) * 32 + col;
    pix[j] = n / TW * P::PW + n % TW;
  }

#pragma unroll
  for (int i = 0; i < NST - 1; ++i) load_weights(i);
  int s = 0;
  for (int g = 0; g < groups; ++g) {
    if (g > 0) {   // every wave has read the patch before
      __builtin_amdgcn_s_waitcnt(kWaitLdsOnly);
      asm volatile("s_barrier" ::: "memory");
    }
    load_patch(g);
    wait_loads<0>();
    asm volatile("s_barrier" ::: "memory");
#pragma unroll
    for (int tap = 0; tap < 9; ++tap) {
      if (tap % TS == 0) {
        // stage s has arrived in every wave, and every wave has read stage
        // s - 1, whose slot is filled again
        if (tap > 0) {
          wait_loads<(NST - 2) * P::WPT>();
          __builtin_amdgcn_s_waitcnt(kWaitLdsOnly);
          asm volatile("s_barrier" ::: "memory");
        }
        load_weights(s + NST - 1);
      }
      const unsigned char* wrow =
          ring + s % NST * P::STAGE + (tap % TS * P::BM + wm * TM * 32 + col) * P::ROWB;
#pragma unroll
      for (int k = 0; k < CG / 16; ++k) {
        int4 a[TM], b[TN];
#pragma unroll
        for (int i = 0; i < TM; ++i)   // (32 rows on, the same permutation)
          a[i] = *reinterpret_cast<const int4*>(wrow + i * 32 * P::ROWB +
                                                16 * ((2 * k + half) ^ patch_swz<CG>(col)));
#pragma unroll
        for (int j = 0; j < TN; ++j) {
          const int p = pix[j] + tap / 3 * P::PW + tap % 3;
          const int px = ((wn * TN + j) * 32 + col) % TW + tap % 3;
          b[j] = *reinterpret_cast<const int4*>(lds + p * P::ROWB +
                                                16 * ((2 * k + half) ^ patch_swz<CG>(px)));
        }
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
          for (int j = 0; j < TN; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(a[i]), as_bf16x8(b[j]),
                                                                acc[i][j], 0, 0, 0);
      }
      if (tap % TS == TS - 1) ++s;
    }
  }
  // no load may still be writing LDS when the workgroup ends
  wait_loads<0>();

  const size_t plane = (size_t)H * W;
#pragma unroll
  for (int j = 0; j < TN; ++j) {
    const int n = (wn * TN + j) * 32 + col;
    const int y = y0 + n / TW, x = x0 + n % TW;
    if (y >= H || x >= W) continue;
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int o = m0 + (wm * TM + i) * 32 + mfma32_row(r, lane);
        if (o < C) Y[(size_t)o * plane + (size_t)y * W + x] = acc[i][j][r];
      }
  }
  group_done(sig);
}

int64_t pixel_tiles(int th, int tw, int64_t H, int64_t W) {
  return ((H + th - 1) / th) * ((W + tw - 1) / tw);
}

template <int WM, int WN, int TM, int TN, int TH, int TW, int CG, int TS, int NST>
OpPlan plan(int64_t C, int64_t H, int64_t W) {
  using P = Patch<WM, WN, TM, TN, TH, TW, CG, TS, NST>;
  OpPlan p;
  p.func = reinterpret_cast<const void*>(
      &conv3x3_bf16_kernel<WM, WN, TM, TN, TH, TW, CG, TS, NST>);
  p.grid = dim3((unsigned)pixel_tiles(TH, TW, H, W), (unsigned)((C + P::BM - 1) / P::BM));
  p.block = dim3(P::NT);
  return p;
}

}  // namespace

// 64 channels of 16 x 16 pixels, two workgroups a CU, once there are enough of
// them and their padding costs less than what they save (a fifth) over 32
// channels of 8 x 16, three a CU: C = 256, 256^2, 1024 / 4096 workgroups, 70
// against 86 us; C = 128, 256^2, 512 / 2048, 23.5 against 26.4; C = 128, 200^2,
// 338 / 1300, 20.3 against 19.4; C = 192, 128^2, 192 / 768, 18.3 against 15.
// Weights by three taps (a tap row) where a CU holds the stages without
// losing a workgroup, else by one.
OpPlan conv3x3_bf16_plan(int64_t C, int64_t H, int64_t W) {
  const int64_t large = pixel_tiles(16, 16, H, W) * ((C + 63) / 64);
  const int64_t small = pixel_tiles(8, 16, H, W) * ((C + 31) / 32);
  if (large >= 384 && 16 * large <= 5 * small)
    return C % 64 == 0 ? plan<1, 4, 2, 2, 16, 16, 64, 1, 3>(C, H, W)
                       : plan<1, 4, 2, 2, 16, 16, 32, 3, 2>(C, H, W);
  return C % 64 == 0 ? plan<1, 4, 1, 1, 8, 16, 64, 3, 2>(C, H, W)
                     : plan<1, 4, 1, 1, 8, 16, 32, 3, 2>(C, H, W);
}

hipError_t conv3x3_bf16_launch(const uint16_t* X, const uint16_t* Wt, float* Y, int64_t C,
                               int64_t H, int64_t W, hipStream_t s, unsigned* sig) {
  const OpPlan p = conv3x3_bf16_plan(C, H, W);
  int c = (int)C, h = (int)H, w = (int)W;
  void* args[] = {&Wt, &X, &Y, &c, &h, &w, &sig};
  return submit(p, args, s);
}

}  // namespace ug
