// 3x3 convolution (cross-correlation, stride 1, zero pad 1, C_out = C_in),
// NCHW FP32, as an implicit GEMM on gfx950:
//   Y[o, p] = sum_{c, dy, dx} W[o, c, dy, dx] * X[c, py + dy - 1, px + dx - 1]
// i.e. M = output channels, N = pixels, K = 9 * input channels, on the BF16
// matrix cores with every value split into three bfloat16 pieces as it is
// staged (split.hpp: error against fp64 below half the FP32 instruction's,
// matrix cycles 2.67 times fewer).
//
// A workgroup owns BM = WM*TM*32 output channels x a TH x TW pixel patch
// (TH*TW = WN*TN*32 pixels) and runs over chunks of 16 input channels (one
// matrix instruction per tap and product): the chunk's weights and its input
// patch with a one-pixel halo are split into LDS, channels innermost, and
// each fragment is 16 bytes (eight channels) of 32 consecutive rows or
// pixels; the nine taps read the same patch at nine offsets, so the im2col
// operand is never formed and a pixel is split once for nine taps.  Two
// buffers: the next chunk is split, from registers loaded a chunk ahead,
// while this one multiplies.
//
// Kernels:
// * conv3x3_f32_kernel <WM, WN, TM, TN, KS, TH, TW>: all nine taps of a chunk
//   in LDS, the taps divided over KS groups of wavefronts (three: one tap row
//   each; nine: one tap) and summed through LDS in a fixed order.  One
//   workgroup a CU (two of the smallest).
// * conv3x3_f32_rows <WM, WN, TM, TN, TH, TW>: the weights of one tap row at
//   a time in LDS, so that two workgroups share a CU and one splits while the
//   other multiplies.
// * conv3x3_f32_few: few channels, with the FP32 instruction.
//
// What bounds it: at C = 256, 256^2 the matrix cores are busy about 65 % of
// the time (MFMA alone about 270 us of 380), the rest is splitting that the
// other workgroup does not cover.  The small tiles are bound by the latency
// of a chunk (loads, split, LDS, barrier: 0.9 to 1.6 us) and by the launch.
// us per launch, FP32 instruction before -> now:
//   C=256 256^2 670 -> 380, C=236 145^2 290 -> 139, C=128 128^2 52 -> 28.8,
//   C=64 256^2 48 -> 30, C=256 64^2 58 -> 28.7, C=64 128^2 17.4 -> 10.0,
//   C=128 64^2 20.5 -> 12.6, C=64 84^2 12.9 -> 8.4, C=32 128^2 9.0 -> 6.2,
//   C=256 32^2 23 -> 17.0, C=16 64^2 5.7 -> 5.4, C=16 336^2 15.1 -> 11.5,
//   C=20 264^2 14.6 -> 13.2.  One NaN in every tile: C=256 256^2 1070,
//   C=128 128^2 69, C=64 84^2 19.0.
#include "mfma.hpp"
#include "ops.hpp"
#include "signal.hpp"
#include "split.hpp"
#include "submit.hpp"
#include "tile_map.hpp"

namespace ug {
namespace {

constexpr int CC = 16;         // input channels per chunk: one matrix instruction a tap

typedef uint32_t u32x3 __attribute__((ext_vector_type(3)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// Geometry of exact_tile.
constexpr int EC = 4;   // input channels per step
template <int WM, int WN, int TM, int TN, int KS, int TH, int TW>
struct ExactCfg {
  static constexpr int NT = 64 * WM * WN * KS, BM = WM * TM * 32;
  static constexpr int PW = TW + 2, PX = (TH + 2) * PW;
  static constexpr int WR = BM + 1;                   // floats per channel and tap
  static constexpr int WU = (BM * 9 * EC + NT - 1) / NT, XU = (PX * EC + NT - 1) / NT;
  static constexpr int BYTES = 4 * EC * (9 * WR + PX);
};

template <int WM, int WN, int TM, int TN, int KS, int TH, int TW, int NB, int XB>
struct ConvCfg {
  static constexpr int WAVES = WM * WN, NT = 64 * WAVES * KS;
  static constexpr int BM = WM * TM * 32;
  static constexpr int PH = TH + 2, PW = TW + 2, PX = PH * PW;   // patch with halo
  static constexpr int PXP = (PX + 63) / 64 * 64;                // whole wavefronts
  static constexpr int TAPS = 9 / KS;                            // taps of a wave
  // LDS, bytes: weights [tap][piece][half][row] and patch [piece][half][pixel]
  // of 16 bytes each (eight channels); 32 bytes between the halves of the
  // weights keep the staging writes of a row, its channels and its tap rows
  // in different banks
  static constexpr int WH = BM * 16 + 32, WT = 6 * WH, XH = PX * 16;
  static constexpr int WS = 9 * WT, XS = 6 * XH, X0 = NB * WS, ALL = X0 + XB * XS;
  static constexpr int RED = (KS - 1) * WAVES * TM * TN * 4096;   // sums handed over at the end
  static constexpr int LDS = ALL > RED ? ALL : RED;
  static constexpr int WU = (BM * 12 + NT - 1) / NT;             // weight units per thread
  static constexpr int XU = (PXP * 4 + NT - 1) / NT;             // patch units per thread
  static_assert(WN * TN * 32 == TH * TW && TW == 16, "pixel tile");
  static_assert(LDS >= ExactCfg<WM, WN, TM, TN, KS, TH, TW>::BYTES, "unsplit values fit in LDS");
};

// Splits four channels into the three pieces at `at`, `piece` bytes apart.
__device__ __forceinline__ void put(float a, float b, float c, float d, unsigned char* at, int piece) {
  uint2 p[3];
  split2(a, b, &p[0].x, &p[1].x, &p[2].x);
  split2(c, d, &p[0].y, &p[1].y, &p[2].y);
#pragma unroll
  for (int j = 0; j < 3; ++j) *reinterpret_cast<uint2*>(at + j * piece) = p[j];
}

// Column of pixel p of a tile: a row of the tile starts two pixels on, so that
// the sixteen pixels of a row and those of the next, 18 apart in the patch,
// lie in LDS banks of their own for the lanes that read them together (C = 256,
// 32^2 17.3 -> 16.6 us, 64^2 29.4 -> 28.3; the large tiles the same).
__device__ __forceinline__ int column(int p) { return (p - 2 * (p / 16)) & 15; }

// Image and first pixel of a workgroup's tile: each XCD takes a contiguous
// band of them.
template <int TH, int TW>
__device__ __forceinline__ void pixels_of(int H, int W, int* n, int* y0, int* x0) {
  const int tiles_x = (W + TW - 1) / TW, tiles_y = (H + TH - 1) / TH;
  const int xcd = blockIdx.x % kXcds;
  const int id = xcd * (gridDim.x / kXcds) + min(xcd, (int)(gridDim.x % kXcds)) + blockIdx.x / kXcds;
  const int pt = id % (tiles_x * tiles_y);
  *n = id / (tiles_x * tiles_y);
  *y0 = (pt / tiles_x) * TH;
  *x0 = (pt % tiles_x) * TW;
}

// A workgroup's tile with the FP32 instruction, on the values as they are
// (inputs without a split, and few channels): four input channels a step, in
// one buffer of FP32 values (weights [channel][tap][row], patch
// [channel][pixel]), the next step's in registers; a wave's taps are those of
// its K slice.  The thread's index is hidden from the compiler, which would
// otherwise keep what it has in common with the kernel's in registers
// throughout.
template <int WM, int WN, int TM, int TN, int KS, int TH, int TW>
__device__ __forceinline__ void exact_tile(f32x16 (&acc)[TM][TN], float* raw,
                                           const float* __restrict__ X,
                                           const float* __restrict__ Wt, int C, int H, int W, int o0,
                                           int y0, int x0) {
  using E = ExactCfg<WM, WN, TM, TN, KS, TH, TW>;
  constexpr int NT = E::NT, BM = E::BM, PW = E::PW, TAPS = 9 / KS;
  int tid = threadIdx.x;
  asm("" : "+v"(tid));
  const int half = tid >> 5 & 1, col = tid & 31, wave = tid >> 6;
  const int t0 = wave / (WM * WN) * TAPS, wm = wave % (WM * WN) / WN, wn = wave % WN;
  const uint32_t plane = (uint32_t)H * W;
  // offsets from a step's first row of weights and first channel plane (four
  // planes of fewer than 2^26 floats); channels before which a unit is read
  uint32_t wo[E::WU], xo[E::XU];
  int wc[E::WU], xc[E::XU];
#pragma unroll
  for (int i = 0; i < E::WU; ++i) {
    const int u = tid + NT * i, o = u / (9 * EC), k = u % (9 * EC);
    wo[i] = (uint32_t)o * (uint32_t)(9 * C) + k;
    wc[i] = u < BM * 9 * EC && o0 + o < C ? C - k / 9 : 0;
  }
#pragma unroll
  for (int i = 0; i < E::XU; ++i) {
    const int u = tid + NT * i, c = u / E::PX, r = u % E::PX;
    const int yy = y0 - 1 + r / PW, xx = x0 - 1 + r % PW;
    xo[i] = c * plane + (uint32_t)yy * W + xx;
    xc[i] = c < EC && yy >= 0 && yy < H && xx >= 0 && xx < W ? C - c : 0;
  }
  float rw[E::WU], rx[E::XU];
  auto load = [&](int c0) {
    const float* w = Wt + ((size_t)o0 * C + c0) * 9;
    const float* x = X + (size_t)c0 * plane;
#pragma unroll
    for (int i = 0; i < E::WU; ++i) rw[i] = c0 < wc[i] ? w[wo[i]] : 0.f;
#pragma unroll
    for (int i = 0; i < E::XU; ++i) rx[i] = c0 < xc[i] ? x[xo[i]] : 0.f;
  };
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] = zero16();
  // the lower half of a wave takes the even channels of a step, the upper the odd ones
  const float* w = raw + (half * 9 + t0) * E::WR + wm * TM * 32 + col;
  const float* x[TN];
#pragma unroll
  for (int j = 0; j < TN; ++j) {
    const int p = (wn * TN + j) * 32 + col;
    x[j] = raw + EC * 9 * E::WR + half * E::PX + p / TW * PW + column(p);
  }
  load(0);
#pragma clang loop unroll(disable)
  for (int c0 = 0; c0 < C; c0 += EC) {
#pragma unroll
    for (int i = 0; i < E::WU; ++i) {
      const int u = tid + NT * i;
      if (u < BM * 9 * EC) raw[u % (9 * EC) * E::WR + u / (9 * EC)] = rw[i];
    }
#pragma unroll
    for (int i = 0; i < E::XU; ++i) {
      const int u = tid + NT * i;
      if (u < E::PX * EC) raw[EC * 9 * E::WR + u] = rx[i];
    }
    __syncthreads();
    if (c0 + EC < C) load(c0 + EC);
#pragma unroll
    for (int t = 0; t < TAPS; ++t) {
      const int at = (t0 + t) / 3 * PW + (t0 + t) % 3;
#pragma unroll
      for (int c = 0; c < EC; c += 2)
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
          for (int j = 0; j < TN; ++j)
            acc[i][j] = mfma_32x32x2(w[(9 * c + t) * E::WR + i * 32], x[j][c * E::PX + at], acc[i][j]);
    }
    __syncthreads();   // read, and at the end free for the sums of the K slices
  }
}

template <int TM, int TN, int TW>
__device__ __forceinline__ void store_tile(const f32x16 (&acc)[TM][TN], float* __restrict__ Y,
                                           int C, int H, int W, int o0, int p0, int y0, int x0) {
  const int lane = threadIdx.x & 63, col = lane & 31;
  const size_t plane = (size_t)H * W;
#pragma unroll
  for (int j = 0; j < TN; ++j) {
    const int p = p0 + j * 32 + col;
    const int yy = y0 + p / TW, xx = x0 + column(p);
    if (yy >= H || xx >= W) continue;
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int q = 0; q < 16; ++q) {
        const int o = o0 + 32 * i + mfma32_row(q, lane);
        if (o < C) Y[(size_t)o * plane + (size_t)yy * W + xx] = acc[i][j][q];
      }
  }
}

// NB: two buffers of weights, or one where all channels are one chunk
// (C <= 16).  XB: as many of the patch, or one, which takes a barrier more a
// chunk (before the last tap, once every wave has read the patch for it) and
// 17 KiB less: 64 x 8x16 then fits beside a tail-executor worker (128 KiB of LDS
// instead of 145 of the 136 left).  The weights staged by then are complete,
// and the next chunk's first ones are read before it starts, under the last
// tap's products (C = 128, 128^2 26.4 us with two, 27.9 with one, 27.1 so).
template <int WM, int WN, int TM, int TN, int KS, int TH, int TW, int NB, int XB>
__global__ __launch_bounds__(64 * WM * WN * KS, 2) void conv3x3_f32_kernel(
    const float* __restrict__ X, const float* __restrict__ Wt, float* __restrict__ Y, int C, int H,
    int W, unsigned* sig) {
  using Cf = ConvCfg<WM, WN, TM, TN, KS, TH, TW, NB, XB>;
  constexpr int BM = Cf::BM, PW = Cf::PW, NT = Cf::NT, TAPS = Cf::TAPS;
  __shared__ __attribute__((aligned(1024))) unsigned char lds[Cf::LDS];
  __shared__ int redo;

  const int tid = threadIdx.x, lane = tid & 63;
  const int wid = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int ks = wid / Cf::WAVES, wave = wid % Cf::WAVES;
  const int wm = wave / WN, wn = wave % WN;
  int n, y0, x0;
  pixels_of<TH, TW>(H, W, &n, &y0, &x0);
  const int o0 = blockIdx.y * BM;
  const size_t plane = (size_t)H * W;
  const float* Xn = X + (size_t)n * C * plane;
  if (tid == 0) redo = 0;

  // Staging units.  Weights: three taps of a row (one ky) of four channels of
  // an output channel, 4 x 12 bytes; a unit's channels are four apart, so that
  // the twelve lanes of a row read 144 bytes in a piece (channels next to each
  // other, with lanes 144 bytes apart, touched three times the lines: C = 256,
  // 32^2 20.4 us against 17.5).  Patch: the same four channels of a pixel,
  // consecutive threads on consecutive pixels.  In LDS a unit's channels are
  // neighbours: channel 4 j + q of the chunk is at 4 q + j in both operands.
  // Output channels past C repeat the last one (never stored).  Buffer loads:
  // what lies past the tensor, a channel past C or a pixel outside the image
  // (offset 2^31) reads as zero.  The resources move along by scalar
  // additions; waves without a unit load nothing.
  uint32_t wo[Cf::WU], xo[Cf::XU];
  int wl[Cf::WU], xl[Cf::XU], xq[Cf::XU];   // LDS places; channel quad of the patch unit
#pragma unroll
  for (int i = 0; i < Cf::WU; ++i) {
    const int u = tid + NT * i, ky = u % 3, q = u / 3 % 4, row = u / 12;
    wo[i] = (((uint32_t)min(row, C - 1 - o0) * C + q) * 9 + 3 * ky) * 4;
    wl[i] = row < BM ? 3 * ky * Cf::WT + (q / 2) * Cf::WH + row * 16 + (q % 2) * 8 : -1;
  }
#pragma unroll
  for (int i = 0; i < Cf::XU; ++i) {
    const int u = tid + NT * i, r = u % Cf::PXP;
    const int q = __builtin_amdgcn_readfirstlane(u / Cf::PXP);
    const int yy = y0 - 1 + r / PW, xx = x0 - 1 + r % PW;
    xo[i] = yy >= 0 && yy < H && xx >= 0 && xx < W ? (uint32_t)((size_t)yy * W + xx) * 4 : 1u << 31;
    xl[i] = r < Cf::PX && q < 4 ? Cf::X0 + (q / 2) * Cf::XH + r * 16 + (q % 2) * 8 : -1;
    xq[i] = min(q, 3);
  }

  float rw[Cf::WU][4][3], rx[Cf::XU][4];   // the chunk staged next
  // the next chunk: its weights and the bytes from them to the end, its first
  // channel plane, the channels left
  const float* wp = Wt + (size_t)o0 * C * 9;
  int64_t left = ((int64_t)C * C - (int64_t)o0 * C) * 36;
  const float* xp = Xn;
  int cl = C;
  auto load = [&]() {
    const auto ws = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(wp), 0,
                                                      left >> 32 ? -1 : (int)left, 0x00027000);
#pragma unroll
    for (int i = 0; i < Cf::WU; ++i) {
      if (BM * 12 % NT != 0 && wid * 64 + NT * i >= BM * 12) continue;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const u32x3 v = __builtin_bit_cast(
            u32x3, __builtin_amdgcn_raw_buffer_load_b96(ws, wo[i] + 144 * j, 0, 0));
#pragma unroll
        for (int t = 0; t < 3; ++t) rw[i][j][t] = __uint_as_float(v[t]);
      }
    }
#pragma unroll
    for (int i = 0; i < Cf::XU; ++i) {
      if (Cf::PXP * 4 % NT != 0 && wid * 64 + NT * i >= Cf::PXP * 4) continue;
      const float* xc = xp + (size_t)xq[i] * plane;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const auto xs = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<float*>(xc + 4 * j * plane), 0,
            xq[i] + 4 * j < cl ? (int)((uint32_t)plane * 4) : 0, 0x00027000);
        rx[i][j] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(xs, xo[i], 0, 0));
      }
    }
    wp += CC * 9;
    left -= CC * 36;
    xp += CC * plane;
    cl -= CC;
  };
  int wst = 0, xst = 0;   // offsets of the buffers staged into
  auto store_w = [&]() {
#pragma unroll
    for (int i = 0; i < Cf::WU; ++i)
      if (BM * 12 % NT == 0 || wl[i] >= 0)
#pragma unroll
        for (int t = 0; t < 3; ++t)
          put(rw[i][0][t], rw[i][1][t], rw[i][2][t], rw[i][3][t], lds + wst + wl[i] + t * Cf::WT,
              2 * Cf::WH);
  };
  auto store_x = [&]() {
#pragma unroll
    for (int i = 0; i < Cf::XU; ++i)
      if (xl[i] >= 0) put(rx[i][0], rx[i][1], rx[i][2], rx[i][3], lds + xst + xl[i], 2 * Cf::XH);
  };

  // fragments of tap t of this wave: rows of output channels and of pixels
  const int half = lane >> 5, col = lane & 31;
  const int ky0 = KS == 3 ? ks : KS == 9 ? ks / 3 : 0, kx0 = KS == 9 ? ks % 3 : 0;
  int fa = (3 * ky0 + kx0) * Cf::WT + half * Cf::WH + (wm * TM * 32 + col) * 16;
  int fb[TN];
#pragma unroll
  for (int j = 0; j < TN; ++j) {
    const int p = (wn * TN + j) * 32 + col;
    fb[j] = Cf::X0 + half * Cf::XH + ((p / TW + ky0) * PW + column(p) + kx0) * 16;
  }
  uint4 a[3][TM], b[3][TN];
  auto frag_w = [&](int t, int p, int buf) {
#pragma unroll
    for (int i = 0; i < TM; ++i)
      a[p][i] = *reinterpret_cast<const uint4*>(lds + fa + buf + t * Cf::WT + p * 2 * Cf::WH +
                                                i * 512);
  };
  auto frag_x = [&](int t, int p) {
#pragma unroll
    for (int j = 0; j < TN; ++j)
      b[p][j] = *reinterpret_cast<const uint4*>(lds + fb[j] + ((t / 3) * PW + t % 3) * 16 +
                                                p * 2 * Cf::XH);
  };
  f32x16 ah[TM][TN], as[TM][TN];   // sums of hh, of the other five products
  auto mul = [&](int p, int q, f32x16 (&d)[TM][TN]) {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) d[i][j] = mfma_bf16(a[p][i], b[q][j], d[i][j]);
  };

  const int chunks = NB == 1 ? 1 : (C + CC - 1) / CC;
  load();
  store_w();
  store_x();
  if (chunks > 1) load();
  lds_barrier();
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) ah[i][j] = as[i][j] = zero16();
  constexpr bool kLate = NB == 2 && XB == 1;   // the patch staged behind a barrier
  int wflip = Cf::WS, xflip = Cf::XS;
  // fragments of piece p for the tap after t, the next chunk's first included
  auto next = [&](int t, int p) {
    if (t + 1 < TAPS) {
      frag_w(t + 1, p, 0);
      frag_x(t + 1, p);
    } else if (kLate) {
      frag_w(0, p, wflip);
    }
  };
  if (kLate) {
#pragma unroll
    for (int p = 0; p < 3; ++p) frag_w(0, p, 0);
  }
#pragma clang loop unroll(disable)
  for (int ch = 0; ch < chunks; ++ch) {
    wst += wflip;
    if (XB == 2) xst += xflip;
    const bool more = ch + 1 < chunks;
    auto stage_x = [&]() {
      store_x();
      if (ch + 2 < chunks) load();
    };
    constexpr int kOrder[3] = {1, 0, 2};
#pragma unroll
    for (int p : kOrder) {
      if (!kLate) frag_w(0, p, 0);
      frag_x(0, p);
    }
#pragma unroll
    for (int t = 0; t < TAPS; ++t) {
      mul(1, 1, as);
      if (kLate && t == TAPS - 1 && more) {
        lds_barrier();
        stage_x();
      }
      mul(1, 0, as);
      mul(0, 1, as);
      next(t, 1);
      if (t == 0 && more) store_w();
      if (!kLate && t == TAPS - 1 && more) stage_x();
      mul(2, 0, as);
      mul(0, 2, as);
      next(t, 2);
      mul(0, 0, ah);
      next(t, 0);
    }
    lds_barrier();
    fa += wflip;
    wflip = -wflip;
    if (XB == 2) {
#pragma unroll
      for (int j = 0; j < TN; ++j) fb[j] += xflip;
      xflip = -xflip;
    }
  }

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
    exact_tile<WM, WN, TM, TN, KS, TH, TW>(ah, reinterpret_cast<float*>(lds), Xn, Wt, C, H, W, o0, y0,
                                           x0);

  if (KS > 1) {
    constexpr int PER = TM * TN * 16 * 64;   // floats per wave
    float* red0 = reinterpret_cast<float*>(lds);
    if (ks > 0) {
      float* red = red0 + ((ks - 1) * Cf::WAVES + wave) * PER;
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
          for (int q = 0; q < 16; ++q) red[((i * TN + j) * 16 + q) * 64 + lane] = ah[i][j][q];
    }
    __syncthreads();
    if (ks > 0) {   // handed over: meet slice 0 at the counter's barrier, then leave
      group_done(sig);
      return;
    }
#pragma unroll
    for (int s = 1; s < KS; ++s) {
      const float* red = red0 + ((s - 1) * Cf::WAVES + wave) * PER;
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
          for (int q = 0; q < 16; ++q) ah[i][j][q] += red[((i * TN + j) * 16 + q) * 64 + lane];
    }
  }

  store_tile<TM, TN, TW>(ah, Y + (size_t)n * C * plane, C, H, W, o0 + wm * TM * 32, wn * TN * 32, y0,
                         x0);
  group_done(sig);
}

// The large tiles: the weights of one tap row (ky) at a time in LDS, so that
// two workgroups share a CU and one splits while the other multiplies.
template <int WM, int WN, int TM, int TN, int TH, int TW>
struct RowsCfg {
  static constexpr int NT = 64 * WM * WN, BM = WM * TM * 32;
  static constexpr int PH = TH + 2, PW = TW + 2, PX = PH * PW;
  static constexpr int PXP = (PX + 31) / 32 * 32;
  // bytes between the halves of the weights: staging writes in different banks,
  // or, for 32 x 8x16, three workgroups a CU (C = 20, 264^2 16.6 -> 13.2 us)
  static constexpr int WP = BM == 32 && TH == 8 ? 16 : 128;
  static constexpr int WH = BM * 16 + WP, WT = 6 * WH, XH = PX * 16;
  static constexpr int WS = 3 * WT, XS = 6 * XH;          // bytes per buffer
  static constexpr int LDS = 2 * (WS + XS);
  static constexpr int XU = (PXP * 4 + NT - 1) / NT;
  static_assert(WN * TN * 32 == TH * TW && TW == 16, "pixel tile");
  static_assert(BM * 4 <= NT, "at most one weight unit a thread");
  static_assert(LDS >= ExactCfg<WM, WN, TM, TN, 1, TH, TW>::BYTES, "unsplit values fit in LDS");
};

template <int WM, int WN, int TM, int TN, int TH, int TW>
__global__ __launch_bounds__(64 * WM * WN, 2) void conv3x3_f32_rows(
    const float* __restrict__ X, const float* __restrict__ Wt, float* __restrict__ Y, int C, int H,
    int W, unsigned* sig) {
  using Cf = RowsCfg<WM, WN, TM, TN, TH, TW>;
  constexpr int BM = Cf::BM, PW = Cf::PW, NT = Cf::NT;
  __shared__ __attribute__((aligned(1024))) unsigned char lds[Cf::LDS];
  __shared__ int redo;

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / WN, wn = wave % WN;
  int n, y0, x0;
  pixels_of<TH, TW>(H, W, &n, &y0, &x0);
  const int o0 = blockIdx.y * BM;
  const size_t plane = (size_t)H * W;
  const float* Xn = X + (size_t)n * C * plane;
  if (tid == 0) redo = 0;

  const bool has_w = BM * 4 == NT || wave < BM * 4 / 64;
  const int row = tid / 4, q = tid % 4;
  const uint32_t wo = ((uint32_t)min(row, C - 1 - o0) * C + 4 * q) * 36;
  int wl = (q / 2) * Cf::WH + row * 16 + (q % 2) * 8;
  uint32_t xo[Cf::XU];
  int xl[Cf::XU], xc[Cf::XU];
#pragma unroll
  for (int i = 0; i < Cf::XU; ++i) {
    const int u = tid + NT * i, sub = u % 2, e = u / 2;
    const int r = e % Cf::PXP, h = __builtin_amdgcn_readfirstlane(e / Cf::PXP);
    const int yy = y0 - 1 + r / PW, xx = x0 - 1 + r % PW;
    xo[i] = yy >= 0 && yy < H && xx >= 0 && xx < W
                ? ((uint32_t)(4 * sub) * (uint32_t)plane + (uint32_t)((size_t)yy * W + xx)) * 4
                : 1u << 31;
    xl[i] = r < Cf::PX && h < 2 ? 2 * Cf::WS + h * Cf::XH + r * 16 + sub * 8 : -1;
    xc[i] = 8 * min(h, 1);
  }
  float rw[36], rx[Cf::XU][4];
  // the next chunk: its weights and the bytes from them to the end; its first
  // channel plane, the channels left
  const float* wp = Wt + (size_t)o0 * C * 9;
  int64_t left = ((int64_t)C * C - (int64_t)o0 * C) * 36;
  const float* xp = Xn;
  int cl = C;
  auto load_w = [&]() {
    const auto ws = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(wp), 0,
                                                      left >> 32 ? -1 : (int)left, 0x00027000);
#pragma unroll
    for (int j = 0; j < 9; ++j) {
      const u32x4 v = __builtin_bit_cast(
          u32x4, __builtin_amdgcn_raw_buffer_load_b128(ws, wo + 16 * j, 0, 0));
#pragma unroll
      for (int t = 0; t < 4; ++t) rw[4 * j + t] = __uint_as_float(v[t]);
    }
    wp += CC * 9;
    left -= CC * 36;
  };
  auto load_x = [&]() {
#pragma unroll
    for (int i = 0; i < Cf::XU; ++i) {
      // (a scalar for the compiler: a resource in vector registers is looped over)
      const int ch = __builtin_amdgcn_readfirstlane(max(0, min(cl - xc[i], 8)));
      const auto xs = __builtin_amdgcn_make_buffer_rsrc(
          const_cast<float*>(xp + (size_t)xc[i] * plane), 0,
          (int)((uint32_t)ch * (uint32_t)plane * 4), 0x00027000);
#pragma unroll
      for (int j = 0; j < 4; ++j)
        rx[i][j] = __uint_as_float(
            __builtin_amdgcn_raw_buffer_load_b32(xs, xo[i] + j * (uint32_t)plane * 4, 0, 0));
    }
    xp += CC * plane;
    cl -= CC;
  };
  int wst = 0, xst = 0;   // offsets of the buffers staged into
  auto store_w = [&](int t) {
    if (has_w) put(rw[t], rw[9 + t], rw[18 + t], rw[27 + t], lds + wst + wl + t % 3 * Cf::WT, 2 * Cf::WH);
  };
  auto store_x = [&]() {
#pragma unroll
    for (int i = 0; i < Cf::XU; ++i)
      if (xl[i] >= 0) put(rx[i][0], rx[i][1], rx[i][2], rx[i][3], lds + xst + xl[i], 2 * Cf::XH);
  };

  const int half = lane >> 5, col = lane & 31;
  int fa = half * Cf::WH + (wm * TM * 32 + col) * 16;
  int fb[TN];
#pragma unroll
  for (int j = 0; j < TN; ++j) {
    const int p = (wn * TN + j) * 32 + col;
    fb[j] = 2 * Cf::WS + half * Cf::XH + ((p / TW) * PW + column(p)) * 16;
  }
  uint4 a[3][TM], b[3][TN];
  auto frag = [&](int ky, int kx, int p) {
#pragma unroll
    for (int i = 0; i < TM; ++i)
      a[p][i] = *reinterpret_cast<const uint4*>(lds + fa + kx * Cf::WT + p * 2 * Cf::WH + i * 512);
#pragma unroll
    for (int j = 0; j < TN; ++j)
      b[p][j] = *reinterpret_cast<const uint4*>(lds + fb[j] + (ky * PW + kx) * 16 + p * 2 * Cf::XH);
  };
  f32x16 ah[TM][TN], as[TM][TN];   // sums of hh, of the other five products
  auto mul = [&](int p, int q, f32x16 (&d)[TM][TN]) {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) d[i][j] = mfma_bf16(a[p][i], b[q][j], d[i][j]);
  };

  const int chunks = (C + CC - 1) / CC;
  load_w();
  load_x();
#pragma unroll
  for (int t = 0; t < 3; ++t) store_w(t);
  store_x();
  if (chunks > 1) load_x();
  lds_barrier();
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) ah[i][j] = as[i][j] = zero16();
  int wflip = Cf::WS, xflip = Cf::XS;
#pragma clang loop unroll(disable)
  for (int ch = 0; ch < chunks; ++ch) {
    const bool more = ch + 1 < chunks;
#pragma unroll
    for (int ky = 0; ky < 3; ++ky) {
      wst += wflip;
      if (ky == 2) xst += xflip;
      frag(ky, 0, 1);
      frag(ky, 0, 0);
      frag(ky, 0, 2);
#pragma unroll
      for (int kx = 0; kx < 3; ++kx) {
        mul(1, 1, as);
        mul(1, 0, as);
        mul(0, 1, as);
        if (kx < 2) frag(ky, kx + 1, 1);
        if (ky < 2 || more) store_w((3 * ky + 3) % 9 + kx);   // the next tap row
        if (ky == 2 && kx == 1 && more) {
          store_x();
          if (ch + 2 < chunks) load_x();
        }
        if (ky == 1 && kx == 2 && more) load_w();
        mul(2, 0, as);
        mul(0, 2, as);
        if (kx < 2) frag(ky, kx + 1, 2);
        mul(0, 0, ah);
        if (kx < 2) frag(ky, kx + 1, 0);
      }
      lds_barrier();
      fa += wflip;
      wflip = -wflip;
    }
#pragma unroll
    for (int j = 0; j < TN; ++j) fb[j] += xflip;
    xflip = -xflip;
  }

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
  __syncthreads();
  if (redo)
    exact_tile<WM, WN, TM, TN, 1, TH, TW>(ah, reinterpret_cast<float*>(lds), Xn, Wt, C, H, W, o0, y0, x0);
  store_tile<TM, TN, TW>(ah, Y + (size_t)n * C * plane, C, H, W, o0 + wm * TM * 32, wn * TN * 32, y0,
                         x0);
  group_done(sig);
}

// Few channels: exact_tile alone.  A chunk of the split is 16 channels, staged
// and multiplied whole however few there are (336^2, C = 4: 10.1 us split, 7.2 so;
// 8: 10.3 and 9.8; 12: 10.6 and, the FP32 instruction's kernel before, 12.1.  64^2,
// C = 3 and 8: 5.3 split, 3.7 and 4.6).
constexpr int kFew = 8;
template <int WM, int WN, int TM, int TN, int TH, int TW>
__global__ __launch_bounds__(64 * WM * WN) void conv3x3_f32_few(
    const float* __restrict__ X, const float* __restrict__ Wt, float* __restrict__ Y, int C, int H,
    int W, unsigned* sig) {
  using E = ExactCfg<WM, WN, TM, TN, 1, TH, TW>;
  static_assert(WN * TN * 32 == TH * TW && TW == 16, "pixel tile");
  __shared__ float lds[E::BYTES / 4];
  int n, y0, x0;
  pixels_of<TH, TW>(H, W, &n, &y0, &x0);
  const int o0 = blockIdx.y * E::BM, wave = threadIdx.x >> 6;
  const size_t image = (size_t)n * C * H * W;
  f32x16 acc[TM][TN];
  exact_tile<WM, WN, TM, TN, 1, TH, TW>(acc, lds, X + image, Wt, C, H, W, o0, y0, x0);
  store_tile<TM, TN, TW>(acc, Y + image, C, H, W, o0 + wave / WN * TM * 32, wave % WN * TN * 32, y0, x0);
  group_done(sig);
}

// Tile shapes, largest first: {BM, TH, TW}.
struct Shape {
  int bm, th, tw;
};
constexpr Shape kShapes[] = {
    {64, 8, 16},    // rows <1,4,2,1> or <1,4,2,1,3>
    {32, 16, 16},   // rows <1,8,1,1>
    {32, 8, 16},    // <1,4,1,1,3> or rows <1,4,1,1>
    {32, 4, 16},    // <1,2,1,1,3>
    {32, 2, 16},    // <1,1,1,1,9>
};

int64_t wgs(const Shape& s, int64_t N, int64_t C, int64_t H, int64_t W) {
  return ((H + s.th - 1) / s.th) * ((W + s.tw - 1) / s.tw) * N * ((C + s.bm - 1) / s.bm);
}

// The smallest tile that one round of the 256 CUs holds: a chunk takes a
// workgroup 0.9 us (32 x 2x16) to 2.3 us (64 x 8x16), so that a second round
// costs more than a larger tile (C=64 128^2: 256 workgroups of 32 x 8x16 take
// 10.2 us, 512 of 32 x 4x16 14.9, 128 of 64 x 8x16 14.6; C=128 64^2: 13.0 at
// 32 x 4x16, 14.9 and 19.3 either side).  One chunk (C <= 16) takes
// 32 x 8x16 on four waves, past a round of them with one buffer, so that more
// share a CU (336^2: 11.5 us against 19.2 with two and 12.2 on twelve waves).
// Up to a round of them the second buffer is there but not used: with one, or
// as 32 x 4x16 on six waves with one (64^2 4.5 us against 5.4, the FP32
// instruction's kernel 5.7), the first three kernels of configuration 0's task,
// nearly all launch, profile below the 20 us at which a test of its launch
// synchronisation has batches close.
int pick(int64_t N, int64_t C, int64_t H, int64_t W) {
  if (C <= CC) return 2;
  for (int i = 4; i > 0; --i)
    if (!(i == 1 && C > 32) && wgs(kShapes[i], N, C, H, W) <= 256) return i;
  return C <= 32 ? 2 : 0;
}

// Nine taps at once where one round of the CUs holds the workgroups, by tap rows
// past that, two and three to a CU.  64 x 8x16: C=128 128^2, 256 workgroups: 27.1 against
// 30.7 us; C=256 80^2, 200: 43.9 and 59.2; C=64 200^2, 325: 29.3 and 24.4; C=128
// 192^2, 576: 75.2 and 73.7; C=236 145^2, 760: 134 and 132; C=256 256^2, 2048: 391
// and 372.  32 x 8x16 by tap rows, three to a CU, against a second round of
// 32 x 16x16: C=20 264^2, 561 workgroups: 13.2 and 18.9 us; C=32 336^2, 882: 19.7 and
// 21.1.
bool by_rows(const Shape& t, int64_t N, int64_t C, int64_t H, int64_t W) {
  return wgs(t, N, C, H, W) > 256;
}

// The variant asked for, else the tuning table's, else the rule above.
int choose(int64_t N, int64_t C, int64_t H, int64_t W, int variant) {
  if (variant < 0) {
    const int64_t key[4] = {N, C, H, W};
    variant = tune_get(UG_OP_CONV3X3_F32, key);
  }
  return variant >= 0 && variant < 5 ? variant : pick(N, C, H, W);
}

template <int WM, int WN, int TM, int TN, int KS, int TH, int TW, int NB = 2, int XB = NB>
OpPlan plan(int64_t N, int64_t C, int64_t H, int64_t W) {
  constexpr int BM = WM * TM * 32;
  OpPlan p;
  p.func =
      reinterpret_cast<const void*>(&conv3x3_f32_kernel<WM, WN, TM, TN, KS, TH, TW, NB, XB>);
  p.grid = dim3((unsigned)(((H + TH - 1) / TH) * ((W + TW - 1) / TW) * N),
                (unsigned)((C + BM - 1) / BM));
  p.block = dim3(64 * WM * WN * KS);
  return p;
}

OpPlan plan_few(int64_t N, int64_t C, int64_t H, int64_t W) {
  OpPlan p;
  p.func = reinterpret_cast<const void*>(&conv3x3_f32_few<1, 4, 1, 1, 8, 16>);
  p.grid = dim3((unsigned)wgs(kShapes[2], N, C, H, W));   // (32 output channels: all)
  p.block = dim3(256);
  return p;
}

template <int WM, int WN, int TM, int TN, int TH, int TW>
OpPlan plan_rows(int64_t N, int64_t C, int64_t H, int64_t W) {
  constexpr int BM = WM * TM * 32;
  OpPlan p;
  p.func = reinterpret_cast<const void*>(&conv3x3_f32_rows<WM, WN, TM, TN, TH, TW>);
  p.grid = dim3((unsigned)(((H + TH - 1) / TH) * ((W + TW - 1) / TW) * N),
                (unsigned)((C + BM - 1) / BM));
  p.block = dim3(64 * WM * WN);
  return p;
}

}  // namespace

OpPlan conv3x3_f32_plan(int64_t N, int64_t C, int64_t H, int64_t W, int variant) {
  switch (choose(N, C, H, W, variant)) {
    case 0:
      return by_rows(kShapes[0], N, C, H, W) ? plan_rows<1, 4, 2, 1, 8, 16>(N, C, H, W)
                                 : plan<1, 4, 2, 1, 3, 8, 16, 2, 1>(N, C, H, W);
    case 1: return plan_rows<1, 8, 1, 1, 16, 16>(N, C, H, W);
    case 2:
      if (C <= kFew) return plan_few(N, C, H, W);
      if (C <= CC)
        return wgs(kShapes[2], N, C, H, W) > 256 ? plan<1, 4, 1, 1, 1, 8, 16, 1>(N, C, H, W)
                                                 : plan<1, 4, 1, 1, 1, 8, 16, 2>(N, C, H, W);
      return by_rows(kShapes[2], N, C, H, W) ? plan_rows<1, 4, 1, 1, 8, 16>(N, C, H, W)
                                             : plan<1, 4, 1, 1, 3, 8, 16>(N, C, H, W);
    case 3: return plan<1, 2, 1, 1, 3, 4, 16>(N, C, H, W);
    default: return plan<1, 1, 1, 1, 9, 2, 16>(N, C, H, W);
  }
}

hipError_t conv3x3_f32_launch(const float* X, const float* Wt, float* Y, int64_t N, int64_t C,
                              int64_t H, int64_t W, hipStream_t s, unsigned* sig, int variant) {
  const OpPlan p = conv3x3_f32_plan(N, C, H, W, variant);
  int c = (int)C, h = (int)H, w = (int)W;
  void* args[] = {&X, &Wt, &Y, &c, &h, &w, &sig};
  return submit(p, args, s);
}

}  // namespace ug
