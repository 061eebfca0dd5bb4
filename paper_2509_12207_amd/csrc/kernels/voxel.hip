// Bird's-eye-view pillar binning of a point cloud (FP32 points -> int cells).
//
// Per cell: count, maximum z and smallest point index; per point: its cell.
// All three reductions are order independent, so all paths below give
// bit-identical outputs.
//
// Three paths, chosen by size:
//
// * direct (clouds below 56 Ki points, and grids that the others do not
//   take): init, then one lane per point with three atomics on its cell in
//   global memory, on values that need no decoding afterwards (zmax as the
//   float itself, see put_zmax; first as unsigned, -1 last): two launches
//   (20 000 points 6.3 us, three launches 8.6).  Bound by the atomics, about
//   27 G/s whatever their scope.  Many points a cell wait for each other there, and
//   the two atomics that the float's sign chooses from cost more than a third
//   launch: such clouds keep zmax as an ordered key, one atomic, and decode it
//   at the end (dense; 27 000 points in 836 cells 18.5 us against 20.3, 487 000
//   in 1316 234 against 299).
//
// * listed (56 Ki to 1 Mi points, no workspace): per chunk, the points sorted
//   by tile of the grid, as 16-bit places kept in the chunk's own part of
//   vidx; per tile, its points of all chunks reduced in LDS and written out;
//   last, the points' cells into vidx.  No atomics on global memory and no
//   partial tiles, at the price of reading the points three times (the second
//   time a 128-byte line for a few of its eight points, which bounds the
//   largest).  us, direct -> listed: 70 000 points 12.5 -> 10.7, 100 000
//   15.4 -> 11.1, 200 000 27.5 -> 12.8, 400 000 49.7 -> 17.7, 1 M 117 -> 31;
//   all points in one cell, 400 000: 5070 -> 1150.  (A cloud almost all
//   outside of the grid has no atomics to save: 400 000 points, 2 % inside,
//   6.9 -> 12.5; 15 % inside, 140 000 points 9.0 -> 11.1.)
//
// * binned (large clouds): the grid is cut into tiles of kTileCells cells,
//   small enough that one tile's accumulators live in LDS.  A tile takes its
//   cells from all over the grid (tiled): with consecutive cells the tiles of
//   a cloud's dense rows held twice the mean, and the reduction waited for
//   them (8 M points 84 -> 71 us, 4 M 46 -> 43, 1.1 M 33.5 -> 31.4; tiles of
//   4096 cells).
//     1. bin:    per chunk of kChunk points (read once), the cell of every
//                point (vidx) and an 8-byte record (z key, cell in tile,
//                index in chunk) per point, counting-sorted by tile in LDS
//                and written as one contiguous block, with the offsets of
//                its tile runs;
//     2. reduce: per (tile, group of chunks), the tile's runs of those
//                chunks reduced in LDS (count / max / min), written out as a
//                partial tile;
//     3. merge:  per cell, the partial tiles of its tile combined into the
//                outputs (empty cells: count 0, zmax -inf, first -1).
//   Global traffic is about 36 bytes per point (16 read and 4 written by
//   the points themselves, a record written and read back), with no global
//   atomics.
#include <algorithm>
#include <climits>
#include <cmath>
#include <cstdint>

#include "ops.hpp"

namespace ug {
namespace {

// Cells per tile: 24 KiB of LDS, five reduce workgroups a CU.  With 4096, two
// a CU, the reduction of a small cloud left half of the CUs idle (1.1 M
// points 31.3 -> 28.7 us, 2 M 33.4 -> 30.1, 4 M 43 -> 39.5, 8 M 70 -> 68).
constexpr int kTileBits = 11;
constexpr int kTileCells = 1 << kTileBits;
constexpr int kMaxTiles = 2048;                   // binned grids: <= 4 Mi cells
constexpr int64_t kChunk = 8192;                  // points per bin workgroup
static_assert(kChunk <= 8192, "a record keeps the index in its chunk in 13 bits");
constexpr int64_t kBinnedMinPoints = int64_t(1) << 20;
constexpr int64_t kMinChunksPerGroup = 64;        // tile reduce: chunks per workgroup, at least
constexpr unsigned kKeyNegInf = 0x007fffffu;      // key of -inf

// Order-preserving unsigned key of a float (-0 < +0).
__device__ __forceinline__ unsigned zkey(float z) {
  const unsigned u = __float_as_uint(z);
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
__device__ __forceinline__ float zval(unsigned k) {
  return __uint_as_float((k & 0x80000000u) ? (k & 0x7fffffffu) : ~k);
}

// Cell of a point, or -1.  Both subtractions and products are single FP32
// operations (no contraction), as the cell definition requires.
__device__ __forceinline__ int cell_of(float4 p, int nx, int ny, float xmin, float ymin,
                                       float scale) {
#pragma clang fp contract(off)
  const float fx = (p.x - xmin) * scale;
  const float fy = (p.y - ymin) * scale;
  // NaN fails every comparison and lands outside
  if (fx >= 0.0f && fx < (float)nx && fy >= 0.0f && fy < (float)ny) return (int)fy * nx + (int)fx;
  return -1;
}

// ------------------------------------------------------------------ direct
// KEYED: zmax holds keys until voxel_decode.
template <bool KEYED>
__global__ __launch_bounds__(256) void voxel_init(int* __restrict__ count,
                                                  float* __restrict__ zmax,
                                                  int* __restrict__ first, int64_t G) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < G; i += stride) {
    count[i] = 0;
    zmax[i] = KEYED ? __uint_as_float(kKeyNegInf) : -INFINITY;
    first[i] = -1;
  }
}

__global__ __launch_bounds__(256) void voxel_decode(float* __restrict__ zmax, int64_t G) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < G; i += stride)
    zmax[i] = zval(__float_as_uint(zmax[i]));
}

// Float maximum (-0 < +0) with integer atomics: of values without the sign
// bit the larger is the larger signed integer, above every value with it; of
// values with it the larger is the smaller unsigned integer, which every
// value without it is below.
__device__ __forceinline__ void put_zmax(float* at, float z) {
  const unsigned u = __float_as_uint(z);
  if (u & 0x80000000u)
    atomicMin(reinterpret_cast<unsigned*>(at), u);
  else
    atomicMax(reinterpret_cast<int*>(at), (int)u);
}

template <bool KEYED>
__global__ __launch_bounds__(256) void voxel_scatter(const float4* __restrict__ pts,
                                                     int* __restrict__ vidx,
                                                     int* __restrict__ count,
                                                     float* __restrict__ zmax,
                                                     int* __restrict__ first, int64_t N, int nx,
                                                     int ny, float xmin, float ymin, float scale) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < N; i += stride) {
    const float4 p = pts[i];
    const int v = cell_of(p, nx, ny, xmin, ymin, scale);
    if (v >= 0) {
      atomicAdd(&count[v], 1);
      if (KEYED)
        atomicMax(reinterpret_cast<unsigned*>(&zmax[v]), zkey(p.z));
      else
        put_zmax(&zmax[v], p.z);
      atomicMin(reinterpret_cast<unsigned*>(&first[v]), (unsigned)i);   // -1 is the largest
    }
    vidx[i] = v;
  }
}

// ------------------------------------------------------------------ binned
// Exclusive prefix sums of n <= 256 PER values (val(i) for i < n) into
// out[0..n], out[n] = total < 2^16, by one 256-lane workgroup (PER values a
// lane).  `wsum` is 4 ints of LDS.  Ends with a barrier.
template <int PER, typename F>
__device__ void block_scan_tiles(int n, F val, uint16_t* out, int* wsum) {
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  int a[PER], s = 0;
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    const int i = PER * t + k;
    a[k] = i < n ? val(i) : 0;
    s += a[k];
  }
  int incl = s;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const int y = __shfl_up(incl, d, 64);
    if (lane >= d) incl += y;
  }
  if (lane == 63) wsum[wave] = incl;
  __syncthreads();
  int off = incl - s;
  for (int w = 0; w < wave; ++w) off += wsum[w];
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    const int i = PER * t + k;
    if (i < n) out[i] = (uint16_t)off;
    off += a[k];
  }
  if (t == 255) out[n] = (uint16_t)off;
  __syncthreads();
}

// Where a cell is kept: blocks of 64 consecutive cells are dealt to the T
// tiles in turn, each round of T blocks one tile further, so that the rows and
// the columns of a dense part of the cloud spread over all tiles.  Returns
// tile << tb | place in the tile of 2^tb cells.  b < 2^16: the
// rounding errors of the quotients (2^-22 of at most 2^16 / T) stay below the
// 0.5 / T that part them from a wrong whole number.
__device__ __forceinline__ int tiled(int v, int T, float invT, int tb) {
  const int b = v >> 6;
  const int r = (int)(((float)b + 0.5f) * invT);   // b / T, below 2^(tb - 6)
  const int m = b - r * T + r;
  const int t = m - (int)(((float)m + 0.5f) * invT) * T;
  return (t << tb) | (r << 6) | (v & 63);
}

// 1. bin: one chunk of kChunk points per workgroup, read once.  Every lane
//    keeps its 32 points' cells and z keys in registers while the chunk's
//    tile histogram builds up in LDS; the exclusive scan of the histogram
//    gives each tile's run, the points are placed into their runs in LDS
//    (a counting sort by tile), and the chunk's records go out as one
//    contiguous block (chunk-major) with the run offsets H[c][0..T].  A
//    record is 8 bytes: z key (bits 0-31), cell within the tile (32-43),
//    point index within the chunk (44-56).
constexpr int kPerLane = kChunk / 256;

__device__ __forceinline__ uint64_t record(unsigned zk, int cell, int idx) {
  return (uint64_t)zk | ((uint64_t)(cell & (kTileCells - 1)) << 32) | ((uint64_t)idx << 44);
}

__global__ __launch_bounds__(256) void voxel_bin(const float4* __restrict__ pts,
                                                 int* __restrict__ vidx,
                                                 uint16_t* __restrict__ H, uint64_t* __restrict__ R, int64_t N, int nx,
                                                 int ny, float xmin, float ymin, float scale,
                                                 int T) {
  __shared__ int cur[kMaxTiles];       // histogram, then cursors
  __shared__ uint16_t off[kMaxTiles + 1];   // exclusive scan of the histogram
  __shared__ int wsum[4];
  __shared__ uint64_t rec[kChunk];     // the chunk's records, sorted by tile
  const int c = blockIdx.x;
  for (int t = threadIdx.x; t < T; t += 256) cur[t] = 0;
  __syncthreads();
  const int64_t beg = (int64_t)c * kChunk;
  const int64_t end = beg + kChunk < N ? beg + kChunk : N;
  const float invT = 1.0f / (float)T;
  int cell[kPerLane];   // as kept (tiled)
  unsigned zk[kPerLane];
  // eight points a lane in flight
#pragma unroll
  for (int u0 = 0; u0 < kPerLane; u0 += 8) {
    float4 p[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int64_t j = beg + threadIdx.x + (int64_t)(u0 + u) * 256;
      p[u] = j < end ? pts[j] : make_float4(0.f, 0.f, 0.f, 0.f);
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int64_t j = beg + threadIdx.x + (int64_t)(u0 + u) * 256;
      int v = -1;
      if (j < end) {
        v = cell_of(p[u], nx, ny, xmin, ymin, scale);
        vidx[j] = v;
        if (v >= 0) {
          v = tiled(v, T, invT, kTileBits);
          atomicAdd(&cur[v >> kTileBits], 1);
        }
      }
      cell[u0 + u] = v;
      zk[u0 + u] = zkey(p[u].z);
    }
  }
  __syncthreads();
  block_scan_tiles<kMaxTiles / 256>(T, [&](int i) { return cur[i]; }, off, wsum);
  uint16_t* h = H + (int64_t)c * (T + 1);
  for (int t = threadIdx.x; t <= T; t += 256) h[t] = off[t];
  for (int t = threadIdx.x; t < T; t += 256) cur[t] = off[t];
  __syncthreads();
#pragma unroll
  for (int u = 0; u < kPerLane; ++u) {
    if (cell[u] >= 0) {
      const int lp = atomicAdd(&cur[cell[u] >> kTileBits], 1);
      rec[lp] = record(zk[u], cell[u], threadIdx.x + u * 256);
    }
  }
  __syncthreads();
  const int n = off[T];
  uint64_t* out = R + beg;
  for (int i = threadIdx.x; i < n; i += 256) out[i] = rec[i];
}

// 2. one workgroup per (tile, group of chunks): the tile's runs of those
//    chunks reduced into LDS accumulators, written out as a partial tile.
//    The runs' bounds of the group's chunks (up to kStage at a time) are
//    staged in LDS first, all loaded at once; then each wavefront takes
//    eight chunks at a time (every fourth block of eight) and reduces their
//    runs in rounds of 128 records of every run, loaded together (sixteen
//    loads a lane in flight) before their atomics.
constexpr int kRunsAtOnce = 8;
constexpr int kStage = 1024;   // chunks whose run bounds sit in LDS at once

__device__ __forceinline__ void reduce_record(uint64_t r, int base, int* acc_c, unsigned* acc_z,
                                              int* acc_f) {
  const int cc = (int)((r >> 32) & (kTileCells - 1));
  atomicAdd(&acc_c[cc], 1);
  atomicMax(&acc_z[cc], (unsigned)r);
  atomicMin(&acc_f[cc], base + (int)(r >> 44));
}

__global__ __launch_bounds__(256) void voxel_tile_reduce(const uint16_t* __restrict__ H,
                                                         const uint64_t* __restrict__ R,
                                                         int* __restrict__ pc,
                                                         unsigned* __restrict__ pz,
                                                         int* __restrict__ pf, int T, int nb,
                                                         int groups, int cpg) {
  __shared__ int acc_c[kTileCells];
  __shared__ unsigned acc_z[kTileCells];
  __shared__ int acc_f[kTileCells];
  __shared__ int2 bnd[kStage];
  // chunk-group major: the workgroups resident together are the tiles of
  // a few chunk groups, which read neighbouring pieces of the same chunk
  // blocks (fewer distinct pages in flight than one tile's groups, which
  // span the whole record array)
  const int g = blockIdx.x / T, t = blockIdx.x % T;
  const int c0 = g * cpg, c1 = c0 + cpg < nb ? c0 + cpg : nb;
  for (int i = threadIdx.x; i < kTileCells; i += 256) {
    acc_c[i] = 0;
    acc_z[i] = kKeyNegInf;
    acc_f[i] = INT_MAX;
  }
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  for (int s0 = c0; s0 < c1; s0 += kStage) {
    const int s1 = s0 + kStage < c1 ? s0 + kStage : c1;
    __syncthreads();   // the previous stage's bounds are no longer read
    for (int c = s0 + threadIdx.x; c < s1; c += 256) {
      const uint16_t* h = H + (int64_t)c * (T + 1) + t;
      bnd[c - s0] = make_int2(h[0], h[1]);
    }
    __syncthreads();
    for (int cb = s0 + wave * kRunsAtOnce; cb < s1; cb += 4 * kRunsAtOnce) {
      int ra[kRunsAtOnce], rb[kRunsAtOnce];
      int longest = 0;   // the same in every lane
#pragma unroll
      for (int k = 0; k < kRunsAtOnce; ++k) {
        const int c = cb + k;
        const int2 ab = c < s1 ? bnd[c - s0] : make_int2(0, 0);
        ra[k] = ab.x;
        rb[k] = ab.y;
        longest = max(longest, ab.y - ab.x);
      }
      // rounds of 128 records of every run: sixteen loads a lane in flight
      for (int off = 0; off < longest; off += 128) {
        uint64_t r0[kRunsAtOnce], r1[kRunsAtOnce];
#pragma unroll
        for (int k = 0; k < kRunsAtOnce; ++k) {
          const uint64_t* run = R + (int64_t)(cb + k) * kChunk;
          const int i = ra[k] + off + lane;
          r0[k] = i < rb[k] ? run[i] : 0;
          r1[k] = i + 64 < rb[k] ? run[i + 64] : 0;
        }
#pragma unroll
        for (int k = 0; k < kRunsAtOnce; ++k) {
          const int base = (cb + k) * (int)kChunk;
          const int i = ra[k] + off + lane;
          if (i < rb[k]) reduce_record(r0[k], base, acc_c, acc_z, acc_f);
          if (i + 64 < rb[k]) reduce_record(r1[k], base, acc_c, acc_z, acc_f);
        }
      }
    }
  }
  __syncthreads();
  const int64_t o = ((int64_t)t * groups + g) * kTileCells;
  for (int i = threadIdx.x; i < kTileCells; i += 256) {
    pc[o + i] = acc_c[i];
    pz[o + i] = acc_z[i];
    pf[o + i] = acc_f[i];
  }
}

// 3. per cell: combine the partial tiles of its tile (the groups' partials
//    of tile t are partial tiles t * groups .. t * groups + groups - 1)
__global__ __launch_bounds__(256) void voxel_merge(const int* __restrict__ pc,
                                                   const unsigned* __restrict__ pz,
                                                   const int* __restrict__ pf,
                                                   int* __restrict__ count, float* __restrict__ zmax,
                                                   int* __restrict__ first, int64_t G, int T,
                                                   int groups) {
  const int64_t v = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (v >= G) return;
  const int at = tiled((int)v, T, 1.0f / (float)T, kTileBits);
  const int t = at >> kTileBits;
  const int l = at & (kTileCells - 1);
  int c = 0, f = INT_MAX;
  unsigned z = kKeyNegInf;
#pragma unroll 4
  for (int s = t * groups; s < (t + 1) * groups; ++s) {
    const int64_t o = (int64_t)s * kTileCells + l;
    c += pc[o];
    z = max(z, pz[o]);
    f = min(f, pf[o]);
  }
  count[v] = c;
  zmax[v] = zval(z);
  first[v] = c ? f : -1;
}

// ------------------------------------------------------------------ listed
// 1. list: per chunk of CHUNK points (the last chunk takes the rest, fewer
//    than two chunks), the points' places in the chunk sorted by tile, 16
//    bits each, behind the T + 1 offsets of the tiles' runs, written over the
//    chunk's own part of vidx (the first 2 (T + 1 + n) of its 4 n bytes).
constexpr int kListTiles = 256;      // tiles, at most: a workgroup a CU in the reduction
constexpr int kListThreads = 1024;   // lanes of the reduction: chunks, at most
constexpr int kListCells = 4096;     // of a tile, at most

template <int CHUNK>
__global__ __launch_bounds__(256) void voxel_list(const float4* __restrict__ pts,
                                                  uint32_t* __restrict__ lists, int64_t N, int nx,
                                                  int ny, float xmin, float ymin, float scale,
                                                  int T, int tb) {
  static_assert(2 * (kListTiles + 1 + CHUNK) < 4 * CHUNK, "the list fits in the chunk's vidx");
  constexpr int PER = 2 * CHUNK / 256;
  __shared__ int cur[kListTiles], wsum[4];
  __shared__ uint16_t off[kListTiles + 1];
  __shared__ uint32_t words[(kListTiles + 1 + 2 * CHUNK + 1) / 2];
  uint16_t* out = reinterpret_cast<uint16_t*>(words);
  const float invT = 1.0f / (float)T;
  const int64_t beg = (int64_t)blockIdx.x * CHUNK;
  const int n = (int)(blockIdx.x + 1 == gridDim.x ? N - beg : CHUNK);
  if ((int)threadIdx.x < T) cur[threadIdx.x] = 0;
  float4 p[PER];
#pragma unroll
  for (int u = 0; u < PER; ++u) {
    if (u >= PER / 2 && n <= CHUNK) break;
    p[u] = pts[beg + min((int)threadIdx.x + 256 * u, n - 1)];
  }
  __syncthreads();
  int tile[PER];
#pragma unroll
  for (int u = 0; u < PER; ++u) {
    if (u >= PER / 2 && n <= CHUNK) break;
    const int v = cell_of(p[u], nx, ny, xmin, ymin, scale);
    tile[u] = v >= 0 && (int)threadIdx.x + 256 * u < n ? tiled(v, T, invT, tb) >> tb : -1;
    if (tile[u] >= 0) atomicAdd(&cur[tile[u]], 1);
  }
  __syncthreads();
  block_scan_tiles<kListTiles / 256>(T, [&](int i) { return cur[i]; }, off, wsum);
  for (int t = threadIdx.x; t <= T; t += 256) {
    out[t] = off[t];
    if (t < T) cur[t] = T + 1 + off[t];
  }
  __syncthreads();
#pragma unroll
  for (int u = 0; u < PER; ++u) {
    if (u >= PER / 2 && n <= CHUNK) break;
    if (tile[u] >= 0) out[atomicAdd(&cur[tile[u]], 1)] = (uint16_t)(threadIdx.x + 256 * u);
  }
  __syncthreads();
  const int m = (T + 1 + off[T] + 1) / 2;
  for (int i = threadIdx.x; i < m; i += 256) lists[beg + i] = words[i];
}

// 2. reduce: one workgroup per tile.  The tile's runs of all chunks (at most
//    kListThreads) are laid end to end by a prefix sum of their lengths, so
//    that every lane has the same share of them whatever their lengths; each
//    point is read again for its cell in the tile and its z.
template <int CHUNK>
__global__ __launch_bounds__(kListThreads) void voxel_list_reduce(
    const float4* __restrict__ pts, const uint16_t* __restrict__ lists, int* __restrict__ count,
    float* __restrict__ zmax, int* __restrict__ first, int64_t G, int nx, int ny, float xmin,
    float ymin, float scale, int T, int tb, int nb) {
  __shared__ int acc_c[kListCells], acc_f[kListCells];
  __shared__ unsigned acc_z[kListCells];
  __shared__ int pre[kListThreads];   // points of the tile in the chunks before
  __shared__ int at[kListThreads];    // where a chunk's run starts in the lists, less pre
  __shared__ int wsum[kListThreads / 64];
  const float invT = 1.0f / (float)T;
  const int t = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  int a = 0, len = 0;
  if (tid < nb) {
    const uint16_t* h = lists + (int64_t)tid * (2 * CHUNK) + t;
    a = h[0];
    len = h[1] - a;
  }
  for (int i = tid; i < 1 << tb; i += kListThreads) {
    acc_c[i] = 0;
    acc_z[i] = kKeyNegInf;
    acc_f[i] = INT_MAX;
  }
  int incl = len;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const int y = __shfl_up(incl, d, 64);
    if (lane >= d) incl += y;
  }
  if (lane == 63) wsum[wave] = incl;
  __syncthreads();
  int base = 0, total = 0;
#pragma unroll
  for (int w = 0; w < kListThreads / 64; ++w) {
    base += w < wave ? wsum[w] : 0;
    total += wsum[w];
  }
  const int excl = base + incl - len;
  pre[tid] = excl;
  at[tid] = tid * (2 * CHUNK) + T + 1 + a - excl;
  __syncthreads();
  constexpr int U = 4;   // points of a lane in flight
  for (int i0 = tid; i0 < total; i0 += U * kListThreads) {
    int64_t j[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int i = min(i0 + u * kListThreads, total - 1);
      int c = 0;   // the last chunk with pre <= i
#pragma unroll
      for (int d = kListThreads / 2; d > 0; d >>= 1)
        if (pre[c + d] <= i) c += d;
      j[u] = (int64_t)c * CHUNK + lists[at[c] + i];
    }
    float4 p[U];
#pragma unroll
    for (int u = 0; u < U; ++u) p[u] = pts[j[u]];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (i0 + u * kListThreads >= total) break;
      const int l =
          tiled(cell_of(p[u], nx, ny, xmin, ymin, scale), T, invT, tb) & ((1 << tb) - 1);
      atomicAdd(&acc_c[l], 1);
      atomicMax(&acc_z[l], zkey(p[u].z));
      atomicMin(&acc_f[l], (int)j[u]);
    }
  }
  __syncthreads();
  for (int l = tid; l < 1 << tb; l += kListThreads) {
    const int r = l >> 6;
    const int m = t - r;   // mod T: the block's place in its round
    const int64_t v = ((int64_t)r * T + m + (T - 1 - m) / T * T) * 64 + (l & 63);
    if (v < G) {
      const int c = acc_c[l];
      count[v] = c;
      zmax[v] = zval(acc_z[l]);
      first[v] = c ? acc_f[l] : -1;
    }
  }
}

// 3. cells: the points' cells into vidx, now that the lists have been read.
__global__ __launch_bounds__(256) void voxel_cells(const float4* __restrict__ pts,
                                                   int* __restrict__ vidx, int64_t N, int nx,
                                                   int ny, float xmin, float ymin, float scale) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < N; i += stride)
    vidx[i] = cell_of(pts[i], nx, ny, xmin, ymin, scale);
}

unsigned grid_for(int64_t work, int64_t cap) {
  int64_t g = (work + 255) / 256;
  if (g > cap) g = cap;
  if (g < 1) g = 1;
  return (unsigned)g;
}

// Workspace of the binned path, in 256-byte aligned pieces: the chunks' run
// offsets, their records (kChunk slots per chunk), the partial tiles.
struct Binned {
  int T = 0, nb = 0, groups = 0, cpg = 0;
  size_t H = 0, R = 0, pc = 0, pz = 0, pf = 0, total = 0;
};

bool use_binned(int64_t N, int64_t G) {
  return N >= kBinnedMinPoints && (G + kTileCells - 1) / kTileCells <= kMaxTiles;
}

Binned binned_layout(int64_t N, int64_t G) {
  Binned b;
  b.T = (int)((G + kTileCells - 1) / kTileCells);
  b.nb = (int)((N + kChunk - 1) / kChunk);
  // The workspace holds the partial tiles of up to about 2048 workgroups of
  // 4096 cells, of at least kMinChunksPerGroup chunks each.
  const int T2 = (b.T + 1) / 2;
  const int most = (int)std::max<int64_t>(
      1, std::min<int64_t>(b.nb / kMinChunksPerGroup, (2048 + T2 - 1) / T2));
  // A workgroup's time grows with its chunks, the partial tiles written and
  // read back with the groups: the best number grows as the root of the
  // chunks (4 M points 39.2 to 39.5 us at 4 to 6 groups, 40 at 3 and 7; 8 M
  // 67.3 to 68 at 4 to 8, 70.5 at 3).
  b.groups = std::max(1, std::min(most, (int)std::lround(std::sqrt((double)b.nb) / 4)));
  b.cpg = (b.nb + b.groups - 1) / b.groups;
  size_t off = 0;
  auto take = [&](size_t bytes) {
    const size_t at = off;
    off += (bytes + 255) / 256 * 256;
    return at;
  };
  b.H = take(sizeof(uint16_t) * (size_t)b.nb * (b.T + 1));
  b.R = take(sizeof(uint64_t) * (size_t)b.nb * kChunk);
  const size_t parts = (size_t)b.T * most * kTileCells;
  b.pc = take(sizeof(int) * parts);
  b.pz = take(sizeof(unsigned) * parts);
  b.pf = take(sizeof(int) * parts);
  b.total = off;
  return b;
}

// The listed path's tiles and chunks (tb 0: not taken).  Below 56 Ki points
// the direct path's two launches are faster (50 000 9.8 against 10.5 us,
// 70 000 12.5 against 10.7); a grid of fewer than 64 tiles of 64 cells leaves
// the reduction too few workgroups, one of more than 256 tiles of 4096 has no
// room for its offsets.  Chunks of 512 points up to 256 Ki (100 000 11.1
// against 11.9; 400 000 equal).
constexpr int64_t kListedMinPoints = 56 << 10, kListedSmallChunk = 256 << 10;
struct Listed {
  int tb = 0, T = 0, nb = 0;
  bool small = false;
};
Listed listed(int64_t N, int64_t G) {
  Listed l;
  if (N < kListedMinPoints || N / 1024 > kListThreads || G <= 63 * 64 ||
      G > (int64_t)kListTiles * kListCells)
    return l;
  l.tb = 6;
  while (((G - 1) >> l.tb) >= kListTiles) ++l.tb;
  l.T = (int)((G - 1) >> l.tb) + 1;
  l.small = N <= kListedSmallChunk;
  l.nb = (int)(N / (l.small ? 512 : 1024));
  return l;
}

}  // namespace

// Direct clouds whose cells are contended (us, float / keys: 52 600 points, 14.5 a
// cell 25.4 / 21.9; 55 000, 17 a cell 15.8 / 15.9; 49 000, 7 a cell 17.3 / 16.7; 30 000, 7 a
// cell 7.7 / 9.3).
static bool dense(int64_t N, int64_t G) { return N >= (24 << 10) && N >= 12 * G; }

size_t voxel_f32_workspace(int64_t N, int nx, int ny) {
  const int64_t G = (int64_t)nx * ny;
  return use_binned(N, G) ? binned_layout(N, G).total : 0;
}

OpPlan voxel_f32_plan(int64_t N, int nx, int ny) {
  OpPlan p;
  p.block = dim3(256);
  const int64_t G = (int64_t)nx * ny;
  if (use_binned(N, G)) {
    // the widest of the three launches: one lane per cell in the merge
    p.func = reinterpret_cast<const void*>(&voxel_merge);
    p.grid = dim3(grid_for(G, INT_MAX));
  } else {
    // one lane per point
    p.func = listed(N, G).tb ? reinterpret_cast<const void*>(&voxel_cells)
             : dense(N, G) ? reinterpret_cast<const void*>(&voxel_scatter<true>)
                           : reinterpret_cast<const void*>(&voxel_scatter<false>);
    p.grid = dim3(grid_for(N, 256 * 32));
  }
  return p;
}

hipError_t voxel_f32_launch(const float* pts, int* vidx, int* count, float* zmax, int* first,
                            int64_t N, int nx, int ny, float xmin, float ymin, float scale,
                            void* ws, size_t ws_bytes, hipStream_t s) {
  const int64_t G = (int64_t)nx * ny;
  const dim3 blk(256);
  const float4* p4 = reinterpret_cast<const float4*>(pts);
  if (use_binned(N, G)) {
    const Binned b = binned_layout(N, G);
    if (!ws || ws_bytes < b.total || (reinterpret_cast<uintptr_t>(ws) & 255))
      return hipErrorInvalidValue;
    char* w = static_cast<char*>(ws);
    uint16_t* H = reinterpret_cast<uint16_t*>(w + b.H);
    uint64_t* R = reinterpret_cast<uint64_t*>(w + b.R);
    int* pc = reinterpret_cast<int*>(w + b.pc);
    unsigned* pz = reinterpret_cast<unsigned*>(w + b.pz);
    int* pf = reinterpret_cast<int*>(w + b.pf);
    hipLaunchKernelGGL(voxel_bin, dim3(b.nb), blk, 0, s, p4, vidx, H, R, N, nx, ny, xmin, ymin,
                       scale, b.T);
    hipLaunchKernelGGL(voxel_tile_reduce, dim3(b.T * b.groups), blk, 0, s, H, R, pc, pz, pf, b.T,
                       b.nb, b.groups, b.cpg);
    hipLaunchKernelGGL(voxel_merge, dim3(grid_for(G, INT_MAX)), blk, 0, s, pc, pz, pf, count,
                       zmax, first, G, b.T, b.groups);
    return hipGetLastError();
  }
  if (const Listed l = listed(N, G); l.tb) {
    uint32_t* lists = reinterpret_cast<uint32_t*>(vidx);
    const uint16_t* lists16 = reinterpret_cast<const uint16_t*>(vidx);
    const dim3 wide(kListThreads);
    if (l.small) {
      hipLaunchKernelGGL(voxel_list<512>, dim3(l.nb), blk, 0, s, p4, lists, N, nx, ny, xmin, ymin,
                         scale, l.T, l.tb);
      hipLaunchKernelGGL(voxel_list_reduce<512>, dim3(l.T), wide, 0, s, p4, lists16, count, zmax,
                         first, G, nx, ny, xmin, ymin, scale, l.T, l.tb, l.nb);
    } else {
      hipLaunchKernelGGL(voxel_list<1024>, dim3(l.nb), blk, 0, s, p4, lists, N, nx, ny, xmin,
                         ymin, scale, l.T, l.tb);
      hipLaunchKernelGGL(voxel_list_reduce<1024>, dim3(l.T), wide, 0, s, p4, lists16, count, zmax,
                         first, G, nx, ny, xmin, ymin, scale, l.T, l.tb, l.nb);
    }
    hipLaunchKernelGGL(voxel_cells, dim3(grid_for(N, 256 * 32)), blk, 0, s, p4, vidx, N, nx, ny,
                       xmin, ymin, scale);
    return hipGetLastError();
  }
  const dim3 cells(grid_for(G, 256 * 8)), points(grid_for(N, 256 * 32));
  if (dense(N, G)) {
    hipLaunchKernelGGL(voxel_init<true>, cells, blk, 0, s, count, zmax, first, G);
    hipLaunchKernelGGL(voxel_scatter<true>, points, blk, 0, s, p4, vidx, count, zmax, first, N, nx,
                       ny, xmin, ymin, scale);
    hipLaunchKernelGGL(voxel_decode, cells, blk, 0, s, zmax, G);
    return hipGetLastError();
  }
  hipLaunchKernelGGL(voxel_init<false>, cells, blk, 0, s, count, zmax, first, G);
  if (N > 0) {
    hipLaunchKernelGGL(voxel_scatter<false>, points, blk, 0, s, p4, vidx, count, zmax, first, N, nx,
                       ny, xmin, ymin, scale);
  }
  return hipGetLastError();
}

}  // namespace ug
