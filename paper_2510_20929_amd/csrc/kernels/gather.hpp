// Object gradient from the per-position window gradients: the transpose of the patch
// extraction summed over positions, done as a gather. Each workgroup owns a 32 x 32
// (or, for objects too small to fill the GPU with such tiles, 16 x 16) tile of one slice and
// walks the positions in order (staged through LDS), adding the part of every valid window
// that covers the tile. Every object pixel is written exactly once (no atomics, fixed
// summation order). Bound by the read of the windows (2500 of 257^2: 1.3 GB, 343 us) where
// tiles fill the GPU, by the latency of a tile's walk where they do not (gather_groups).
#pragma once
#include <climits>

#include "../device/common.hpp"
#include "launch.hpp"

namespace ptyhip {

__device__ __forceinline__ float vadd(float a, float b) { return a + b; }
__device__ __forceinline__ float2 vadd(float2 a, float2 b) { return cadd(a, b); }
template <class V> __device__ __forceinline__ V vzero();
template <> __device__ __forceinline__ float vzero<float>() { return 0.f; }
template <> __device__ __forceinline__ float2 vzero<float2>() { return make_float2(0.f, 0.f); }

// One TS x TS tile (bx, by) of slice bz; GP groups of 256 threads (4 waves), a thread
// owning TS^2 / 256 pixels of a column.
// Positions are taken in chunks: every thread tests a position for overlap with the
// tile, the hits are compacted in position order (wave ballots + a block prefix, so the
// order never depends on timing), and then the groups take runs of HB hits in turn, each
// thread issuing the loads of a run at its pixels before adding them in order. The groups'
// sums are added in group order at the end.
// `win` holds [K][S][N+1][N+1] windows of value type V (float2 gradients, float
// illumination), `out` the [S][H][W] result.
// `rep` windows share one position (window k belongs to position k / rep; the mode-split
// form writes one window per mode group).
template <class V, int TS, int GP>
__device__ __forceinline__ void gather_tile_at(const V* __restrict__ win, const int* __restrict__ wvalid,
                                               const float* __restrict__ pos, V* out_all, int K, int S, int N,
                                               int H, int W, int accumulate, int rep, int bx, int by, int bz) {
  constexpr int NT = 256;
  constexpr int CH = 1024;  // positions examined per chunk
  __shared__ int hy[CH], hx[CH], hk[CH];
  __shared__ int wcnt[GP * NT / 64];
  constexpr int RPP = NT / TS;  // rows per pass
  constexpr int PJ = TS / RPP;   // passes (pixels per thread)
  constexpr int HB = PJ == 1 ? 8 : 4;  // hits whose loads are in flight together
  static_assert(RPP * TS == NT && PJ * RPP == TS, "the tile must split evenly over the threads");
  __shared__ V part[GP > 1 ? (GP - 1) * PJ * NT : 1];
  const int WN = N + 1;
  const int tx0 = bx * TS, ty0 = by * TS, s = bz;
  const int t = threadIdx.x % NT, c = t % TS, r0 = t / TS;
  const int x = tx0 + c;
  const int lane = threadIdx.x & 63, wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), grp = wid / (NT / 64);
  V acc[PJ];
#pragma unroll
  for (int j = 0; j < PJ; ++j) acc[j] = vzero<V>();
  const size_t wsz = size_t(WN) * WN;
  const V z = vzero<V>();
  for (int k0 = 0; k0 < K; k0 += CH) {
    const int n = min(CH, K - k0);
    int nh = 0;
    __syncthreads();  // the previous chunk's hits are consumed
    for (int r = 0; r < CH / (GP * NT); ++r) {
      const int i = r * GP * NT + int(threadIdx.x);
      const int k = k0 + i;
      int y0 = 0, x0 = 0;
      bool hit = false;
      if (i < n && wvalid[k]) {
        const int kp = rep > 1 ? k / rep : k;
        y0 = int(floorf(pos[2 * kp]));
        x0 = int(floorf(pos[2 * kp + 1]));
        hit = !(y0 > ty0 + TS - 1 || y0 + WN - 1 < ty0 || x0 > tx0 + TS - 1 || x0 + WN - 1 < tx0);
      }
      const unsigned long long b = __ballot(hit);
      if (lane == 0) wcnt[wid] = __popcll(b);
      __syncthreads();
      int base = nh, tot = 0;
#pragma unroll
      for (int w = 0; w < GP * NT / 64; ++w) {
        base += w < wid ? wcnt[w] : 0;
        tot += wcnt[w];
      }
      if (hit) {
        const int at = base + __popcll(b & ((1ull << lane) - 1));
        hy[at] = y0;
        hx[at] = x0;
        hk[at] = k;
      }
      nh += tot;
      __syncthreads();  // wcnt is rewritten by the next round; the hits are visible
    }
    for (int h = grp * HB; h < nh; h += GP * HB) {
      V v[HB][PJ];
#pragma unroll
      for (int u = 0; u < HB; ++u) {
        const bool on = h + u < nh;
        const int hh = on ? h + u : nh - 1;  // in-range LDS slot also for the unused tail
        const int y0 = hy[hh], px = on ? x - hx[hh] : -1;
        const V* w = win + (size_t(hk[hh]) * S + s) * wsz;
#pragma unroll
        for (int j = 0; j < PJ; ++j) {
          const int py = ty0 + r0 + RPP * j - y0;
          v[u][j] = (px >= 0 && px < WN && py >= 0 && py < WN) ? w[size_t(py) * WN + px] : z;
        }
      }
#pragma unroll
      for (int u = 0; u < HB; ++u)
#pragma unroll
        for (int j = 0; j < PJ; ++j) acc[j] = vadd(acc[j], v[u][j]);
    }
  }
  if constexpr (GP > 1) {
    if (grp > 0) {
#pragma unroll
      for (int j = 0; j < PJ; ++j) part[((grp - 1) * PJ + j) * NT + t] = acc[j];
    }
    __syncthreads();
    if (grp > 0) return;
#pragma unroll
    for (int g = 1; g < GP; ++g)
#pragma unroll
      for (int j = 0; j < PJ; ++j) acc[j] = vadd(acc[j], part[((g - 1) * PJ + j) * NT + t]);
  }
  if (x >= W) return;
  V* out = out_all + size_t(s) * H * W;
#pragma unroll
  for (int j = 0; j < PJ; ++j) {
    const int y = ty0 + r0 + RPP * j;
    if (y < H) {
      V* o = out + size_t(y) * W + x;
      *o = accumulate ? vadd(*o, acc[j]) : acc[j];
    }
  }
}

// Tile b of a launch of gather_tiles() workgroups: the tile rows go round the eight XCDs
// (workgroup b runs on XCD b mod 8), so that the lines which a tile's unaligned rows share
// with its neighbours' are read into one L2 (6732 positions of 128^2, four groups of threads: 299 ->
// 271 us; 2500 of 256^2, one group: 418 -> 390). False: no tile.
__device__ __forceinline__ bool gather_tile_of(int b, int tiles_x, int tiles_y, int S, int& bx, int& by, int& bz) {
  const int j = b >> 3, row = j / tiles_x * 8 + (b & 7);
  bx = j % tiles_x;
  by = row % tiles_y;
  bz = row / tiles_y;
  return row < tiles_y * S;
}

template <class V, int TS, int GP>
__device__ __forceinline__ void gather_tile_t(const V* __restrict__ win, const int* __restrict__ wvalid,
                                              const float* __restrict__ pos, V* out_all, int K, int S, int N,
                                              int H, int W, int accumulate, int rep = 1) {
  int bx, by, bz;
  if (!gather_tile_of(blockIdx.x, (W + TS - 1) / TS, (H + TS - 1) / TS, S, bx, by, bz)) return;
  gather_tile_at<V, TS, GP>(win, wvalid, pos, out_all, K, S, N, H, W, accumulate, rep, bx, by, bz);
}

}  // namespace ptyhip
