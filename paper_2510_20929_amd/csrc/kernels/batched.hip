// Many independent reconstructions of uneven frame size in a few persistent launches.
//
// Datasets are grouped by frame size (64^2, 128^2, 256^2, 512^2) and loss form, and each
// class runs as one persistent launch with that frame size's thread layout (the loss form
// a compile-time choice, as in the per-plan kernels). A launch's workgroups are
// partitioned among its datasets so that the longest of them is shortest in whole rounds of
// positions; every workgroup reads its
// dataset's call arguments from a device descriptor table (sorted by class, then by
// first workgroup) and runs the same per-position body as the per-plan kernels (512
// threads for 64^2; 1024 for 128^2, with the frame in LDS; 1024 and 512 for the
// four-step frames 256^2 and 512^2). Gathers, probe reductions and final reductions follow, one
// launch each for all datasets of the class; they too read their pointers from the
// table, so a captured graph stays valid when the caller rebinds buffers.
#include <algorithm>

#include "big_body.hpp"
#include "gather.hpp"
#include "launch.hpp"
#include "lds_body.hpp"

namespace ptyhip {

// 128^2: the frame resident in LDS, dl/dI in registers (640 positions of 2 modes and 263 of 4:
// 568 us; 546 against 572 with patch and frame in registers, both on other transforms)
template <int LOSS>
__global__ __launch_bounds__(1024) void batched_128_kernel(const BatchEntry* __restrict__ tab, int n) {
  __shared__ LdsShared<128, 1024> sh;
  const int d = batch_dataset(tab, n);
  const CallArgs a = tab[d].a;
  const int wg = int(blockIdx.x) - tab[d].first_wg, nwg = tab[d].n_wg;
  if (a.mode == MODE_FWD_ADJ) lds_body<128, 1024, LOSS, true, true>(a, sh, wg, nwg);
  else lds_body<128, 1024, LOSS, true, false>(a, sh, wg, nwg);
}

template <int N, int T, int LOSS>
__global__ __launch_bounds__(T, N == 256 ? 4 : 2) void batched_big_kernel(const BatchEntry* __restrict__ tab, int n) {
  __shared__ BigShared<N, T> sh;
  const int d = batch_dataset(tab, n);
  const CallArgs a = tab[d].a;
  const int wg = int(blockIdx.x) - tab[d].first_wg, nwg = tab[d].n_wg;
  if (a.mode == MODE_FWD_ADJ) big_body<N, T, LOSS, 0, true>(a, sh, wg, nwg);
  else big_body<N, T, LOSS, 0, false>(a, sh, wg, nwg);
}

int batch_class(int N, int loss) { return 2 * (N <= 64 ? 0 : (N == 128 ? 1 : (N == 256 ? 2 : 3))) + (loss ? 1 : 0); }

int batch_variant(int N) { return N == 128 ? 6 : 0; }

size_t batched_scratch_elems(int N, int M, int E, int recompute, size_t* pacc_off) {
  if (N <= 128) return fused_small_scratch_elems(N, 1, M, E, recompute, pacc_off, batch_variant(N));
  return big_scratch_elems(N, M, E, pacc_off);
}

// Window gathers of every dataset of a class in one launch: the class's datasets own
// consecutive ranges of workgroups (first_tile; gather_tiles() of tile side gts each, none
// for a dataset without an object gradient). GP: two groups of threads per tile if every dataset
// asks for more than one (gather_groups; 4 dense scans of 64^2, 300 positions on 110^2: the whole launch
// 124 us with two, 156 with one; 2 of 256^2, 400 positions on 500^2: 900 and 936), otherwise one (a
// dataset of few windows loses more by two than another gains: 2 + 2 + 2 + 2 datasets of 64^2 to
// 512^2, 492 us with one, 552 with two).
template <int GP>
__global__ __launch_bounds__(256 * GP) void batch_gather_kernel(const BatchEntry* __restrict__ tab, int n) {
  int d = 0;
  while (d + 1 < n && int(blockIdx.x) >= tab[d + 1].first_tile) ++d;
  const BatchEntry& e = tab[d];
  const GatherArgs& g = e.g;
  const int b = int(blockIdx.x) - e.first_tile;
  int bx, by, bz;
  // no gather for this dataset, or padding of its range (uniform per workgroup)
  if (b < 0 || e.tiles_x == 0 || !gather_tile_of(b, e.tiles_x, e.tiles_y, g.S, bx, by, bz)) return;
  if (e.gts == GT)
    gather_tile_at<float2, GT, GP>(g.gwin, g.wvalid, g.pos, g.gobj, g.K, g.S, g.N, g.H, g.W, g.accumulate, g.rep, bx,
                                   by, bz);
  else
    gather_tile_at<float2, GT / 2, GP>(g.gwin, g.wvalid, g.pos, g.gobj, g.K, g.S, g.N, g.H, g.W, g.accumulate, g.rep,
                                       bx, by, bz);
}

// probe gradients of every dataset of a class (blockIdx.y: dataset): the sum of the
// dataset's workgroup accumulators; the 64^2 body stores element i of thread t at
// i*T + t, the others in natural order
template <int N, int T = 512>
__global__ void batch_probe_reduce_kernel(const BatchEntry* __restrict__ tab) {
  const BatchEntry& e = tab[blockIdx.y];
  if (e.g_probe == nullptr || e.a.mode != MODE_FWD_ADJ) return;
  const CallArgs& a = e.a;
  float2* out = e.g_probe;
  const int groups = e.n_wg;
  constexpr size_t NN = size_t(N) * N;
  const size_t n = size_t(a.E) * a.M * NN;
  for (size_t g = size_t(blockIdx.x) * blockDim.x + threadIdx.x; g < n; g += size_t(gridDim.x) * blockDim.x) {
    const size_t em = g / NN, r = g % NN;
    const float2* src = a.scratch + a.pacc_off + em * NN + r;
    float2 s = make_float2(0.f, 0.f);
    // eight workgroups' loads in flight, added in order
    int w = 0;
    for (; w + 8 <= groups; w += 8) {
      float2 v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] = src[size_t(w + u) * a.scratch_stride];
#pragma unroll
      for (int u = 0; u < 8; ++u) s = cadd(s, v[u]);
    }
    for (; w < groups; ++w) s = cadd(s, src[size_t(w) * a.scratch_stride]);
    size_t pix = r;
    if constexpr (N < 128) pix = size_t(SmallCtx<N, T>::a_pix(int(r % T), int(r / T)));
    out[em * NN + pix] = s;
  }
}

// loss, position and weight gradients of every dataset of a class (blockIdx.x: dataset)
__global__ __launch_bounds__(1024) void batch_finalize_kernel(const BatchEntry* __restrict__ tab) {
  __shared__ double red[1024 / WAVE];
  const BatchEntry& e = tab[blockIdx.x];
  const CallArgs& a = e.a;
  double s = 0.0;
  for (int k = threadIdx.x; k < a.K; k += 1024) s += a.loss_part[k];
  s = block_sum<1024>(s, red);
  if (threadIdx.x == 0 && e.loss) *e.loss = s;
  if (e.g_pos && a.pos_part)
    for (int i = threadIdx.x; i < 2 * a.K; i += 1024) e.g_pos[i] = float(a.pos_part[i]);
  if (e.g_w && a.w_part)
    for (int i = threadIdx.x; i < a.E * a.K; i += 1024) e.g_w[i] = float(a.w_part[i]);
}

// One frame-size class: its persistent launch, then one launch each for the window
// gathers, the probe reductions and the final reductions of its datasets (table entries
// [cls_first[c], cls_first[c] + cls_count[c])).
hipError_t launch_batched_class(const BatchEntry* dev_tab, const BatchEntry* host_tab, int c, const int* cls_first,
                                const int* cls_count, const int* cls_wg, hipStream_t st) {
  const int nc = cls_count[c];
  if (nc == 0) return hipSuccess;
  const BatchEntry* t = dev_tab + cls_first[c];
  const BatchEntry* h = host_tab + cls_first[c];
  const dim3 grid{unsigned(cls_wg[c])};
  switch (c) {
    case 0: launch_batched64(t, nc, 0, grid, st); break;
    case 1: launch_batched64(t, nc, 1, grid, st); break;
    case 2: hipLaunchKernelGGL(batched_128_kernel<0>, grid, dim3(1024), 0, st, t, nc); break;
    case 3: hipLaunchKernelGGL(batched_128_kernel<1>, grid, dim3(1024), 0, st, t, nc); break;
    case 4: hipLaunchKernelGGL((batched_big_kernel<256, 1024, 0>), grid, dim3(1024), 0, st, t, nc); break;
    case 5: hipLaunchKernelGGL((batched_big_kernel<256, 1024, 1>), grid, dim3(1024), 0, st, t, nc); break;
    case 6: hipLaunchKernelGGL((batched_big_kernel<512, 512, 0>), grid, dim3(512), 0, st, t, nc); break;
    default: hipLaunchKernelGGL((batched_big_kernel<512, 512, 1>), grid, dim3(512), 0, st, t, nc); break;
  }
  int tiles = 0, groups = 2;
  size_t nel = 0;
  for (int d = 0; d < nc; ++d) {
    if (h[d].a.mode != MODE_FWD_ADJ) continue;
    if (h[d].tiles_x) {
      const GatherArgs& g = h[d].g;
      tiles = std::max(tiles, h[d].first_tile + gather_tiles(g.H, g.W, g.S, h[d].gts));
      groups = std::min(groups, gather_groups(g.K, g.S, g.N, g.H, g.W, h[d].gts));
    }
    if (h[d].g_probe) nel = std::max(nel, size_t(h[d].a.E) * h[d].a.M * h[d].N * h[d].N);
  }
  if (tiles > 0 && groups > 1)
    hipLaunchKernelGGL(batch_gather_kernel<2>, dim3(unsigned(tiles)), dim3(512), 0, st, t, nc);
  else if (tiles > 0)
    hipLaunchKernelGGL(batch_gather_kernel<1>, dim3(unsigned(tiles)), dim3(256), 0, st, t, nc);
  if (nel > 0) {
    const dim3 pg(unsigned(std::min<size_t>(4096, (nel + 255) / 256)), unsigned(nc));
    switch (h[0].N) {
      case 64: hipLaunchKernelGGL(batch_probe_reduce_kernel<64>, pg, dim3(256), 0, st, t); break;
      case 128: hipLaunchKernelGGL((batch_probe_reduce_kernel<128, 1024>), pg, dim3(256), 0, st, t); break;
      case 256: hipLaunchKernelGGL(batch_probe_reduce_kernel<256>, pg, dim3(256), 0, st, t); break;
      case 512: hipLaunchKernelGGL(batch_probe_reduce_kernel<512>, pg, dim3(256), 0, st, t); break;
      default: return hipErrorInvalidValue;
    }
  }
  hipLaunchKernelGGL(batch_finalize_kernel, dim3(unsigned(nc)), dim3(1024), 0, st, t);
  return hipGetLastError();
}

hipError_t launch_batched(const BatchEntry* dev_tab, const BatchEntry* host_tab, int n, const int* cls_first,
                          const int* cls_count, const int* cls_wg, hipStream_t st) {
  (void)n;
  for (int c = 0; c < BATCH_CLASSES; ++c) {
    const hipError_t e = launch_batched_class(dev_tab, host_tab, c, cls_first, cls_count, cls_wg, st);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace ptyhip
