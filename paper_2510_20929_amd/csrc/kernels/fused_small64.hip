// Fused kernels of 64^2 frames, per plan and batched.
#include "fused_small.hpp"

namespace ptyhip {

// 512 threads: the state of a thread's eight pixels fits in registers (variants 0 and 2). Bound by
// the latency of a position's chain of loads and barriers: 625 positions on 512 workgroups
// 36.0 us, 24 positions of 2 modes 22.9 (43.9 and 28.6 with the patch in scratch, four loads
// per pixel, the measured intensities loaded when needed, per-pixel window indices and the
// accumulator cleared and read by every workgroup)
hipError_t launch_fused_small64(const CallArgs& a, int variant, int grid, hipStream_t st) {
  if (variant == 1) return launch_small_t<64, 256>(a, grid, st);
  if (variant == 3) return launch_small_t<64, 256, true>(a, grid, st);
  if (variant == 4) return launch_small_t<64, 256, true, false>(a, grid, st);
  return launch_small_t<64, 512, true>(a, grid, st);
}

hipError_t launch_probe_reduce64(const CallArgs& a, int threads, int grid, float2* g_probe, int accumulate,
                                 hipStream_t st) {
  return threads == 256 ? probe_reduce_t<64, 256>(a, grid, g_probe, accumulate, st)
                        : probe_reduce_t<64, 512>(a, grid, g_probe, accumulate, st);
}

// the 64^2 class of a batched launch (entries tab[0..n), a dataset per range of workgroups)
template <int LOSS>
__global__ __launch_bounds__(512, 4) void batched_64_kernel(const BatchEntry* __restrict__ tab, int n) {
  __shared__ SmallShared<64, 512> sh;
  const int d = batch_dataset(tab, n);
  const CallArgs a = tab[d].a;
  const int wg = int(blockIdx.x) - tab[d].first_wg, nwg = tab[d].n_wg;
  small_body<64, 512, LOSS, true>(a, sh, wg, nwg);
}

void launch_batched64(const BatchEntry* tab, int n, int loss, dim3 grid, hipStream_t st) {
  if (loss == 0) hipLaunchKernelGGL(batched_64_kernel<0>, grid, dim3(512), 0, st, tab, n);
  else hipLaunchKernelGGL(batched_64_kernel<1>, grid, dim3(512), 0, st, tab, n);
}

}  // namespace ptyhip
