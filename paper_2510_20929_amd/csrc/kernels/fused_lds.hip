// Fused forward + adjoint kernels of 128^2 frames with the working frame resident in LDS
// (tune variants 5 and 6): single-slice (lds_body) and multislice (lds_ms_body); and the
// near field of every variant (lds_near_body).
#include "launch.hpp"
#include "lds_body.hpp"
#include "lds_ms.hpp"
#include "lds_near.hpp"

namespace ptyhip {

template <int N, int T, int LOSS, bool CFREG, bool FA>
__global__ __launch_bounds__(T) void fused_small_lds_kernel(CallArgs a) {
  __shared__ LdsShared<N, T> sh;
  lds_body<N, T, LOSS, CFREG, FA>(a, sh, blockIdx.x, gridDim.x);
}

template <int N, int T, int LOSS, bool LZ, bool FA>
__global__ __launch_bounds__(T) void fused_small_lds_ms_kernel(CallArgs a) {
  __shared__ LdsShared<N, T> sh;
  lds_ms_body<N, T, LOSS, LZ, FA>(a, sh, blockIdx.x, gridDim.x);
}

template <int N, int T, int LOSS, bool FA>
__global__ __launch_bounds__(T) void fused_small_lds_near_kernel(CallArgs a) {
  __shared__ LdsShared<N, T> sh;
  lds_near_body<N, T, LOSS, FA>(a, sh, blockIdx.x, gridDim.x);
}

template <int LOSS, bool FA>
static void launch_lds_t(const CallArgs& a, int variant, int grid, hipStream_t st) {
  const dim3 g{unsigned(grid)}, t{1024};
  if (a.near) {
    hipLaunchKernelGGL((fused_small_lds_near_kernel<128, 1024, LOSS, FA>), g, t, 0, st, a);
  } else if (a.S > 1) {
    // the slice-spacing gradient needs the adjoint and its per-position partials
    if (FA && (a.want & WANT_LZ) && a.lz_part != nullptr)
      hipLaunchKernelGGL((fused_small_lds_ms_kernel<128, 1024, LOSS, FA, FA>), g, t, 0, st, a);
    else hipLaunchKernelGGL((fused_small_lds_ms_kernel<128, 1024, LOSS, false, FA>), g, t, 0, st, a);
  } else if (variant == 5) {
    hipLaunchKernelGGL((fused_small_lds_kernel<128, 1024, LOSS, false, FA>), g, t, 0, st, a);
  } else {
    hipLaunchKernelGGL((fused_small_lds_kernel<128, 1024, LOSS, true, FA>), g, t, 0, st, a);
  }
}

// 128^2 frames, bilinear patch (the plan checks)
hipError_t launch_fused_lds(const CallArgs& a, int variant, int grid, hipStream_t st) {
  const bool fa = a.mode == MODE_FWD_ADJ;
  if (a.loss == 0) fa ? launch_lds_t<0, true>(a, variant, grid, st) : launch_lds_t<0, false>(a, variant, grid, st);
  else fa ? launch_lds_t<1, true>(a, variant, grid, st) : launch_lds_t<1, false>(a, variant, grid, st);
  return hipGetLastError();
}

// per-workgroup scratch below the probe accumulator (float2 elements)
size_t lds_scratch_base(int S, int M, int recompute, int variant, bool near) {
  const size_t fr = size_t(128) * 128;
  if (near) return fr * (2 + size_t(M)) + fr / 2;
  if (S > 1) return fr * (size_t(2) * S + (recompute ? 0 : size_t(M) * S)) + fr / 2;
  return variant == 5 ? fr / 2 : 0;  // far fields always recomputed
}

}  // namespace ptyhip
