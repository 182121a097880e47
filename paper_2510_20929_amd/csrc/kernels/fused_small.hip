// Dispatch of the fused kernels of on-chip frames (N <= 128), and those of 16^2 and 32^2
// frames.
#include "fused_small.hpp"

namespace ptyhip {

// variants: 0 = 512 threads, scratch-resident patch (64^2: as 2); 1 = 1024 (128^2) or 256 (64^2)
// threads, scratch-resident patch; 2 = 512 threads, register-resident patch;
// 3 = 1024 (128^2) or 256 (64^2) threads, register-resident patch and patch gradient;
// 4 = as 3 with the patch gradient in scratch; 5, 6 (128^2 only) = 1024 threads, the
// working frame resident in LDS, patch and running patch gradient in registers, dl/dI
// in scratch (5) or in registers (6); with several slices both run the LDS-resident
// multislice kernel (dl/dI in scratch). The near field of 128^2 frames has one layout, the
// LDS-resident one, whatever the variant.
int fused_small_threads(int N, int variant, bool near) {
  const bool wide = variant == 1 || variant == 3 || variant == 4 || (N == 128 && (variant >= 5 || near));
  switch (N) {
    case 16: return 64;
    case 32: return 128;
    case 64: return wide ? 256 : 512;
    case 128: return wide ? 1024 : 512;
    default: return 0;
  }
}

// per-workgroup scratch (float2 elements) and the offset of the probe accumulator
size_t fused_small_scratch_elems(int N, int S, int M, int E, int recompute, size_t* pacc_off, int variant,
                                 bool near, bool fshift) {
  const size_t fr = size_t(N) * N;
  size_t base;
  if (N == 128 && (variant >= 5 || near)) base = lds_scratch_base(S, M, recompute, variant, near);
  else if (S > 1) base = fr * (size_t(2) * S + (recompute ? 0 : size_t(M) * S));
  else if (near) base = fr * (2 + size_t(M));
  else if (fshift) base = fr * (M > 1 ? (recompute ? 2 : size_t(M) + 1) : 1) + fr;  // + shifted window spectrum
  else if ((variant == 2 || variant == 3) && N >= 64) base = fr / 2 + (recompute ? 0 : fr * size_t(M - 1));
  else if (variant == 4 && N >= 64) base = fr / 2 + fr + (recompute ? 0 : fr * size_t(M - 1));
  else base = fr * (M > 1 ? (recompute ? 2 : size_t(M) + 1) : 1);
  *pacc_off = base;
  return base + fr * size_t(E) * M;
}

hipError_t launch_fused_small(const CallArgs& a, int N, int variant, int grid, hipStream_t st) {
  if (a.fshift) return launch_fused_small_fs(a, N, fused_small_threads(N, variant), grid, st);
  switch (N) {
    case 16: return launch_small_t<16, 64>(a, grid, st);
    case 32: return launch_small_t<32, 128>(a, grid, st);
    case 64: return launch_fused_small64(a, variant, grid, st);
    case 128:
      if (variant >= 5 || a.near) return launch_fused_lds(a, variant, grid, st);
      return launch_fused_small128(a, variant, grid, st);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_probe_reduce_small(const CallArgs& a, int N, int variant, int grid, float2* g_probe,
                                     int accumulate, hipStream_t st) {
  switch (N) {
    case 16: return probe_reduce_t<16, 64>(a, grid, g_probe, accumulate, st);
    case 32: return probe_reduce_t<32, 128>(a, grid, g_probe, accumulate, st);
    case 64: return launch_probe_reduce64(a, fused_small_threads(64, variant), grid, g_probe, accumulate, st);
    case 128: return launch_probe_reduce128(a, variant, grid, g_probe, accumulate, st);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace ptyhip
