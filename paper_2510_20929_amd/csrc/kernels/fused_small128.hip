// Register-resident fused kernels of 128^2 frames (variants 0 to 4), compiled by themselves: beside
// those of 16^2 and 32^2 frames the compiler spills 76 registers of variant 0 instead of none, 67 instead
// of 20 of variant 1 and 61 instead of 24 of variant 4 (a call of 100 forward positions: 50 us beside
// them, 43 by themselves; 1000 positions of 2 modes, forward and adjoint: 661 and 640).
#include "fused_small.hpp"

namespace ptyhip {

hipError_t launch_fused_small128(const CallArgs& a, int variant, int grid, hipStream_t st) {
  if (variant == 1) return launch_small_t<128, 1024>(a, grid, st);
  if (variant == 3) return launch_small_t<128, 1024, true>(a, grid, st);
  if (variant == 4) return launch_small_t<128, 1024, true, false>(a, grid, st);
  if (variant == 2) return launch_small_t<128, 512, true>(a, grid, st);
  return launch_small_t<128, 512>(a, grid, st);
}

hipError_t launch_probe_reduce128(const CallArgs& a, int variant, int grid, float2* g_probe, int accumulate,
                                  hipStream_t st) {
  if (variant >= 5 || a.near) return probe_reduce_t<128, 1024, true>(a, grid, g_probe, accumulate, st);
  return fused_small_threads(128, variant) == 1024 ? probe_reduce_t<128, 1024>(a, grid, g_probe, accumulate, st)
                                                   : probe_reduce_t<128, 512>(a, grid, g_probe, accumulate, st);
}

}  // namespace ptyhip
