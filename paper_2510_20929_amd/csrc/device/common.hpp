// Device helpers shared by every ptyhip kernel: complex arithmetic on float2,
// compile-time loops and twiddles, atomics and block reductions (gfx950, wave64).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <type_traits>

namespace ptyhip {

constexpr int WAVE = 64;

// ----------------------------------------------------------------------------- complex
__device__ __forceinline__ float2 cadd(float2 a, float2 b) { return make_float2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ float2 csub(float2 a, float2 b) { return make_float2(a.x - b.x, a.y - b.y); }
__device__ __forceinline__ float2 cscale(float2 a, float s) { return make_float2(a.x * s, a.y * s); }
__device__ __forceinline__ float2 cmul(float2 a, float2 b) {
  return make_float2(fmaf(a.x, b.x, -a.y * b.y), fmaf(a.x, b.y, a.y * b.x));
}
// conj(a) * b
__device__ __forceinline__ float2 cmulc(float2 a, float2 b) {
  return make_float2(fmaf(a.x, b.x, a.y * b.y), fmaf(a.x, b.y, -a.y * b.x));
}
// a * conj(b)
__device__ __forceinline__ float2 cmul_conjb(float2 a, float2 b) {
  return make_float2(fmaf(a.x, b.x, a.y * b.y), fmaf(a.y, b.x, -a.x * b.y));
}
__device__ __forceinline__ float cabs2(float2 a) { return fmaf(a.x, a.x, a.y * a.y); }
// Re(conj(a) * b)
__device__ __forceinline__ float cdotre(float2 a, float2 b) { return fmaf(a.x, b.x, a.y * b.y); }
// multiply by -i (forward) or +i (inverse)
template <bool INV>
__device__ __forceinline__ float2 mul_mi(float2 a) {
  if constexpr (INV) return make_float2(-a.y, a.x);
  else return make_float2(a.y, -a.x);
}

// ----------------------------------------------------------------------------- buffer-resource frames
// A workgroup-private frame of complex values addressed through a buffer resource:
// element (i, t) of a [E][T] layout is at byte t*8 (one VGPR per thread) plus i*T*8 (a
// scalar offset), so unrolled loops over i need no per-element 64-bit addresses.
typedef float f2v_t __attribute__((ext_vector_type(2)));
constexpr int BUF_RSRC_WORD3 = 0x00020000;  // raw buffer, 32-bit data format (gfx9 family)

struct BufFrame {
  __amdgpu_buffer_rsrc_t r;
  __device__ __forceinline__ BufFrame(const void* base, uint32_t bytes)
      : r(__builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, int(bytes), BUF_RSRC_WORD3)) {}
  __device__ __forceinline__ float2 ld(int voff, int soff) const {
    const f2v_t v = __builtin_bit_cast(f2v_t, __builtin_amdgcn_raw_buffer_load_b64(r, voff, soff, 0));
    return make_float2(v.x, v.y);
  }
  __device__ __forceinline__ void st(float2 x, int voff, int soff) const {
    const f2v_t v = {x.x, x.y};
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(decltype(__builtin_amdgcn_raw_buffer_load_b64(r, 0, 0, 0)), v),
                                          r, voff, soff, 0);
  }
  // two neighbouring complex values (any 4-byte alignment)
  __device__ __forceinline__ float4 ld2(int voff, int soff) const {
    return __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(r, voff, soff, 0));
  }
  __device__ __forceinline__ void st2(float4 x, int voff, int soff) const {
    __builtin_amdgcn_raw_buffer_store_b128(
        __builtin_bit_cast(decltype(__builtin_amdgcn_raw_buffer_load_b128(r, 0, 0, 0)), x), r, voff, soff, 0);
  }
  __device__ __forceinline__ float ldf(int voff, int soff) const {
    return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, voff, soff, 0));
  }
  __device__ __forceinline__ void stf(float x, int voff, int soff) const {
    __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, x), r, voff, soff, 0);
  }
};

// two neighbouring complex values of a 16-byte access
__device__ __forceinline__ float2 lo2(float4 v) { return make_float2(v.x, v.y); }
__device__ __forceinline__ float2 hi2(float4 v) { return make_float2(v.z, v.w); }
__device__ __forceinline__ float4 cat2(float2 a, float2 b) { return make_float4(a.x, a.y, b.x, b.y); }

// ----------------------------------------------------------------------------- optimisation barriers
// An empty asm statement that makes a value opaque to the optimiser, so that values
// derived from it inside a loop body are recomputed there instead of being hoisted
// out of the loop and kept live (which would exhaust the register file).
__device__ __forceinline__ int opaque(int x) {
  asm volatile("" : "+v"(x));
  return x;
}
__device__ __forceinline__ int opaque_scalar(int x) {  // the same for a value in a scalar register
  asm volatile("" : "+s"(x));
  return x;
}
// Computes a value here: without it the arithmetic may be sunk past following branches to
// its first use, which keeps all of its operands live instead.
__device__ __forceinline__ void pin(float2& x) { asm volatile("" : "+v"(x.x), "+v"(x.y)); }
__device__ __forceinline__ int opaque_tid() { return opaque(int(threadIdx.x)); }

// ----------------------------------------------------------------------------- compile-time loops
template <int I, int END, typename F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (I < END) {
    f(std::integral_constant<int, I>{});
    static_for<I + 1, END>(f);
  }
}

// ----------------------------------------------------------------------------- compile-time trig
// Taylor series on [-pi, pi] in double precision; only used to build constant twiddles
// of the small register DFTs, whose angles are 2 pi j / R with R <= 32.
constexpr double kPi = 3.14159265358979323846264338327950288;
constexpr double ct_reduce(double x) {
  while (x > kPi) x -= 2.0 * kPi;
  while (x < -kPi) x += 2.0 * kPi;
  return x;
}
constexpr double ct_sin(double x) {
  x = ct_reduce(x);
  double term = x, sum = x;
  for (int n = 1; n < 30; ++n) {
    term *= -x * x / ((2.0 * n) * (2.0 * n + 1.0));
    sum += term;
  }
  return sum;
}
constexpr double ct_cos(double x) {
  x = ct_reduce(x);
  double term = 1.0, sum = 1.0;
  for (int n = 1; n < 30; ++n) {
    term *= -x * x / ((2.0 * n - 1.0) * (2.0 * n));
    sum += term;
  }
  return sum;
}
// exp(-+ 2 pi i j / R): forward sign for INV == false
template <int R, int J, bool INV>
struct Twiddle {
  static constexpr double ang = 2.0 * kPi * double(J % R) / double(R);
  static constexpr float re = float(ct_cos(ang));
  static constexpr float im = INV ? float(ct_sin(ang)) : float(-ct_sin(ang));
};

// ----------------------------------------------------------------------------- atomics
// Hardware float add at device scope (the buffers are ordinary device allocations).
__device__ __forceinline__ void atomic_add_f32(float* p, float v) {
  __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void atomic_add_c(float2* p, float2 v) {
  float* f = reinterpret_cast<float*>(p);
  atomic_add_f32(f, v.x);
  atomic_add_f32(f + 1, v.y);
}

// Workgroups go to the 8 XCDs in turn, each with its own L2. The place of workgroup `wg` of
// `nwg` in an order that takes one XCD's workgroups after another's: persistent kernels
// hand out consecutive work items by it, so that neighbouring scan positions, whose windows
// overlap, share an L2. (Only the order depends on the distribution, no result does.)
__device__ __forceinline__ int xcd_rank(int wg, int nwg) {
  const int s = wg & 7, q = nwg >> 3, rem = nwg & 7;
  return s * q + min(s, rem) + (wg >> 3);
}

// ----------------------------------------------------------------------------- reductions
__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
  for (int o = WAVE / 2; o > 0; o >>= 1) v += __shfl_xor(v, o, WAVE);
  return v;
}

// Sum of one double per thread over the block; `red` holds T/64 doubles of LDS.
// Every thread receives the total.
template <int T>
__device__ __forceinline__ double block_sum(double v, double* red) {
  constexpr int NW = T / WAVE;
  v = wave_sum(v);
  const int lane = threadIdx.x & (WAVE - 1), w = threadIdx.x / WAVE;
  __syncthreads();
  if (lane == 0) red[w] = v;
  __syncthreads();
  double t = 0.0;
#pragma unroll
  for (int i = 0; i < NW; ++i) t += red[i];
  return t;
}

// Several sums at once (NV values per thread); red holds NV * T/64 doubles.
template <int T, int NV>
__device__ __forceinline__ void block_sum_n(double (&v)[NV], double* red) {
  constexpr int NW = T / WAVE;
  const int lane = threadIdx.x & (WAVE - 1), w = threadIdx.x / WAVE;
#pragma unroll
  for (int i = 0; i < NV; ++i) v[i] = wave_sum(v[i]);
  __syncthreads();
  if (lane == 0) {
#pragma unroll
    for (int i = 0; i < NV; ++i) red[i * NW + w] = v[i];
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < NV; ++i) {
    double t = 0.0;
#pragma unroll
    for (int j = 0; j < NW; ++j) t += red[i * NW + j];
    v[i] = t;
  }
}

// Error latch bits (mirrors the public header)
constexpr uint32_t FLAG_BOUNDS = 1u;
constexpr uint32_t FLAG_NONFINITE = 2u;

__device__ __forceinline__ void latch(uint32_t* flags, uint32_t bit) {
  __hip_atomic_fetch_or(flags, bit, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

}  // namespace ptyhip
