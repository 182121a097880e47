// Complex FFTs for ptychographic frames on gfx950.
//
// A length-N transform is split as N = N1 * N2 (N1 <= N2): with input index
// n = n1 + N1 n2 and output index k = k2 + N2 k1,
//   X[k2 + N2 k1] = sum_n1 W_N^{n1 k2} W_N1^{n1 k1} sum_n2 x[n1 + N1 n2] W_N2^{n2 k2},
// i.e. N1 register DFTs of size N2, a twiddle W_N^{n1 k2}, then N2 register DFTs of size
// N1. The two register stages exchange data through LDS. A 2D
// N x N transform runs that over the rows and then over the columns (4 register stages, 3 LDS
// exchanges). The inverse runs the adjoint stages in reverse order, so a forward
// transform leaves each thread holding exactly the frequencies its inverse needs,
// and the inverse returns every pixel to the thread that supplied it.
//
// All transforms here are unnormalised; callers apply 1/N per 2D transform
// (the unitary convention).
#pragma once
#include "common.hpp"

namespace ptyhip {

// ----------------------------------------------------------------------------- register DFTs
// Radix-4 butterflies of plain sums with one constant twiddle between them: a value meets few
// rounded constants on its way. (Radix-2 butterflies of six fused operations with the second
// stage's twiddles inside them carried log2 R rounded factors per value: relative error of a 2D
// transform of 128^2 1.39e-7 instead of 1.27e-7, and its gain error, which adds up over the
// transforms of a position, -6.2e-8 instead of -4.2e-8; 256^2 1.57e-7 and -8.1e-8 instead of
// 1.40e-7 and -5.3e-8. 6732 positions of 30 modes took 24.8 ms with them instead of 25.8, 331 forward
// positions of 256^2 504 us instead of 477.)

// multiply by the constant twiddle W_R^J, with the trivial angles special-cased
template <int R, int J, bool INV>
__device__ __forceinline__ float2 twiddle_const(float2 a) {
  constexpr int j = J % R;
  if constexpr (j == 0) {
    return a;
  } else if constexpr (4 * j == R) {
    return mul_mi<INV>(a);
  } else if constexpr (2 * j == R) {
    return make_float2(-a.x, -a.y);
  } else if constexpr (4 * j == 3 * R) {
    return mul_mi<!INV>(a);
  } else {
    return cmul(a, make_float2(Twiddle<R, J, INV>::re, Twiddle<R, J, INV>::im));
  }
}

template <int R, bool INV>
struct Dft;

template <bool INV>
struct Dft<1, INV> {
  __device__ __forceinline__ static void run(float2*) {}
};

template <bool INV>
struct Dft<2, INV> {
  __device__ __forceinline__ static void run(float2* v) {
    float2 a = v[0], b = v[1];
    v[0] = cadd(a, b);
    v[1] = csub(a, b);
  }
};

template <bool INV>
struct Dft<4, INV> {
  __device__ __forceinline__ static void run(float2* v) {
    float2 s02 = cadd(v[0], v[2]), d02 = csub(v[0], v[2]);
    float2 s13 = cadd(v[1], v[3]), d13 = mul_mi<INV>(csub(v[1], v[3]));
    v[0] = cadd(s02, s13);
    v[2] = csub(s02, s13);
    v[1] = cadd(d02, d13);
    v[3] = csub(d02, d13);
  }
};

// Cooley-Tukey split R = A * B with constant twiddles (register renaming only).
template <int A, int B, bool INV>
__device__ __forceinline__ void dft_split(float2* v) {
  constexpr int R = A * B;
  float2 t[R];
  static_for<0, A>([&](auto n1c) {
    constexpr int n1 = decltype(n1c)::value;
    float2 u[B];
#pragma unroll
    for (int n2 = 0; n2 < B; ++n2) u[n2] = v[n1 + A * n2];
    Dft<B, INV>::run(u);
    static_for<0, B>([&](auto k2c) {
      constexpr int k2 = decltype(k2c)::value;
      t[n1 * B + k2] = twiddle_const<R, n1 * k2, INV>(u[k2]);
    });
  });
#pragma unroll
  for (int k2 = 0; k2 < B; ++k2) {
    float2 u[A];
#pragma unroll
    for (int n1 = 0; n1 < A; ++n1) u[n1] = t[n1 * B + k2];
    Dft<A, INV>::run(u);
#pragma unroll
    for (int k1 = 0; k1 < A; ++k1) v[k2 + B * k1] = u[k1];
  }
}

template <bool INV>
struct Dft<8, INV> {
  __device__ __forceinline__ static void run(float2* v) { dft_split<2, 4, INV>(v); }
};
template <bool INV>
struct Dft<16, INV> {
  __device__ __forceinline__ static void run(float2* v) { dft_split<4, 4, INV>(v); }
};
template <bool INV>
struct Dft<32, INV> {
  __device__ __forceinline__ static void run(float2* v) { dft_split<4, 8, INV>(v); }
};

// DFT of size R of v[n] w^n with w = W_N^p (p < N / R), the second factor of a transform of
// size N: every element is multiplied by its own table entry w^n, one rounded twiddle.
// Table (load_twiddles): entry n of every p consecutive, so that the entries of a lane are at
// constant distances.
template <int R, int N, bool INV>
struct TwiddledDft {
  static constexpr int PITCH = N / R;
  const float2* c;
  __device__ __forceinline__ TwiddledDft(const float2* tab, int p) : c(tab + p) {}
  __device__ __forceinline__ void run(float2* v) const {
#pragma unroll
    for (int n = 1; n < R; ++n) v[n] = INV ? cmul_conjb(v[n], c[n * PITCH]) : cmul(v[n], c[n * PITCH]);
    Dft<R, INV>::run(v);
  }
};

// ----------------------------------------------------------------------------- factorisations
template <int N>
struct Split;
template <> struct Split<16>  { static constexpr int N1 = 4,  N2 = 4;  };
template <> struct Split<32>  { static constexpr int N1 = 4,  N2 = 8;  };
template <> struct Split<64>  { static constexpr int N1 = 8,  N2 = 8;  };
template <> struct Split<128> { static constexpr int N1 = 8,  N2 = 16; };
template <> struct Split<256> { static constexpr int N1 = 16, N2 = 16; };
template <> struct Split<512> { static constexpr int N1 = 16, N2 = 32; };

// The LDS tables of a transform of N points, N entries each from tw (W_N^j): W_N^{n p} at
// n N2 + p for a second stage of size N1, and at n N1 + p for one of size N2 (the inverse of Frame2D
// and LineTile).
template <int N>
__device__ __forceinline__ void load_twiddles(float2* tws, const float2* __restrict__ tw) {
  constexpr int N2 = Split<N>::N2;
  for (int i = threadIdx.x; i < N; i += blockDim.x) tws[i] = tw[(i / N2) * (i % N2)];
}
template <int N>
__device__ __forceinline__ void load_inverse_twiddles(float2* tws, const float2* __restrict__ tw) {
  constexpr int N1 = Split<N>::N1;
  for (int i = threadIdx.x; i < N; i += blockDim.x) tws[i] = tw[(i / N1) * (i % N1)];
}

// ----------------------------------------------------------------------------- on-chip 2D frame
// A whole N x N frame spread over T threads (N <= 128). Each thread owns E elements.
//
// Layout A (pixels): element v[l*N2 + j] of thread t is pixel (y, x) with slot
//   s = t + T l, y = s / N1, x = (s % N1) + N1 j.
// Layout D (frequencies): element v[l*N2 + jj*N1 + l1] of thread t is frequency
//   (ky, kx) with s = t + T l, kx = s % N, q = s / N, ky = (q + N1 jj) + N2 l1.
//
// LDS holds N rows of pitch P = N + N1 float2. Inside a row, the row-stage exchange
// stores element (n1, k2) at N1 k2 + (n1 ^ (k2 mod N1)) so that both the writes and
// the reads of that exchange touch distinct banks within each 16-lane group.
// `tw`: 2 N entries, load_twiddles' table and from N load_inverse_twiddles'.
template <int N, int T>
struct Frame2D {
  static_assert(WAVE % Split<N>::N1 == 0 && (T % WAVE == 0 || T == N * Split<N>::N1),
                "the N1 threads of a row must share a wavefront");
  static constexpr int N1 = Split<N>::N1;
  static constexpr int N2 = Split<N>::N2;
  static constexpr int SLOTS = N * N1;
  static_assert(SLOTS % T == 0, "thread count must divide N * N1");
  static constexpr int L = SLOTS / T;
  static constexpr int E = L * N2;
  static constexpr int P = N + N1;
  static constexpr int LDS_ELEMS = N * P;

  __device__ __forceinline__ static int a_y(int t, int l) { return (t + T * l) / N1; }
  __device__ __forceinline__ static int a_x(int t, int l, int j) { return (t + T * l) % N1 + N1 * j; }
  __device__ __forceinline__ static int d_kx(int t, int l) { return (t + T * l) % N; }
  // frequency row of element (l, i) with i = jj*N1 + l1 in layout D
  __device__ __forceinline__ static int d_ky(int t, int l, int i) {
    const int q = (t + T * l) / N;
    const int jj = i / N1, l1 = i % N1;
    return q + N1 * jj + N2 * l1;
  }
  __device__ __forceinline__ static int sw(int n1, int k2) { return N1 * k2 + (n1 ^ (k2 & (N1 - 1))); }

  // Exchange discipline (3 block barriers per transform): the row stages only touch
  // rows owned by the wave (the N1 threads of a row are adjacent lanes), and LDS
  // operations of one wave execute in program order, so their exchanges need only a
  // compiler fence; the first column stage writes back exactly the cells it read.
  __device__ __forceinline__ static void wave_fence() { __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront"); }

  // layout A (pixels) -> layout D (frequencies), times `scale`
  __device__ __forceinline__ static void forward(float2 (&v)[E], float2* lds, const float2* __restrict__ tw,
                                                 float scale) {
    const int t = opaque_tid();
    __syncthreads();
    // row stage 1: DFT over n2, exchange within the wave
#pragma unroll
    for (int l = 0; l < L; ++l) {
      const int s = t + T * l, y = s / N1, n1 = s % N1;
      float2* u = &v[l * N2];
      Dft<N2, false>::run(u);
#pragma unroll
      for (int k2 = 0; k2 < N2; ++k2) lds[y * P + sw(n1, k2)] = u[k2];
    }
    wave_fence();
    // row stage 2: DFT over n1 for the thread's k2 values
#pragma unroll
    for (int l = 0; l < L; ++l) {
      const int s = t + T * l, y = s / N1, q = s % N1;
#pragma unroll
      for (int jj = 0; jj < N2 / N1; ++jj) {
        const int k2 = q + N1 * jj;
        float2* u = &v[l * N2 + jj * N1];
#pragma unroll
        for (int n1 = 0; n1 < N1; ++n1) u[n1] = lds[y * P + sw(n1, k2)];
        TwiddledDft<N1, N, false>(tw, k2).run(u);
      }
    }
    wave_fence();
#pragma unroll
    for (int l = 0; l < L; ++l) {
      const int s = t + T * l, y = s / N1, q = s % N1;
#pragma unroll
      for (int jj = 0; jj < N2 / N1; ++jj)
#pragma unroll
        for (int k1 = 0; k1 < N1; ++k1) lds[y * P + q + N1 * jj + N2 * k1] = v[l * N2 + jj * N1 + k1];
    }
    __syncthreads();
    // column stage 1 (in place): thread owns column kx, residue m1; DFT over m2
#pragma unroll
    for (int l = 0; l < L; ++l) {
      const int s = t + T * l, kx = s % N, m1 = s / N;
      float2 u[N2];
#pragma unroll
      for (int m2 = 0; m2 < N2; ++m2) u[m2] = lds[(m1 + N1 * m2) * P + kx];
      Dft<N2, false>::run(u);
#pragma unroll
      for (int l2 = 0; l2 < N2; ++l2) lds[(m1 + N1 * l2) * P + kx] = u[l2];
    }
    __syncthreads();
    // column stage 2: DFT over m1
#pragma unroll
    for (int l = 0; l < L; ++l) {
      const int s = t + T * l, kx = s % N, q = s / N;
#pragma unroll
      for (int jj = 0; jj < N2 / N1; ++jj) {
        const int l2 = q + N1 * jj;
        float2* u = &v[l * N2 + jj * N1];
#pragma unroll
        for (int n1 = 0; n1 < N1; ++n1) u[n1] = lds[(n1 + N1 * l2) * P + kx];
        TwiddledDft<N1, N, false>(tw, l2).run(u);
#pragma unroll
        for (int l1 = 0; l1 < N1; ++l1) u[l1] = cscale(u[l1], scale);
      }
    }
  }

  // layout D (frequencies) -> layout A (pixels): the adjoint of `forward`, times `scale`
  __device__ __forceinline__ static void inverse(float2 (&v)[E], float2* lds, const float2* __restrict__ tw,
                                                 float scale) {
    const int t = opaque_tid();
#pragma unroll
    for (int l = 0; l < L; ++l)
#pragma unroll
      for (int jj = 0; jj < N2 / N1; ++jj) Dft<N1, true>::run(&v[l * N2 + jj * N1]);
    __syncthreads();
#pragma unroll
    for (int l = 0; l < L; ++l) {
      const int s = t + T * l, kx = s % N, q = s / N;
#pragma unroll
      for (int jj = 0; jj < N2 / N1; ++jj) {
        const int l2 = q + N1 * jj;
#pragma unroll
        for (int n1 = 0; n1 < N1; ++n1) lds[(n1 + N1 * l2) * P + kx] = v[l * N2 + jj * N1 + n1];
      }
    }
    __syncthreads();
    // column stage 1 adjoint (in place)
#pragma unroll
    for (int l = 0; l < L; ++l) {
      const int s = t + T * l, kx = s % N, m1 = s / N;
      float2 u[N2];
#pragma unroll
      for (int l2 = 0; l2 < N2; ++l2) u[l2] = lds[(m1 + N1 * l2) * P + kx];
      TwiddledDft<N2, N, true>(tw + N, m1).run(u);
#pragma unroll
      for (int m2 = 0; m2 < N2; ++m2) lds[(m1 + N1 * m2) * P + kx] = u[m2];
    }
    __syncthreads();
    // row stage 2 adjoint, exchange within the wave
#pragma unroll
    for (int l = 0; l < L; ++l) {
      const int s = t + T * l, y = s / N1, q = s % N1;
#pragma unroll
      for (int jj = 0; jj < N2 / N1; ++jj) {
        float2* u = &v[l * N2 + jj * N1];
#pragma unroll
        for (int k1 = 0; k1 < N1; ++k1) u[k1] = lds[y * P + q + N1 * jj + N2 * k1];
        Dft<N1, true>::run(u);
      }
    }
    wave_fence();
#pragma unroll
    for (int l = 0; l < L; ++l) {
      const int s = t + T * l, y = s / N1, q = s % N1;
#pragma unroll
      for (int jj = 0; jj < N2 / N1; ++jj) {
        const int k2 = q + N1 * jj;
#pragma unroll
        for (int n1 = 0; n1 < N1; ++n1) lds[y * P + sw(n1, k2)] = v[l * N2 + jj * N1 + n1];
      }
    }
    wave_fence();
    // row stage 1 adjoint
#pragma unroll
    for (int l = 0; l < L; ++l) {
      const int s = t + T * l, y = s / N1, n1 = s % N1;
      float2* u = &v[l * N2];
#pragma unroll
      for (int k2 = 0; k2 < N2; ++k2) u[k2] = lds[y * P + sw(n1, k2)];
      TwiddledDft<N2, N, true>(tw + N, n1).run(u);
#pragma unroll
      for (int n2 = 0; n2 < N2; ++n2) u[n2] = cscale(u[n2], scale);
    }
  }

  // Write a layout-A register frame to LDS in natural (y, x) order (pitch P).
  __device__ __forceinline__ static void store_natural(const float2 (&v)[E], float2* lds) {
    const int t = opaque_tid();
    __syncthreads();
#pragma unroll
    for (int l = 0; l < L; ++l)
#pragma unroll
      for (int j = 0; j < N2; ++j) lds[a_y(t, l) * P + a_x(t, l, j)] = v[l * N2 + j];
    __syncthreads();
  }
};

// ----------------------------------------------------------------------------- line tiles
// 1D transforms of NL lines of length N that live in LDS (for frames too large to
// stay on chip: 256 and 512). Element i of line ln is at lds[ln * LS + i * ES].
// Each line is served by N1 threads; T threads cover T / N1 lines per round.
template <int N, int NL, int T>
struct LineTile {
  static constexpr int N1 = Split<N>::N1;
  static constexpr int N2 = Split<N>::N2;
  static_assert(T % N1 == 0, "");
  static constexpr int LPR = T / N1;               // lines per round
  static_assert(NL % LPR == 0, "lines must fill whole rounds");
  static constexpr int ROUNDS = NL / LPR;
  // Position of the intermediate element (n1, k2) inside a line: N1 k2 + (n1 ^ (k2 mod
  // N1)). The XOR spreads the N1 lanes of a line over distinct LDS banks both where
  // stage 1 writes (fixed k2, lanes n1) and where stage 2 reads (fixed n1, lanes k2),
  // which in natural order would all hit one bank.
  __device__ __forceinline__ static int sw(int n1, int k2) { return N1 * k2 + (n1 ^ (k2 & (N1 - 1))); }

  // In-place transform of all NL lines. Caller syncs before (data in LDS) and after.
  template <bool INV>
  __device__ __forceinline__ static void run(float2* lds, int LS, int ES, const float2* __restrict__ tw_) {
    const int t = opaque_tid();
    const float2* __restrict__ tw = tw_;
    const int q = t % N1, lr = t / N1;
    if constexpr (!INV) {
      // stage 1 in place: x[n1 + N1 n2] -> Y[n1][k2] stored at sw(n1, k2)
#pragma unroll 1
      for (int r = 0; r < ROUNDS; ++r) {
        float2* base = lds + (lr + LPR * r) * LS;
        float2 u[N2];
#pragma unroll
        for (int n2 = 0; n2 < N2; ++n2) u[n2] = base[(q + N1 * n2) * ES];
        Dft<N2, false>::run(u);
#pragma unroll
        for (int k2 = 0; k2 < N2; ++k2) base[sw(q, k2) * ES] = u[k2];
      }
      __syncthreads();
      float2 w[ROUNDS][N2];
#pragma unroll
      for (int r = 0; r < ROUNDS; ++r) {
        float2* base = lds + (lr + LPR * r) * LS;
#pragma unroll
        for (int jj = 0; jj < N2 / N1; ++jj) {
          const int k2 = q + N1 * jj;
          float2* u = &w[r][jj * N1];
#pragma unroll
          for (int n1 = 0; n1 < N1; ++n1) u[n1] = base[sw(n1, k2) * ES];
          TwiddledDft<N1, N, false>(tw, k2).run(u);
        }
      }
      __syncthreads();
#pragma unroll
      for (int r = 0; r < ROUNDS; ++r) {
        float2* base = lds + (lr + LPR * r) * LS;
#pragma unroll
        for (int jj = 0; jj < N2 / N1; ++jj)
#pragma unroll
          for (int k1 = 0; k1 < N1; ++k1) base[(q + N1 * jj + N2 * k1) * ES] = w[r][jj * N1 + k1];
      }
    } else {
      float2 w[ROUNDS][N2];
#pragma unroll
      for (int r = 0; r < ROUNDS; ++r) {
        float2* base = lds + (lr + LPR * r) * LS;
#pragma unroll
        for (int jj = 0; jj < N2 / N1; ++jj) {
          float2* u = &w[r][jj * N1];
#pragma unroll
          for (int k1 = 0; k1 < N1; ++k1) u[k1] = base[(q + N1 * jj + N2 * k1) * ES];
          Dft<N1, true>::run(u);
        }
      }
      __syncthreads();
#pragma unroll
      for (int r = 0; r < ROUNDS; ++r) {
        float2* base = lds + (lr + LPR * r) * LS;
#pragma unroll
        for (int jj = 0; jj < N2 / N1; ++jj) {
          const int k2 = q + N1 * jj;
#pragma unroll
          for (int n1 = 0; n1 < N1; ++n1) base[sw(n1, k2) * ES] = w[r][jj * N1 + n1];
        }
      }
      __syncthreads();
#pragma unroll 1
      for (int r = 0; r < ROUNDS; ++r) {
        float2* base = lds + (lr + LPR * r) * LS;
        float2 u[N2];
#pragma unroll
        for (int k2 = 0; k2 < N2; ++k2) u[k2] = base[sw(q, k2) * ES];
        TwiddledDft<N2, N, true>(tw + N, q).run(u);
#pragma unroll
        for (int n2 = 0; n2 < N2; ++n2) base[(q + N1 * n2) * ES] = u[n2];
      }
    }
  }
};

// ----------------------------------------------------------------------------- wave lines
// 1D transforms of four lines of N = 16 N2 points by one wavefront (256 and 512 points),
// input and output in registers. Stage 1: thread (line, n1) holds x[n1 + 16 n2] in
// u[n2] and runs a register DFT of size N2; the wave exchanges through its own 4 N cells of
// LDS (no block barrier: a wave's LDS operations execute in order); stage 2: thread
// (line, kq) runs N2 / 16 twiddled DFTs of size 16 and holds frequency
// kq + 16 kk in v[kk]. The inverse runs the adjoint stages in reverse order.
// Cell of the intermediate (line, n1, k2): the XORs put the 32 lanes of a half-wave into
// distinct 8-byte banks in both stages, for lanes that are 16 consecutive n1 (or k2) of two
// lines, 8 of four lines (column order), or 4 + 4 of four lines (tile order).
template <int N>
struct WaveLines {
  static constexpr int N1 = 16, N2 = N / 16;
  static_assert(N2 == 16 || N2 == 32, "256- and 512-point lines");
  // table in LDS: W_N^{n1 k2} at k2 16 + n1. The twiddles are applied one by one at the
  // exchange, four at a time (a thread of a 256^2 frame has 128 registers and 32 pixels: eight or
  // more factors live through a stage make the loss of the forward kernel spill).
  __device__ __forceinline__ static void table(float2* tws, const float2* __restrict__ tw) {
    for (int i = threadIdx.x; i < N; i += blockDim.x) tws[i] = tw[(i & 15) * (i >> 4)];
  }
  __device__ __forceinline__ static int cell0(int line, int i) {  // XORed with (k2, n1 ^ k2) parts
    return line * N + 16 * (line & 1) + (i ^ ((line >> 1) << 3));
  }
  __device__ __forceinline__ static void wave_fence() { __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront"); }

  // `ex`: the wave's cells; `tw`: the table
  __device__ __forceinline__ static void forward(float2* ex, const float2* tw, int line1, int n1, int line2, int kq,
                                                 float2 (&u)[N2], float2 (&v)[N2]) {
    Dft<N2, false>::run(u);
    const int c1 = opaque(cell0(line1, n1));
    wave_fence();
#pragma unroll
    for (int k2 = 0; k2 < N2; ++k2) {
      if (k2 > 0) u[k2] = cmul(u[k2], tw[k2 * 16 + n1]);
      ex[c1 ^ (16 * k2 + (k2 & 15))] = u[k2];
      if (k2 % 4 == 3) __builtin_amdgcn_sched_barrier(0);
    }
    wave_fence();
#pragma unroll
    for (int jj = 0; jj < N2 / 16; ++jj) {
      const int c2 = opaque(cell0(line2, 0) ^ (16 * (kq + 16 * jj) + kq));
      float2 w[16];
#pragma unroll
      for (int i = 0; i < 16; ++i) w[i] = ex[c2 ^ i];
      Dft<16, false>::run(w);
#pragma unroll
      for (int k1 = 0; k1 < 16; ++k1) v[jj + (N2 / 16) * k1] = w[k1];
    }
    wave_fence();
  }
  __device__ __forceinline__ static void inverse(float2* ex, const float2* tw, int line2, int kq, int line1, int n1,
                                                 float2 (&v)[N2], float2 (&u)[N2]) {
    wave_fence();
#pragma unroll
    for (int jj = 0; jj < N2 / 16; ++jj) {
      const int c2 = opaque(cell0(line2, 0) ^ (16 * (kq + 16 * jj) + kq));
      float2 w[16];
#pragma unroll
      for (int k1 = 0; k1 < 16; ++k1) w[k1] = v[jj + (N2 / 16) * k1];
      Dft<16, true>::run(w);
#pragma unroll
      for (int i = 0; i < 16; ++i) ex[c2 ^ i] = w[i];
    }
    const int c1 = opaque(cell0(line1, n1));
    wave_fence();
#pragma unroll
    for (int k2 = 0; k2 < N2; ++k2) {
      u[k2] = ex[c1 ^ (16 * k2 + (k2 & 15))];
      if (k2 > 0) u[k2] = cmul_conjb(u[k2], tw[k2 * 16 + n1]);
      if (k2 % 4 == 3) __builtin_amdgcn_sched_barrier(0);
    }
    wave_fence();
    Dft<N2, true>::run(u);
  }
};

// ----------------------------------------------------------------------------- LDS-resident frame
// A whole N x N frame kept in LDS (natural order, pitch P = N + N1) and transformed in
// place by T = N * N1 threads, rows first, then columns. Each line is served by N1 lanes
// of one wavefront, so the two stages of a line exchange through LDS with only a
// compiler fence (a wave's LDS operations execute in order);
// a 2D transform needs a block barrier before the rows, between rows and columns, and
// after the columns. Registers hold one line stage at a time (N2 elements per thread),
// which leaves the rest of the register file to the caller's per-pixel state.
// Each line runs the same split as Frame2D: N1 register DFTs of size N2 over
// x[n1 + N1 n2], the twiddle W_N^{n1 k2}, then for each k2 a DFT of size N1 giving
// X[k2 + N2 k1]; the inverse is the same split with W_N^-1 (unnormalised). Stage-1
// results are stored at N1 k2 + (n1 XOR (k2 mod N1)), as in LineTile.
// Transforms are unnormalised (tws: load_twiddles' table). Cells are addressed by byte
// offsets: a row and a column pitch of 2^a + 2^b bytes make the XOR of the swizzle an XOR
// of offsets, one instruction per cell and none for its position.
template <int N, int T>
struct FrameLds {
  static constexpr int N1 = Split<N>::N1;
  static constexpr int N2 = Split<N>::N2;
  static_assert(T == N * N1, "one line per N1 threads");
  static_assert(WAVE % N1 == 0, "the N1 threads of a line must share a wavefront");
  static constexpr int LW = WAVE / N1;  // lines per wave in the column pass
  static constexpr int P = N + N1;
  static constexpr int PB = P * 8;      // row pitch in bytes
  static constexpr int LDS_ELEMS = N * P;
  static constexpr int EL = N * N / T;  // pixels per thread in the element passes
  static_assert((N & (N - 1)) == 0 && N1 == 8 && N >= 64, "offsets of rows 0..7 and cells 0..7 XOR like their numbers");
  __device__ __forceinline__ static void wave_fence() { __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront"); }
  __device__ __forceinline__ static float2& at(float2* lds, int off) {
    return *reinterpret_cast<float2*>(reinterpret_cast<char*>(lds) + off);
  }

  // Rows: line t / N1, lane q = t mod N1 (a half-wave reads four rows' consecutive cells);
  // columns: the lines of a wave are WAVE / N1 adjacent columns and lane
  // q = (t mod WAVE) / N1, so a half-wave reads WAVE / N1 consecutive cells in each of four
  // rows (with P = N + N1 both fall in distinct LDS banks).
  template <bool COLS>
  struct Line {
    int t, q, org;  // org: byte offset of the line's first cell
    __device__ __forceinline__ Line() {
      t = opaque_tid();
      q = COLS ? (t % WAVE) / LW : t % N1;
      org = COLS ? ((t / WAVE) * LW + t % LW) * 8 : (t / N1) * PB;
    }
    static constexpr int ES = COLS ? PB : 8;  // bytes from cell to cell of a line
    // cell q + N1 n2
    __device__ __forceinline__ int cell(int n2) const { return org + q * ES + n2 * N1 * ES; }
    // cell N1 k2 + (n1 XOR (k2 mod N1)) of the intermediate, for the lane's n1 = q ...
    __device__ __forceinline__ int mid1(int k2) const { return ((q * ES) ^ ((k2 % N1) * ES)) + org + k2 * N1 * ES; }
    // ... and for its k2 = q + N1 jj
    __device__ __forceinline__ int mid2(int n1, int jj) const {
      return ((q * ES) ^ (n1 * ES)) + (org + q * N1 * ES) + jj * N1 * N1 * ES;
    }
  };

  // Stage 1 and the exchange: u holds x[q + N1 n2] on entry and, as jj N1 + n1, the stage-2
  // inputs of k2 = q + N1 jj transformed to X[k2 + N2 k1] at jj N1 + k1 on return.
  template <bool INV, bool COLS>
  __device__ __forceinline__ static void line(const Line<COLS>& L, float2* lds, const float2* tws, float2 (&u)[N2]) {
    Dft<N2, INV>::run(u);
#pragma unroll
    for (int k2 = 0; k2 < N2; ++k2) at(lds, L.mid1(k2)) = u[k2];
    wave_fence();
#pragma unroll
    for (int jj = 0; jj < N2 / N1; ++jj) {
#pragma unroll
      for (int n1 = 0; n1 < N1; ++n1) u[jj * N1 + n1] = at(lds, L.mid2(n1, jj));
      TwiddledDft<N1, N, INV>(tws, L.q + N1 * jj).run(&u[jj * N1]);
    }
  }
  // every line of the frame transformed in place, its stage-1 input in u (`from`) or read
  // from the thread's cells
  template <bool INV, bool COLS>
  __device__ __forceinline__ static void lines_from(float2* lds, const float2* tws, float2 (&u)[N2]) {
    const Line<COLS> L;
    line<INV, COLS>(L, lds, tws, u);
    wave_fence();
    // X[q + N1 (jj + (N2 / N1) k1)] is cell jj + (N2 / N1) k1 of the thread
#pragma unroll
    for (int i = 0; i < N2; ++i) at(lds, L.cell(i)) = u[reg_of(i)];
  }
  template <bool COLS>
  __device__ __forceinline__ static void read_cells(float2* lds, float2 (&u)[N2]) {
    const Line<COLS> L;
#pragma unroll
    for (int n2 = 0; n2 < N2; ++n2) u[n2] = at(lds, L.cell(n2));
  }

  // Column and row of element e (0 <= e < N2) that cols_to_regs leaves in thread t:
  // column col(t), row row(t, e); these are the cells the thread's column pass reads and
  // writes, so a caller that writes exactly them needs no barrier before cols_from().
  __device__ __forceinline__ static int col(int t) { return (t / WAVE) * LW + t % LW; }
  __device__ __forceinline__ static int row(int t, int e) { return (t % WAVE) / LW + N1 * (e / N1) + N2 * (e % N1); }

  // The passes; the caller places the block barriers. A row pass reads and writes only the
  // rows of its wave, and thread t only the cells (t / N1, t mod N1 + N1 j), which it may
  // therefore fill or read itself without a barrier; a column pass touches only the
  // columns of its wave. Rows and columns need a barrier between them.
  template <bool INV>
  __device__ __forceinline__ static void rows(float2* lds, const float2* tws) {
    float2 u[N2];
    read_cells<false>(lds, u);
    lines_from<INV, false>(lds, tws, u);
  }
  // Row (column) pass whose stage-1 input is already in registers: u[n2] is the cell the
  // pass would read, (t / N1, t mod N1 + N1 n2) for rows, (row(t, e), col(t)) with
  // e = reg_of(n2) for columns (so that a caller holding the cols_to_regs layout passes
  // v[reg_of(n2)] as u[n2]).
  template <bool INV>
  __device__ __forceinline__ static void rows_from(float2* lds, const float2* tws, float2 (&u)[N2]) {
    lines_from<INV, false>(lds, tws, u);
  }
  template <bool INV>
  __device__ __forceinline__ static void cols_from(float2* lds, const float2* tws, float2 (&u)[N2]) {
    lines_from<INV, true>(lds, tws, u);
  }
  // Row pass that ends in registers: h[i] is cell (t / N1, t mod N1 + N1 i) of the
  // transformed rows; the LDS cells keep the stage-1 intermediate.
  template <bool INV>
  __device__ __forceinline__ static void rows_to_regs(float2* lds, const float2* tws, float2 (&h)[N2]) {
    const Line<false> L;
    float2 u[N2];
    read_cells<false>(lds, u);
    line<INV, false>(L, lds, tws, u);
#pragma unroll
    for (int i = 0; i < N2; ++i) h[i] = u[reg_of(i)];
  }
  // row(t, reg_of(n2)) = (t mod WAVE) / LW + N1 n2
  __host__ __device__ static constexpr int reg_of(int n2) { return (n2 % (N2 / N1)) * N1 + n2 / (N2 / N1); }

  // Forward column pass that ends in registers: v[e] is frequency (row(t, e), col(t));
  // the LDS cells keep the stage-1 intermediate.
  __device__ __forceinline__ static void cols_to_regs(float2* lds, const float2* tws, float2 (&v)[N2]) {
    const Line<true> L;
    read_cells<true>(lds, v);
    line<false, true>(L, lds, tws, v);
  }
};

}  // namespace ptyhip
