// Multislice fused forward + adjoint with the working frame resident in LDS (128^2 frames,
// 1024 threads; tune variants 5 and 6 of a plan with several slices).
//
// Each slice-to-slice step is a forward transform, the Fresnel transfer function and an
// inverse transform. As in lds_body.hpp, the spatial state of a pixel lives with the
// thread whose row pass reads its cell, (t / 8, t mod 8 + 8 i), and the frequency state
// in the layout the column pass leaves in registers; a row pass is fed from registers
// and the inverse row pass ends in registers, so a propagation costs two block barriers
// (rows to columns, columns to rows) and no element pass through LDS. Patches, stored
// incident waves (slices s > 0; slice 0's is the probe) and, with several modes, the patch
// gradients of every slice stay in the workgroup's scratch as pairs (elements 2 j and
// 2 j + 1 of thread t at (j T + t) 16 bytes), dl/dI in the scratch's last half frame before
// the probe-gradient accumulator (column layout: element e of thread t at e T + t). That scratch
// traffic bounds the kernel (23 GB at 4.0 TB/s, VALU busy 43%), so a frame is touched as rarely
// as its order allows: the first mode writes a slice's patch gradient without reading it, the
// last mode adds its own and goes straight to the window, and the last mode's far field is
// scaled in the registers that hold it after the forward pass. The transforms are unnormalised; 1/N^2 (a power of two) is applied with
// the transfer function and with dl/dI. Measured at 1500 positions of 2 modes and 8 slices:
// 5.64 ms, 8.03 ms with every mode reading and writing every slice's gradient and 8-byte
// accesses.
// FA: a forward + adjoint call (a.mode). LZ: also dL/d(lambda z) of the slice spacing, from F g_psi_s and F psi_s for s > 0.
#pragma once
#include "lds_body.hpp"

namespace ptyhip {

// Probe side of one mode: the gradient v (R) of its incident probe wave into the staging
// frame or the accumulator frames ([E][M] from byte pacc_b of `sb`; `fresh`: written, not
// read), and the weight terms Re<v, U_e,m> (`pb`: the probe).
template <int N, int T>
__device__ __forceinline__ void lds_probe_side(const CallArgs& a, int k, int m, const float* wk,
                                               const float2 (&v)[FrameLds<N, T>::EL], const BufFrame& pb,
                                               const BufFrame& sb, int pacc_b, bool fresh, double* wacc) {
  constexpr int EL = FrameLds<N, T>::EL, N1 = FrameLds<N, T>::N1, NN = N * N;
  const int t = opaque_tid();
  const int vp = ((t / N1) * N + t % N1) * 8;
  if ((a.want & WANT_PROBE) && a.gpstage) {
    const BufFrame st(a.gpstage + (size_t(k) * a.M + m) * NN, NN * 8);
#pragma unroll
    for (int i = 0; i < EL; ++i) st.st(v[i], vp + 8 * N1 * i, 0);
  } else if (a.want & WANT_PROBE) {
    const int ne = wk ? a.E : 1;
    for (int e = 0; e < ne; ++e) {
      const int fb = pacc_b + (e * a.M + m) * NN * 8;
      const float w = wk ? wk[e] : 1.f;
#pragma unroll
      for (int i0 = 0; i0 < EL; i0 += 4) {
        float2 acc[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) acc[u] = make_float2(0.f, 0.f);
        if (!fresh) {
#pragma unroll
          for (int u = 0; u < 4; ++u) acc[u] = sb.ld(vp + 8 * N1 * (i0 + u), fb);
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          acc[u].x = fmaf(w, v[i0 + u].x, acc[u].x);
          acc[u].y = fmaf(w, v[i0 + u].y, acc[u].y);
          sb.st(acc[u], vp + 8 * N1 * (i0 + u), fb);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  }
  if ((a.want & WANT_WEIGHTS) && wk != nullptr) {
    for (int e = 0; e < a.E; ++e) {
      float sf = 0.f;
#pragma unroll
      for (int i = 0; i < EL; ++i) sf += cdotre(v[i], pb.ld(vp + 8 * N1 * i, (e * a.M + m) * NN * 8));
      const double sw = wave_sum(double(sf));
      if ((threadIdx.x & (WAVE - 1)) == 0) wacc[e * (T / WAVE) + threadIdx.x / WAVE] += sw;
    }
  }
}

template <int N, int T, int LOSS, bool LZ, bool FA>
__device__ __forceinline__ void lds_ms_body(const CallArgs& a, LdsShared<N, T>& sh, int wg, int nwg) {
  using F = FrameLds<N, T>;
  constexpr int EL = F::EL;
  constexpr int NN = N * N;
  constexpr int P = F::P;
  constexpr int N1 = F::N1;
  constexpr size_t FR = size_t(EL) * T;  // one frame in scratch
  float2* lds = sh.lds;
  float2* tws = sh.tws;
  double* red = sh.red;
  float* wsh = sh.wsh;
  double* wacc = sh.wacc;
  const int tid = threadIdx.x;
  const int S = a.S;
  const float inv_n = 1.f / float(N), inv_nn = inv_n * inv_n;
  const bool fwd = FA || a.mode != MODE_APPLY_AH;
  constexpr bool fa = FA;
  const bool adj = fa || !fwd;
  const bool recompute = a.recompute || !fwd;
  const bool want_pos = (a.want & WANT_POS) && fa;
  const bool want_probe = (a.want & WANT_PROBE) != 0;
  load_twiddles<N>(tws, a.tw);
  float2* scr = a.scratch + size_t(wg) * a.scratch_stride;
  constexpr int FB = int(FR * sizeof(float2));  // bytes of a frame: S patches, S patch gradients, M S waves
  const auto op_b = [&](int s) { return s * FB; };
  const auto gp_b = [&](int s) { return (S + s) * FB; };
  const auto ps_b = [&](int m, int s) { return (2 * S + m * S + s) * FB; };
  const BufFrame sb(scr, uint32_t(a.scratch_stride * sizeof(float2)));
  const int pacc_b = int(a.pacc_off * sizeof(float2));
  const int cf_b = pacc_b - NN * 4;  // dl/dI, NN floats just below the accumulator
  const size_t HW = size_t(a.H) * a.W;
  // (the accumulator is written, not read, by the first finished position, as in lds_body)
  const bool acc_lazy = adj && a.zero_acc && want_probe && !a.gpstage && (a.weights || a.E == 1);
  if (adj && a.zero_acc && want_probe && !a.gpstage && !acc_lazy) zero_probe_acc<N, T>(a, scr + a.pacc_off);
  bool acc_fresh = acc_lazy;
  auto cell = [](int t, int i) { return (t / N1) * P + t % N1 + N1 * i; };
  auto vpix = [](int t) { return ((t / N1) * N + t % N1) * 8; };
  auto fpix = [](int t, int e) { return F::row(t, e) * N + F::col(t); };
  const BufFrame pb(a.probe, uint32_t(size_t(a.E) * a.M * NN * sizeof(float2)));
  const BufFrame tfb(a.tf, NN * 8);
  // four pairs' loads are issued at a time
  const auto chunk = [](int j) {
    if (j % 4 == 3) __builtin_amdgcn_sched_barrier(0);
  };
  const auto store_frame = [&](int fb, const float2 (&x)[EL]) {
    const int t16 = opaque_tid() * 16;
#pragma unroll
    for (int j = 0; j < EL / 2; ++j) sb.st2(cat2(x[2 * j], x[2 * j + 1]), t16, fb + j * T * 16);
  };
  const auto load_frame = [&](int fb, float2 (&x)[EL]) {
    const int t16 = opaque_tid() * 16;
#pragma unroll
    for (int j = 0; j < EL / 2; ++j) {
      const float4 q = sb.ld2(t16, fb + j * T * 16);
      x[2 * j] = lo2(q);
      x[2 * j + 1] = hi2(q);
    }
  };
  // x *= frame (or its conjugate)
  const auto mul_frame = [&](int fb, float2 (&x)[EL], auto conj) {
    const int t16 = opaque_tid() * 16;
#pragma unroll
    for (int j = 0; j < EL / 2; ++j) {
      const float4 q = sb.ld2(t16, fb + j * T * 16);
      x[2 * j] = decltype(conj)::value ? cmulc(lo2(q), x[2 * j]) : cmul(x[2 * j], lo2(q));
      x[2 * j + 1] = decltype(conj)::value ? cmulc(hi2(q), x[2 * j + 1]) : cmul(x[2 * j + 1], hi2(q));
      chunk(j);
    }
  };
  using Plain = std::false_type;
  using Conj = std::true_type;

  // spatial (R) -> frequency (C2, registers); ends in the column phase
  auto fwd_t = [&](float2 (&x)[EL], float2 (&X)[EL]) {
    F::template rows_from<false>(lds, tws, x);
    __syncthreads();
    F::cols_to_regs(lds, tws, X);
  };
  // frequency (C2) -> spatial (R); starts in the column phase
  auto inv_t = [&](const float2 (&X)[EL], float2 (&x)[EL]) {
    float2 u[EL];
#pragma unroll
    for (int n2 = 0; n2 < EL; ++n2) u[n2] = X[F::reg_of(n2)];
    F::template cols_from<true>(lds, tws, u);
    __syncthreads();
    F::template rows_to_regs<true>(lds, tws, x);
  };
  // X *= H / N^2 (or conj(H) / N^2), the slice transfer function at the thread's frequencies
  auto apply_tf = [&](float2 (&X)[EL], auto conj) {
    const int t = opaque_tid();
    const int vf = fpix(t, 0) * 8;
#pragma unroll
    for (int e = 0; e < EL; ++e) {
      const float2 h = cscale(tfb.ld(vf, (N1 * (e / N1) + F::N2 * (e % N1)) * N * 8), inv_nn);
      X[e] = decltype(conj)::value ? cmulc(h, X[e]) : cmul(h, X[e]);
      chunk(e);
    }
  };
  auto probe_r = [&](const float* wk, int m, float2 (&v)[EL]) {
    const int vp = vpix(opaque_tid());
    if (wk == nullptr) {
#pragma unroll
      for (int i = 0; i < EL; ++i) v[i] = pb.ld(vp + 8 * N1 * i, m * NN * 8);
      return;
    }
#pragma unroll
    for (int i = 0; i < EL; ++i) v[i] = make_float2(0.f, 0.f);
    for (int e = 0; e < a.E; ++e) {
#pragma unroll
      for (int i = 0; i < EL; ++i) {
        const float2 u = pb.ld(vp + 8 * N1 * i, (e * a.M + m) * NN * 8);
        v[i].x = fmaf(wk[e], u.x, v[i].x);
        v[i].y = fmaf(wk[e], u.y, v[i].y);
        chunk(i);
      }
    }
  };
  // incident wave of mode m at slice s (R), from the probe; leaves the row phase
  auto incident = [&](float2 (&v)[EL], int m, int s, const float* wk) {
    probe_r(wk, m, v);
    for (int u = 0; u < s; ++u) {
      float2 X[EL];
      mul_frame(op_b(u), v, Plain{});
      fwd_t(v, X);
      apply_tf(X, Plain{});
      inv_t(X, v);
    }
  };
  // the same, stored or recomputed
  auto wave_at = [&](float2 (&v)[EL], int m, int s, const float* wk) {
    if (s == 0) probe_r(wk, m, v);
    else if (!recompute) load_frame(ps_b(m, s), v);
    else incident(v, m, s, wk);
  };

  for (int it = xcd_rank(wg, nwg); it < a.K; it += nwg) {
    const int k = opaque_scalar(it);
    const PosInfo p = wave_position(a.pos, k, N, a.H, a.W, want_pos);
    if (!p.ok) {
      skip_position<N, T>(a, k, p);
      if (LZ && tid == 0) a.lz_part[k] = 0.0;
      continue;
    }
    __syncthreads();
    if (a.weights && tid < a.E) wsh[tid] = a.weights[size_t(k) * a.E + tid];
    for (int i = tid; i < MAX_EIG * (T / WAVE); i += T) wacc[i] = 0.0;
    __syncthreads();
    const float* wk = a.weights ? wsh : nullptr;
    double lz = 0.0;

    for (int s = 0; s < S; ++s) {
      const PatchWindow pw(a.obj + size_t(s) * HW, a.W, N, p);
      const int t = opaque_tid();
      const int vo = ((t / N1) * a.W + t % N1) * 8;
#pragma unroll
      for (int j = 0; j < EL / 2; ++j) {
        sb.st2(cat2(pw.at(vo + 16 * N1 * j), pw.at(vo + 16 * N1 * j + 8 * N1)), t * 16, op_b(s) + j * T * 16);
        if (j % 2 == 1) __builtin_amdgcn_sched_barrier(0);
      }
    }

    float2 v[EL];
    if (fwd) {
      float2 X[EL];
      float cf[EL];
#pragma unroll
      for (int e = 0; e < EL; ++e) cf[e] = 0.f;
      for (int m = 0; m < a.M; ++m) {
        if (m > 0) __syncthreads();  // column phase done before the next mode's row pass
        probe_r(wk, m, v);
        for (int s = 0; s < S; ++s) {
          if (!recompute && fa && s > 0) store_frame(ps_b(m, s), v);
          mul_frame(op_b(s), v, Plain{});
          fwd_t(v, X);
          if (s < S - 1) {
            apply_tf(X, Plain{});
            inv_t(X, v);
          }
        }
        const int t = opaque_tid();
#pragma unroll
        for (int e = 0; e < EL; ++e) {
          cf[e] += cabs2(X[e]);
          if (!FA && a.mode == MODE_APPLY_A) a.psi_out[(size_t(k) * a.M + m) * NN + fpix(t, e)] = cscale(X[e], inv_n);
        }
      }
      if (!FA && a.mode == MODE_APPLY_A) continue;
      // loss and dl/dI (detector DC-centred)
      {
        const int t = opaque_tid();
        const float* im = a.imeas + size_t(k) * NN;
        float imv[EL];
#pragma unroll
        for (int e = 0; e < EL; ++e) imv[e] = __builtin_nontemporal_load(im + centred_index(F::row(t, e), F::col(t), N));
#pragma unroll
        for (int e = 0; e < EL; ++e) cf[e] *= inv_nn;
        if (a.ipred) {
          float* ip = a.ipred + size_t(k) * NN;
#pragma unroll
          for (int e = 0; e < EL; ++e) __builtin_nontemporal_store(cf[e], ip + centred_index(F::row(t, e), F::col(t), N));
        }
        double lsum = 0.0;
#pragma unroll
        for (int e = 0; e < EL; ++e) {
          float l, c;
          loss_terms<LOSS>(cf[e], imv[e], a.eps, l, c);
          lsum += double(l);
          cf[e] = a.gscale * inv_nn * c;
          chunk(e);
        }
        const double tot = block_sum<T>(lsum, red);
        const bool fin = isfinite(tot);
        if (tid == 0) {
          a.loss_part[k] = fin ? tot * double(a.lscale) : 0.0;
          if (!fin) {
            latch(a.flags, FLAG_NONFINITE);
            if (a.pos_part) {
              a.pos_part[2 * k] = 0.0;
              a.pos_part[2 * k + 1] = 0.0;
            }
            if (a.wvalid) a.wvalid[k] = 0;
            if (LZ) a.lz_part[k] = 0.0;
          }
        }
        if (!fin) {
          if (a.w_part && tid < a.E) a.w_part[size_t(k) * a.E + tid] = 0.0;
          continue;
        }
        if (fwd && !FA) continue;
#pragma unroll
        for (int e = 0; e < EL; ++e) {
          X[e] = cscale(X[e], cf[e]);  // the last mode's, which the adjoint starts with
          if (a.M > 1) sb.stf(cf[e], t * 4, cf_b + e * T * 4);
        }
      }
      inv_t(X, v);
    }

    double gy = 0.0, gx = 0.0;
    for (int mm = 0; mm < a.M; ++mm) {
      const int m = fa ? (mm == 0 ? a.M - 1 : mm - 1) : mm;
      const bool first = mm == 0, last = mm == a.M - 1;
      // the scaled far field of mode m (C2), then back to slice S-1's exit wave gradient
      if (!fwd) {
        float2 X[EL];
        const int t = opaque_tid();
        const float2* y = a.Y + (size_t(k) * a.M + m) * NN;
#pragma unroll
        for (int e = 0; e < EL; ++e) X[e] = cscale(y[fpix(t, e)], inv_n);
        __syncthreads();  // after the previous mode's row phase
        inv_t(X, v);
      } else if (!first) {
        float2 X[EL];
        wave_at(v, m, S - 1, wk);
        mul_frame(op_b(S - 1), v, Plain{});
        fwd_t(v, X);
        const int t = opaque_tid();
#pragma unroll
        for (int e = 0; e < EL; ++e) X[e] = cscale(X[e], sb.ldf(t * 4, cf_b + e * T * 4));
        inv_t(X, v);
      }
      for (int s = S - 1; s >= 0; --s) {
        // the slice's patch gradient, summed over the modes so far: kept in scratch until the
        // last mode, whose sum goes through the frame into the window
        {
          float2 g[EL];
          wave_at(g, m, s, wk);
#pragma unroll
          for (int i = 0; i < EL; ++i) g[i] = cmulc(g[i], v[i]);
          const int t16 = opaque_tid() * 16;
          if (!first) {
#pragma unroll
            for (int j = 0; j < EL / 2; ++j) {
              const float4 q = sb.ld2(t16, gp_b(s) + j * T * 16);
              g[2 * j] = cadd(g[2 * j], lo2(q));
              g[2 * j + 1] = cadd(g[2 * j + 1], hi2(q));
              chunk(j);
            }
          }
          if (!last) {
            store_frame(gp_b(s), g);
          } else {
            float2* c0 = lds + cell(opaque_tid(), 0);
#pragma unroll
            for (int i = 0; i < EL; ++i) c0[N1 * i] = g[i];
          }
        }
        if (last) {
          __syncthreads();
          const PatchWindow pw(a.obj + size_t(s) * HW, a.W, N, p);
          window_rows<N, T, P>(a, p, lds, pw.win,
                               a.gwin ? a.gwin + (size_t(k) * S + s) * (N + 1) * (N + 1) : nullptr, gy, gx);
          __syncthreads();
        }
        mul_frame(op_b(s), v, Conj{});
        if (s > 0) {
          float2 X[EL];
          fwd_t(v, X);  // F g_psi_s
          if constexpr (LZ) {
            // F psi_s, the incident wave's spectrum (a second forward transform)
            float2 ps[EL], Q[EL];
            __syncthreads();
            wave_at(ps, m, s, wk);
            fwd_t(ps, Q);
            const int t2 = opaque_tid();
#pragma unroll
            for (int e = 0; e < EL; ++e) {
              const int ky = F::row(t2, e), kx = F::col(t2);
              const float fy = float(ky < N / 2 ? ky : ky - N) / float(N);
              const float fx = float(kx < N / 2 ? kx : kx - N) / float(N);
              lz += double(3.14159265358979323846f * (fy * fy + fx * fx) * inv_nn * (X[e].x * Q[e].y - X[e].y * Q[e].x));
            }
          }
          apply_tf(X, Conj{});
          inv_t(X, v);
        }
      }
      lds_probe_side<N, T>(a, k, m, wk, v, pb, sb, pacc_b, acc_fresh, wacc);
    }
    if constexpr (LZ) {
      const double tot = block_sum<T>(lz, red);
      if (tid == 0) a.lz_part[k] = tot;
    }

    acc_fresh = false;
    finish_position<N, T>(a, k, gy, gx, red, wacc);
  }
  if (acc_fresh) zero_probe_acc<N, T>(a, scr + a.pacc_off);
}

}  // namespace ptyhip
