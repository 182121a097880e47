// Near-field fused forward + adjoint with the working frame resident in LDS (128^2 frames,
// 1024 threads): the detector wave is Psi = F^-1(H F chi), the detector in natural pixel
// order.
//
// Layouts as in lds_ms.hpp: spatial state of a pixel with the thread whose row pass reads
// its cell, frequency state in the layout the column pass leaves in registers, frames of the
// workgroup's scratch as pairs. Per mode the forward keeps z = H F chi / N^2 in scratch; the
// adjoint transforms it back to Psi, scales by dl/dI, transforms to F g_Psi, takes the
// det_lambda_z gradient Re sum_f conj(F g_Psi) (-i pi q^2) z, and brings conj(H) F g_Psi
// back. The last mode starts from the Psi that the forward leaves in registers. The
// transforms are unnormalised, 1/N^2 goes with H. Scratch: patch [NN], patch-gradient sum
// [NN], z of every mode [M][NN], dl/dI [NN floats], probe accumulator.
// Bound by the ten (two modes) transforms' arithmetic and LDS passes of a position and, for
// few positions, by the last round of workgroups. 300 positions of 2 modes: 275 us, 396 with the
// frame in the registers of 512 threads, every spatial state through scratch and one more
// transform per position.
// FA: a forward + adjoint call (a.mode), otherwise the forward alone.
#pragma once
#include "lds_ms.hpp"

namespace ptyhip {

template <int N, int T, int LOSS, bool FA>
__device__ __forceinline__ void lds_near_body(const CallArgs& a, LdsShared<N, T>& sh, int wg, int nwg) {
  using F = FrameLds<N, T>;
  constexpr int EL = F::EL, NN = N * N, P = F::P, N1 = F::N1;
  constexpr int FB = NN * 8;  // bytes of a frame
  float2* lds = sh.lds;
  float2* tws = sh.tws;
  double* red = sh.red;
  float* wsh = sh.wsh;
  double* wacc = sh.wacc;
  const int tid = threadIdx.x;
  const float inv_nn = 1.f / float(NN);
  const bool want_pos = FA && (a.want & WANT_POS);
  const bool want_lz = FA && (a.want & WANT_LZ) && a.lz_part != nullptr;
  const bool want_probe = (a.want & WANT_PROBE) != 0;
  load_twiddles<N>(tws, a.tw);
  float2* scr = a.scratch + size_t(wg) * a.scratch_stride;
  const BufFrame sb(scr, uint32_t(a.scratch_stride * sizeof(float2)));
  constexpr int O_B = 0, G_B = FB;
  const auto z_b = [](int m) { return (2 + m) * FB; };
  const int pacc_b = int(a.pacc_off * sizeof(float2));
  const int cf_b = pacc_b - NN * 4;
  // (the accumulator is written, not read, by the first finished position, as in lds_body)
  const bool acc_lazy = FA && a.zero_acc && want_probe && !a.gpstage && (a.weights || a.E == 1);
  if (FA && a.zero_acc && want_probe && !a.gpstage && !acc_lazy) zero_probe_acc<N, T>(a, scr + a.pacc_off);
  bool acc_fresh = acc_lazy;
  const BufFrame pb(a.probe, uint32_t(size_t(a.E) * a.M * NN * sizeof(float2)));
  const BufFrame hb(a.tfd, FB);
  // four pairs' loads are issued at a time
  const auto chunk = [](int j) {
    if (j % 4 == 3) __builtin_amdgcn_sched_barrier(0);
  };
  const auto vpix = [](int t) { return ((t / N1) * N + t % N1) * 8; };
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
  const auto mul_patch = [&](float2 (&x)[EL], auto conj) {
    const int t16 = opaque_tid() * 16;
#pragma unroll
    for (int j = 0; j < EL / 2; ++j) {
      const float4 q = sb.ld2(t16, O_B + j * T * 16);
      x[2 * j] = decltype(conj)::value ? cmulc(lo2(q), x[2 * j]) : cmul(x[2 * j], lo2(q));
      x[2 * j + 1] = decltype(conj)::value ? cmulc(hi2(q), x[2 * j + 1]) : cmul(x[2 * j + 1], hi2(q));
      chunk(j);
    }
  };
  using Plain = std::false_type;
  using Conj = std::true_type;
  // spatial (R) -> frequency (C2, registers); starts in the row phase, ends in the column phase
  const auto fwd_t = [&](float2 (&x)[EL], float2 (&X)[EL]) {
    F::template rows_from<false>(lds, tws, x);
    __syncthreads();
    F::cols_to_regs(lds, tws, X);
  };
  // frequency (C2) -> spatial (R); starts in the column phase, ends in the row phase
  const auto inv_t = [&](const float2 (&X)[EL], float2 (&x)[EL]) {
    float2 u[EL];
#pragma unroll
    for (int n2 = 0; n2 < EL; ++n2) u[n2] = X[F::reg_of(n2)];
    F::template cols_from<true>(lds, tws, u);
    __syncthreads();
    F::template rows_to_regs<true>(lds, tws, x);
  };
  // X *= H / N^2 (or its conjugate) at the thread's frequencies
  const auto apply_h = [&](float2 (&X)[EL], auto conj) {
    const int t = opaque_tid();
    const int vf = (F::row(t, 0) * N + F::col(t)) * 8;
#pragma unroll
    for (int e = 0; e < EL; ++e) {
      const float2 h = cscale(hb.ld(vf, (N1 * (e / N1) + F::N2 * (e % N1)) * N * 8), inv_nn);
      X[e] = decltype(conj)::value ? cmulc(h, X[e]) : cmul(h, X[e]);
      chunk(e);
    }
  };
  const auto probe_r = [&](const float* wk, int m, float2 (&v)[EL]) {
    const int vp = vpix(opaque_tid());
    if (wk == nullptr) {
#pragma unroll
      for (int i = 0; i < EL; ++i) v[i] = pb.ld(vp + 8 * N1 * i, m * FB);
      return;
    }
#pragma unroll
    for (int i = 0; i < EL; ++i) v[i] = make_float2(0.f, 0.f);
    for (int e = 0; e < a.E; ++e) {
#pragma unroll
      for (int i = 0; i < EL; ++i) {
        const float2 u = pb.ld(vp + 8 * N1 * i, (e * a.M + m) * FB);
        v[i].x = fmaf(wk[e], u.x, v[i].x);
        v[i].y = fmaf(wk[e], u.y, v[i].y);
        chunk(i);
      }
    }
  };

  for (int it = xcd_rank(wg, nwg); it < a.K; it += nwg) {
    const int k = opaque_scalar(it);
    const PosInfo p = wave_position(a.pos, k, N, a.H, a.W, want_pos);
    if (!p.ok) {
      skip_position<N, T>(a, k, p);
      if (tid == 0 && a.lz_part) a.lz_part[k] = 0.0;
      continue;
    }
    __syncthreads();
    if (a.weights && tid < a.E) wsh[tid] = a.weights[size_t(k) * a.E + tid];
    for (int i = tid; i < MAX_EIG * (T / WAVE); i += T) wacc[i] = 0.0;
    __syncthreads();
    const float* wk = a.weights ? wsh : nullptr;
    const PatchWindow pw(a.obj, a.W, N, p);
    {
      const int t = opaque_tid();
      const int vo = ((t / N1) * a.W + t % N1) * 8;
#pragma unroll
      for (int j = 0; j < EL / 2; ++j) {
        sb.st2(cat2(pw.at(vo + 16 * N1 * j), pw.at(vo + 16 * N1 * j + 8 * N1)), t * 16, O_B + j * T * 16);
        if (j % 2 == 1) __builtin_amdgcn_sched_barrier(0);
      }
    }
    float2 v[EL];
    float cf[EL];
#pragma unroll
    for (int i = 0; i < EL; ++i) cf[i] = 0.f;
    for (int m = 0; m < a.M; ++m) {
      float2 X[EL];
      probe_r(wk, m, v);
      mul_patch(v, Plain{});
      fwd_t(v, X);
      apply_h(X, Plain{});
      if (FA && (m < a.M - 1 || want_lz)) store_frame(z_b(m), X);
      inv_t(X, v);
#pragma unroll
      for (int i = 0; i < EL; ++i) cf[i] += cabs2(v[i]);
    }
    // loss and dl/dI (detector in natural order, the thread's own pixels)
    {
      const int pix = vpix(opaque_tid()) / 8;
      const float* im = a.imeas + size_t(k) * NN + pix;
      float imv[EL];
#pragma unroll
      for (int i = 0; i < EL; ++i) imv[i] = __builtin_nontemporal_load(im + N1 * i);
      if (a.ipred) {
        float* ip = a.ipred + size_t(k) * NN + pix;
#pragma unroll
        for (int i = 0; i < EL; ++i) __builtin_nontemporal_store(cf[i], ip + N1 * i);
      }
      double lsum = 0.0;
#pragma unroll
      for (int i = 0; i < EL; ++i) {
        float l, c;
        loss_terms<LOSS>(cf[i], imv[i], a.eps, l, c);
        lsum += double(l);
        cf[i] = a.gscale * c;
        chunk(i);
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
          if (a.lz_part) a.lz_part[k] = 0.0;
        }
      }
      if (!fin) {
        if (a.w_part && tid < a.E) a.w_part[size_t(k) * a.E + tid] = 0.0;
        continue;
      }
      if constexpr (!FA) continue;
    }
    {
      const int t4 = opaque_tid() * 4;
#pragma unroll
      for (int i = 0; i < EL; ++i) {
        if (a.M > 1) sb.stf(cf[i], t4, cf_b + i * T * 4);
        v[i] = cscale(v[i], cf[i]);  // g_Psi of the last mode, which the adjoint starts with
      }
    }

    double gy = 0.0, gx = 0.0, lz = 0.0;
    for (int mm = 0; mm < a.M; ++mm) {
      const int m = mm == 0 ? a.M - 1 : mm - 1;
      const bool first = mm == 0, last = mm == a.M - 1;
      float2 X[EL];
      if (!first) {
        load_frame(z_b(m), X);
        __syncthreads();  // the previous mode's row phase is done
        inv_t(X, v);
        const int t4 = opaque_tid() * 4;
#pragma unroll
        for (int i = 0; i < EL; ++i) v[i] = cscale(v[i], sb.ldf(t4, cf_b + i * T * 4));
      }
      fwd_t(v, X);  // F g_Psi
      if (want_lz) {
        const int t = opaque_tid(), t16 = t * 16, zb = z_b(m);
#pragma unroll
        for (int j = 0; j < EL / 2; ++j) {
          const float4 q = sb.ld2(t16, zb + j * T * 16);
#pragma unroll
          for (int u = 0; u < 2; ++u) {
            const int e = 2 * j + u;
            const float2 z = u ? hi2(q) : lo2(q);
            const int ky = F::row(t, e), kx = F::col(t);
            const float fy = float(ky < N / 2 ? ky : ky - N) / float(N);
            const float fx = float(kx < N / 2 ? kx : kx - N) / float(N);
            lz += double(3.14159265358979323846f * (fy * fy + fx * fx) * (X[e].x * z.y - X[e].y * z.x));
          }
          chunk(j);
        }
      }
      apply_h(X, Conj{});
      inv_t(X, v);  // gradient of the exit wave
      // patch gradient, summed over the modes so far: kept in scratch until the last mode, whose
      // sum goes through the frame into the window
      {
        float2 g[EL];
        probe_r(wk, m, g);
#pragma unroll
        for (int i = 0; i < EL; ++i) g[i] = cmulc(g[i], v[i]);
        const int t = opaque_tid();
        if (!first) {
#pragma unroll
          for (int j = 0; j < EL / 2; ++j) {
            const float4 q = sb.ld2(t * 16, G_B + j * T * 16);
            g[2 * j] = cadd(g[2 * j], lo2(q));
            g[2 * j + 1] = cadd(g[2 * j + 1], hi2(q));
            chunk(j);
          }
        }
        if (!last) {
          store_frame(G_B, g);
        } else {
          float2* c0 = lds + (t / N1) * P + t % N1;
#pragma unroll
          for (int i = 0; i < EL; ++i) c0[N1 * i] = g[i];
        }
      }
      mul_patch(v, Conj{});
      lds_probe_side<N, T>(a, k, m, wk, v, pb, sb, pacc_b, acc_fresh, wacc);
    }
    __syncthreads();
    window_rows<N, T, P>(a, p, lds, pw.win, a.gwin ? a.gwin + size_t(k) * (N + 1) * (N + 1) : nullptr, gy, gx);
    if (want_lz) {
      const double tot = block_sum<T>(lz, red);
      if (tid == 0) a.lz_part[k] = tot;
    }
    acc_fresh = false;
    finish_position<N, T>(a, k, gy, gx, red, wacc);
  }
  if (acc_fresh) zero_probe_acc<N, T>(a, scr + a.pacc_off);
}

}  // namespace ptyhip
