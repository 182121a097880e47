// Per-position body of the fused forward + adjoint with the working frame resident in
// LDS (128^2 frames, 1024 threads; tune variants 5 and 6).
//
// The register-resident layouts keep the working frame in registers across each 2D
// transform, so the patch, the running patch gradient and dl/dI do not all fit beside it
// and go through the workgroup's scratch once per mode. Here the frame lives in LDS
// (FrameLds: a line stage at a time in registers), and each thread keeps its own pixels
// of the per-position state in registers for the whole position: the patch o,
// the running patch gradient sum_m conj(P_m) g_m and (variant 6) dl/dI. Per position
// the scratch then sees only the probe-gradient accumulator (variant 5: and dl/dI).
// The thread that owns a pixel in the element passes is the one that reads and writes
// that cell in the row pass (cells (t / 8, t mod 8 + 8 i)), and the frequency-domain
// state is held in the layout the column pass leaves in registers, whose cells the
// thread's inverse column pass reads; so element passes and transforms meet without
// block barriers, and a forward + inverse pair costs two barriers (between rows and
// columns) instead of six. The transforms are unnormalised; every 1/N is a power of two and
// is folded into dl/dI (and into the intensity once).
//
// Per position: gather the patch; per mode form P_m o, transform, add |Psi_m|^2;
// loss and dl/dI; per mode from the last (whose far field is still in registers): the
// recomputed far field, scaled by 2 dl/dI / (K_norm N^2), transformed back; one
// element pass accumulates the probe gradient conj(o) g_m and the patch gradient
// conj(P_m) g_m (the OPR forms: the probe side and its weight terms first); the patch
// gradient is written into the frame, from which the window pass forms the window
// gradient and the position gradient.
//
// Bound by the transforms' arithmetic and the accumulator's traffic (2000 positions of 4 modes: VALU
// busy 65%, 3.5 GB at 3.3 TB/s; 6732 positions of 30 modes: 59%, 76 GB at 2.9 TB/s). Measured at 2000
// positions of 4 modes, Poisson: 1.08 ms; at 6732 positions of 30 modes 26.1 ms (28.2 with scaled
// transforms, separate probe and object passes, per-pixel window indices and 119 spilled registers).
// Of that 7% keep rounding down: radix-4 transforms with separate twiddles (fft.hpp), and sums that add one
// rounded term at a time. Keeping the far fields of 4 modes in scratch instead of recomputing
// them took 1.17-1.21 ms where recomputing took 0.97: 128 KB a mode more each way through the same memory.
// Eight pixels at a time in the element passes took 1.03 (registers spilled), sixteen probe loads at a
// time changed nothing.
#pragma once
#include "small_body.hpp"

namespace ptyhip {

template <int N, int T>
struct LdsShared {
  float2 lds[FrameLds<N, T>::LDS_ELEMS];
  float2 tws[N];
  double red[2 * (T / WAVE)];
  float wsh[MAX_EIG];
  double wacc[MAX_EIG * (T / WAVE)];
};

// CFREG: dl/dI stays in registers (variant 6); otherwise it is parked in the first half
// frame of the workgroup's scratch between its uses (variant 5). FA: a forward + adjoint
// call (a.mode).
template <int N, int T, int LOSS, bool CFREG, bool FA>
__device__ __forceinline__ void lds_body(const CallArgs& a, LdsShared<N, T>& sh, int wg, int nwg) {
  using F = FrameLds<N, T>;
  constexpr int EL = F::EL;
  constexpr int NN = N * N;
  constexpr int P = F::P;
  float2* lds = sh.lds;
  float2* tws = sh.tws;
  double* red = sh.red;
  float* wsh = sh.wsh;
  double* wacc = sh.wacc;
  const float inv_n = 1.f / float(N), inv_nn = inv_n * inv_n;
  const bool fwd = FA || a.mode != MODE_APPLY_AH;
  const bool apply_a = !FA && a.mode == MODE_APPLY_A;
  const bool adj = FA || !fwd;
  const bool want_pos = FA && (a.want & WANT_POS);
  const bool want_probe = (a.want & WANT_PROBE) != 0;
  load_twiddles<N>(tws, a.tw);
  float2* scr = a.scratch + size_t(wg) * a.scratch_stride;
  const BufFrame sb(scr, uint32_t(a.scratch_stride * sizeof(float2)));
  const int pacc_b = int(a.pacc_off * sizeof(float2));
  // A call that starts the accumulator from zero does not clear it first: the workgroup's
  // first position with a finished adjoint writes every accumulator frame without reading
  // it (acc_fresh), and a workgroup that finishes none clears it at the end. That needs
  // every frame written per position, i.e. one eigenprobe or per-position weights.
  const bool acc_lazy = adj && a.zero_acc && want_probe && !a.gpstage && (a.weights || a.E == 1);
  if (adj && a.zero_acc && want_probe && !a.gpstage && !acc_lazy) zero_probe_acc<N, T>(a, scr + a.pacc_off);
  bool acc_fresh = acc_lazy;
  // pixel (y, x) = (t / N1, t mod N1 + N1 i) of element i of thread t: the thread part of its
  // byte offset (8 N1 i further per element), its LDS cell; element loops issue four
  // elements' loads at a time (a scheduling barrier after every fourth)
  constexpr int N1 = F::N1;
  auto cell = [](int t, int i) { return (t / N1) * P + t % N1 + N1 * i; };
  auto vpix = [](int t) { return ((t / N1) * N + t % N1) * 8; };
  auto chunk = [](int i) {
    if (i % 4 == 3) __builtin_amdgcn_sched_barrier(0);
  };
  // probe reads through a buffer resource: the thread part is the vector offset and the
  // element, mode and eigenprobe parts constant and scalar offsets, so the unrolled loops
  // keep no per-element address registers live across the transforms
  const BufFrame pb(a.probe, uint32_t(size_t(a.E) * a.M * NN * sizeof(float2)));
  auto probe_px = [&](auto wc, const float* wk, int m, int vp, int i) -> float2 {
    if constexpr (!decltype(wc)::value) return pb.ld(vp + 8 * N1 * i, m * NN * 8);
    float2 acc = make_float2(0.f, 0.f);
    for (int e = 0; e < a.E; ++e) {
      const float2 u = pb.ld(vp + 8 * N1 * i, (e * a.M + m) * NN * 8);
      acc.x = fmaf(wk[e], u.x, acc.x);
      acc.y = fmaf(wk[e], u.y, acc.y);
    }
    return acc;
  };

  for (int it = xcd_rank(wg, nwg); it < a.K; it += nwg) {
    const int k = opaque_scalar(it);
    const PosInfo p = wave_position(a.pos, k, N, a.H, a.W, want_pos);
    if (!p.ok) {
      skip_position<N, T>(a, k, p);
      continue;
    }
    __syncthreads();
    if (a.weights && int(threadIdx.x) < a.E) wsh[threadIdx.x] = a.weights[size_t(k) * a.E + threadIdx.x];
    for (int i = threadIdx.x; i < MAX_EIG * (T / WAVE); i += T) wacc[i] = 0.0;
    __syncthreads();
    const PatchWindow pw(a.obj, a.W, N, p);
    // the rest of the position, with the weighted (OPR) and unweighted probe loops as
    // separate instantiations
    auto position = [&](auto wc) {
    constexpr bool WT = decltype(wc)::value;
    const float* wk = WT ? wsh : nullptr;

    float2 o[EL];
    {
      const int t = opaque_tid();
      const int vo = ((t / N1) * a.W + t % N1) * 8;
#pragma unroll
      for (int i = 0; i < EL; ++i) {
        o[i] = pw.at(vo + 8 * N1 * i);
        pin(o[i]);
        chunk(i);
      }
    }
    // forward row pass of the exit wave P_m o of mode m, fed from registers (element i
    // is the row pass's input n2 = i)
    auto exit_rows = [&](int m) {
      const int vp = vpix(opaque_tid());
      float2 u[EL];
#pragma unroll
      for (int i = 0; i < EL; ++i) {
        u[i] = cmul(probe_px(wc, wk, m, vp, i), o[i]);
        chunk(i);
      }
      F::template rows_from<false>(lds, tws, u);
    };

    // frequency-domain state (intensity, dl/dI, far fields) in the layout the forward
    // transform leaves in registers: element e of thread t is frequency (row(t, e), col(t))
    auto fpix = [](int t, int e) { return F::row(t, e) * N + F::col(t); };
    float cf[EL];
    // inverse column pass of the far field v (registers), scaled by dl/dI and its constants
    auto scaled_cols = [&](const float2 (&v)[EL]) {
      const int t4 = opaque_tid() * 4;
      float2 u[EL];
#pragma unroll
      for (int n2 = 0; n2 < EL; ++n2) {
        const int e = F::reg_of(n2);
        u[n2] = cscale(v[e], CFREG ? cf[e] : sb.ldf(t4, e * T * 4));
      }
      F::template cols_from<true>(lds, tws, u);
    };
    if (fwd) {
      float2 v[EL];
#pragma unroll
      for (int i = 0; i < EL; ++i) cf[i] = 0.f;
      for (int m = 0; m < a.M; ++m) {
        exit_rows(m);
        __syncthreads();
        F::cols_to_regs(lds, tws, v);
#pragma unroll
        for (int e = 0; e < EL; ++e) cf[e] += cabs2(v[e]);
        if (apply_a) {
          const int t = opaque_tid();
#pragma unroll
          for (int e = 0; e < EL; ++e) a.psi_out[(size_t(k) * a.M + m) * NN + fpix(t, e)] = cscale(v[e], inv_n);
        }
        if (m < a.M - 1) __syncthreads();  // column phase done before the next exit wave
      }
      if (apply_a) return;
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
        if (threadIdx.x == 0) {
          a.loss_part[k] = fin ? tot * double(a.lscale) : 0.0;
          if (!fin) {
            latch(a.flags, FLAG_NONFINITE);
            if (a.pos_part) {
              a.pos_part[2 * k] = 0.0;
              a.pos_part[2 * k + 1] = 0.0;
            }
            if (a.wvalid) a.wvalid[k] = 0;
          }
        }
        if (!fin) {
          if (a.w_part && int(threadIdx.x) < a.E) a.w_part[size_t(k) * a.E + threadIdx.x] = 0.0;
          return;
        }
      }
      if (!FA) return;
      if constexpr (!CFREG) {
        const int t4 = opaque_tid() * 4;
#pragma unroll
        for (int e = 0; e < EL; ++e) sb.stf(cf[e], t4, e * T * 4);
      }
      scaled_cols(v);  // the first adjoint step's inverse column pass (the last mode)
    }

    // adjoint, last mode first (its inverse column pass is done)
    float2 go[EL];
#pragma unroll
    for (int i = 0; i < EL; ++i) go[i] = make_float2(0.f, 0.f);
    for (int mm = 0; mm < a.M; ++mm) {
      const int m = a.M - 1 - mm;
      const bool first = mm == 0;
      // inverse transform: columns (from registers), rows
      if (!fwd) {
        // the given far field, read in the order of the thread's inverse column pass
        if (!first) __syncthreads();
        const int t = opaque_tid();
        const float2* y = a.Y + (size_t(k) * a.M + m) * NN;
        float2 u[EL];
#pragma unroll
        for (int n2 = 0; n2 < EL; ++n2) u[n2] = cscale(y[fpix(t, F::reg_of(n2))], inv_n);
        F::template cols_from<true>(lds, tws, u);
      } else if (!first) {
        float2 v[EL];
        exit_rows(m);
        __syncthreads();
        F::cols_to_regs(lds, tws, v);
        scaled_cols(v);
      }
      __syncthreads();
      F::template rows<true>(lds, tws);
      const int t = opaque_tid();
      const int vp = vpix(t);
      const float2* c0 = lds + cell(t, 0);
      if constexpr (WT) {
        // probe side: conj(o) g_m into each eigenprobe's accumulator (or the staging
        // frame), and the OPR weight terms
        if (want_probe && a.gpstage) {
          const BufFrame st(a.gpstage + (size_t(k) * a.M + m) * NN, NN * 8);
#pragma unroll
          for (int i = 0; i < EL; ++i) {
            st.st(cmulc(o[i], c0[N1 * i]), vp + 8 * N1 * i, 0);
            chunk(i);
          }
        } else if (want_probe) {
          for (int e = 0; e < a.E; ++e) {
            const int fb = pacc_b + (e * a.M + m) * NN * 8;
            const float w = wk[e];
#pragma unroll
            for (int i0 = 0; i0 < EL; i0 += 4) {
              float2 g[4];
#pragma unroll
              for (int u = 0; u < 4; ++u) g[u] = make_float2(0.f, 0.f);
              if (!acc_fresh) {
#pragma unroll
                for (int u = 0; u < 4; ++u) g[u] = sb.ld(vp + 8 * N1 * (i0 + u), fb);
              }
#pragma unroll
              for (int u = 0; u < 4; ++u) {
                const float2 gp = cmulc(o[i0 + u], c0[N1 * (i0 + u)]);
                g[u].x = fmaf(w, gp.x, g[u].x);
                g[u].y = fmaf(w, gp.y, g[u].y);
                sb.st(g[u], vp + 8 * N1 * (i0 + u), fb);
              }
              __builtin_amdgcn_sched_barrier(0);
            }
          }
        }
        if (a.want & WANT_WEIGHTS) {
          for (int e = 0; e < a.E; ++e) {
            float sf = 0.f;
#pragma unroll
            for (int i = 0; i < EL; ++i) {
              sf += cdotre(cmulc(o[i], c0[N1 * i]), pb.ld(vp + 8 * N1 * i, (e * a.M + m) * NN * 8));
              chunk(i);
            }
            const double s = wave_sum(double(sf));
            if ((threadIdx.x & (WAVE - 1)) == 0) wacc[e * (T / WAVE) + threadIdx.x / WAVE] += s;
          }
        }
        // object side: the running patch gradient
#pragma unroll
        for (int i = 0; i < EL; ++i) {
          go[i] = cadd(go[i], cmulc(probe_px(wc, wk, m, vp, i), c0[N1 * i]));
          pin(go[i]);
          chunk(i);
        }
      } else {
        // both sides, four pixels at a time: conj(o) g_m into the accumulator (or the
        // staging frame), conj(P_m) g_m into the running patch gradient
        const BufFrame st(a.gpstage ? a.gpstage + (size_t(k) * a.M + m) * NN : scr + a.pacc_off + size_t(m) * NN,
                          NN * 8);
        const bool read = !a.gpstage && !acc_fresh;
#pragma unroll
        for (int i0 = 0; i0 < EL; i0 += 4) {
          float2 g[4], Pm[4], acc[4];
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            Pm[u] = pb.ld(vp + 8 * N1 * (i0 + u), m * NN * 8);
            acc[u] = make_float2(0.f, 0.f);
            g[u] = c0[N1 * (i0 + u)];
          }
          if (want_probe && read) {
#pragma unroll
            for (int u = 0; u < 4; ++u) acc[u] = st.ld(vp + 8 * N1 * (i0 + u), 0);
          }
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            go[i0 + u] = cadd(go[i0 + u], cmulc(Pm[u], g[u]));
            pin(go[i0 + u]);
          }
          if (want_probe) {
#pragma unroll
            for (int u = 0; u < 4; ++u) st.st(cadd(acc[u], cmulc(o[i0 + u], g[u])), vp + 8 * N1 * (i0 + u), 0);
          }
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    }
    {
      float2* c0 = lds + cell(opaque_tid(), 0);
#pragma unroll
      for (int i = 0; i < EL; ++i) c0[N1 * i] = go[i];
    }
    acc_fresh = false;  // every accumulator frame holds this position's terms now
    __syncthreads();
    double gy = 0.0, gx = 0.0;
    window_rows<N, T, P>(a, p, lds, pw.win, a.gwin ? a.gwin + size_t(k) * (N + 1) * (N + 1) : nullptr, gy, gx);
    finish_position<N, T>(a, k, gy, gx, red, wacc);
    };
    if (a.weights) position(std::true_type{});
    else position(std::false_type{});
  }
  if (acc_fresh) zero_probe_acc<N, T>(a, scr + a.pacc_off);
}

}  // namespace ptyhip
