// Per-position body of the fused forward + adjoint for 256^2 and 512^2 frames,
// shared by the per-plan kernels and the batched kernel.
//
// One workgroup owns one scan position at a time. A frame does not fit on chip, so a 2D
// transform runs as a pass over the rows and a pass over the columns whose intermediate
// is the workgroup's work frame in scratch. Each pass is a loop of independent wavefronts:
// a wave takes four lines at a time from memory into registers, transforms them
// (WaveLines, exchange through the wave's own LDS cells) and works on the results in
// registers, so the only block barriers are those between passes and a wave's loads
// overlap the other waves' arithmetic. Rows of natural frames (probe, object, staged
// gradients, windows) are read and written as pairs of pixels, 16 bytes a lane: a wave's
// access costs the address unit 16 cycles at 8 and at 16 bytes a lane, and it was the
// busiest unit. Measured against line blocks shared by the workgroup in LDS: 2500
// positions of 256^2 with 8 eigenprobes 2.84 ms (4.19), 331 forward positions of 256^2
// with 3 modes 0.47 ms (0.74); 10.9 GB cross the far side of the L2s at 256^2 (10.4), but at 3.9
// instead of 2.5 TB/s (a device copy reaches 5.1), the VALU busy 44%: the streamed frames, not the
// transforms, bound the kernel now. The passes
// are arranged so that a frame crosses scratch as few times as possible:
//   - the exit wave P_m o is formed as the row pass loads (patch taps from the object,
//     probe from the eigenprobes), so neither is stored;
//   - the column pass of the last mode completes the incoherent intensity, the loss and
//     dl/dI, and (forward + adjoint) runs that mode's inverse column transforms on the
//     same registers; earlier modes keep their far fields and the partial intensity;
//   - the inverse row pass forms both conjugate products and in the last mode emits the
//     window gradient and the position-gradient terms from registers, so the patch
//     gradient of a single-mode position never leaves the chip.
// The work frame is stored in 4 x 4 pixel tiles (tile row, tile column, row, column), one
// 128-byte line each: a row pass writes 4 rows x 16 columns per instruction as 512
// contiguous bytes and a column pass reads 16 rows x 4 columns as four whole lines.
// Far fields, intensities and dl/dI are kept in the order the column pass holds them in
// (four columns cg, then element kk, then lane), again 512 contiguous bytes.
// The probe gradient accumulates in the workgroup's own scratch slice or is staged per
// position; the window gradient goes to the window buffer (no atomics).
#pragma once
#include "../device/fft.hpp"
#include "../device/model.hpp"
#include "args.hpp"

namespace ptyhip {

constexpr int BIG_MAX_EIG = 16;

template <int N, int TT>
struct Big {
  static constexpr int T = TT;
  static constexpr int NW = TT / WAVE;
  static constexpr int N2 = N / 16;        // elements of a line per thread
  static constexpr int GROUPS = N / 4;     // groups of four lines
  static constexpr int GPW = GROUPS / NW;  // of which a wave takes
  static_assert(GPW * NW == GROUPS, "the waves must share the lines evenly");
  static constexpr int NN = N * N;
  static constexpr int WN = N + 1;
};

// LDS the body needs (owned by the caller): 4 N cells of exchange per wave
template <int N, int TT>
struct BigShared {
  float2 ex[Big<N, TT>::NW][4 * N];
  float2 tw[N];
  double red[2 * Big<N, TT>::NW];
  double wred[BIG_MAX_EIG * Big<N, TT>::NW];
  float wsh[BIG_MAX_EIG];
};
static_assert(sizeof(BigShared<256, 1024>) <= 160 * 1024 && sizeof(BigShared<512, 512>) <= 160 * 1024, "LDS of a CU");

// scratch per workgroup: work frame F; with M > 1 also the patch gradient summed over
// modes G and the far fields of modes 0..M-2; the partial intensity / dl/dI (NN
// floats); the probe accumulator [E][M] at pacc_off
inline size_t big_scratch_elems(int N, int M, int E, size_t* pacc_off) {
  const size_t nn = size_t(N) * N;
  *pacc_off = nn * (1 + (M > 1 ? size_t(M) : 0)) + nn / 2;
  return *pacc_off + nn * size_t(E) * M;
}

// Lane moves within the 16 lanes of a row (lanes outside the bank mask keep `old`):
// CTRL 0x128 rotates by 8, 0x111 takes the lane to the left, 0x101 the lane to the right,
// 0x121 and 0x12f the same with wrap-around.
template <int CTRL, int BANKS = 0xf>
__device__ __forceinline__ float2 row_dpp(float2 old, float2 x) {
  const auto f = [](float o, float v) {
    return __builtin_bit_cast(
        float, __builtin_amdgcn_update_dpp(__builtin_bit_cast(int, o), __builtin_bit_cast(int, v), CTRL, 0xf, BANKS, false));
  };
  return make_float2(f(old.x, x.x), f(old.y, x.y));
}
// A row's pixels as pairs (lane q holds pixels 32 i + 2 q and + 1: one 16-byte access) to and
// from the transform's order (lane q holds pixels n1 + 16 n2 with n1 = 2 (q mod 8) + q / 8):
// lanes q and q ^ 8 swap one pixel of each pair. The exchange is its own inverse.
__device__ __forceinline__ void swap_pair(float2& x0, float2& x1) {
  const float2 a = row_dpp<0x128, 0xc>(x0, x1);
  x1 = row_dpp<0x128, 0x3>(x1, x0);
  x0 = a;
}

// Workgroup `wg` of `nwg` processes every nwg-th work item of the call `a`, starting at its
// place in the order of XCDs.
// PH 0: an item is a position (every mode, loss and adjoint). The mode-split form
// (a.groups > 1) makes every (position k, mode group g) pair an item k G + g and runs
// in three passes: PH 1 writes the far fields of the item's modes to a.far (forward +
// adjoint) and the partial intensity sum_{m in g} |Psi_m|^2 to ipart; a loss pass sums a
// position's partials and writes 2 dl/dI / (K_norm N^2) to cfr; PH 2 scales each far field
// of the group by cfr, transforms it back and forms the products (staged probe-wave
// gradients, window k G + g, per-item position partial sums).
// FA: a forward + adjoint call (a.mode), whose instance then carries no other mode's
// conditions and addresses through its passes.
template <int N, int TT, int LOSS, int PH, bool FA>
__device__ __forceinline__ void big_body(const CallArgs& a, BigShared<N, TT>& sh, int wg, int nwg) {
  using B = Big<N, TT>;
  using WL = WaveLines<N>;
  constexpr int T = B::T, NN = B::NN, NW = B::NW, N2 = B::N2, GPW = B::GPW, WN = B::WN;
  constexpr int BAT = 8;       // pixels whose loads are in flight together
  constexpr bool HREG = N == 512;  // 256 registers a thread: the row above is kept in them
  constexpr int BP = BAT / 2;  // as pairs of neighbouring pixels, 16 bytes per access
  const int tid = threadIdx.x;
  const int lane = tid & (WAVE - 1), wave = __builtin_amdgcn_readfirstlane(tid / WAVE);
  // lanes of a row pass: row r of the group and pixel n1 + 16 n2 (stage 1; memory is read
  // and written as pairs, pixels 32 i + 2 q and + 1), row tr and frequency tq + 16 kk (stage 2, the order of the tiles); of a column pass: column cc of
  // the group and row (frequency) cq + 16 n2 (kk)
  const int r = lane >> 4, q = lane & 15, n1 = 2 * (q & 7) + (q >> 3);
  const int tr = (lane >> 2) & 3, tq = (lane & 3) + 4 * (lane >> 4);
  const int cc = lane & 3, cq = lane >> 2;
  float2* ex = sh.ex[wave];
  const float2* tws = sh.tw;
  double* red = sh.red;
  float* wsh = sh.wsh;
  const float inv_n = 1.f / float(N);
  const bool fwd = FA || a.mode != MODE_APPLY_AH;
  const bool apply_a = !FA && a.mode == MODE_APPLY_A;
  constexpr bool fa = FA;
  const bool want_pos = (a.want & WANT_POS) && fa;
  const bool want_probe = (a.want & WANT_PROBE) != 0;
  const int M = a.M;
  float2* scr = a.scratch + size_t(wg) * a.scratch_stride;
  float2* Fr = scr;
  float2* G = Fr + NN;
  float2* Ps = G + NN;
  float* cf = reinterpret_cast<float*>(M > 1 ? Ps + size_t(M - 1) * NN : G);
  float2* pacc = scr + a.pacc_off;
  const BufFrame fr(Fr, NN * 8);
  const BufFrame gb(G, NN * 8);  // patch gradient over modes (M > 1)
  const BufFrame cfb(cf, NN * 4);
  // byte offsets of the thread in: a group's 4 N contiguous elements, element i at
  // 64 i (LIN); the natural layout, pair 32 i + 2 q of row r; the patch window
  // (bases made opaque where they are used, so that the elements' constants fold into the
  // instructions instead of being added outside the loops and kept in registers)
  const int v_lin0 = lane * 8, v_nat0 = (r * N + 2 * q) * 8, v_win0 = (r * a.W + 2 * q) * 8;
  const int v_colw = ((cq >> 2) * 4 * N + (lane & 15)) * 8;  // work frame, column order
  const auto lin_v = [](int v_lin, int i) { return v_lin + (i & 7) * 512; };
  const auto linf_v = [](int v_lin4, int i) { return v_lin4 + (i & 7) * 256; };  // frames of floats
  const auto linf_s = [](int g, int i) { return g * 4 * N * 4 + (i >> 3) * 2048; };
  const auto lin_s = [](int g, int i) { return g * 4 * N * 8 + (i >> 3) * 4096; };
  // The probe accumulator is not cleared: the workgroup's first position with a finished
  // adjoint writes every frame without reading it, a workgroup that finishes none clears it.
  const bool acc_lazy = PH == 0 && (fa || !fwd) && a.zero_acc && want_probe && !a.gpstage &&
                        (a.weights || a.E == 1);
  const auto clear_acc = [&]() {
    for (size_t i = tid; i < size_t(a.E) * M * NN; i += T) pacc[i] = make_float2(0.f, 0.f);
  };
  if (PH == 0 && (fa || !fwd) && a.zero_acc && want_probe && !a.gpstage && !acc_lazy) clear_acc();
  bool acc_fresh = acc_lazy;
  WL::table(sh.tw, a.tw);
  __syncthreads();

  // columns of group cg between the work frame and registers (row cq + 16 n2 of column cc)
  const auto cols_load = [&](int cg, float2 (&u)[N2]) {
#pragma unroll
    for (int i = 0; i < N2; ++i) u[i] = fr.ld(v_colw, cg * 128 + i * 16 * N * 8);
  };
  const auto cols_store = [&](int cg, const float2 (&u)[N2]) {
#pragma unroll
    for (int i = 0; i < N2; ++i) fr.st(u[i], v_colw, cg * 128 + i * 16 * N * 8);
  };
  // |x|^2 of a column group's far field added into a frame of intensities
  const auto add_intensity = [&](const BufFrame& f, int vf, int cg, bool init, const float2 (&x)[N2]) {
    float I[N2];
#pragma unroll
    for (int i = 0; i < N2; ++i) I[i] = 0.f;
    if (!init) {
#pragma unroll
      for (int i = 0; i < N2; ++i) I[i] = f.ldf(linf_v(vf, i), linf_s(cg, i));
    }
#pragma unroll
    for (int i = 0; i < N2; ++i) f.stf(I[i] + cabs2(x[i]), linf_v(vf, i), linf_s(cg, i));
  };
  // detector index (DC-centred) of element kk of the thread in column group cg
  const auto det = [&](int cg, int kk) {
    return cq * N + cc + (kk ^ (N2 / 2)) * 16 * N + ((4 * cg + N / 2) & (N - 1));
  };

  // work items: positions (PH 0) or (position, mode group) pairs (PH 1, 2)
  const int NG = PH == 0 ? 1 : a.groups;
  const int items = a.K * NG;
  for (int j = xcd_rank(wg, nwg); j < items; j += nwg) {
    // mode-split items in the order of the groups: neighbours share their modes' eigenprobes
    const int it = PH == 0 ? j : (j % a.K) * NG + j / a.K;
    // (opaque: the addresses of the item's frames are formed where they are used, not
    // carried from item to item in registers)
    const int k = opaque_scalar(PH == 0 ? it : it / NG);
    const int m0 = PH == 0 ? 0 : (it - k * NG) * a.group_modes;
    const int m1 = PH == 0 ? M : min(M, m0 + a.group_modes);
    if constexpr (PH == 2) {
      if (!a.kvalid[k]) {
        if (tid == 0) {
          a.wvalid[it] = 0;
          if (a.pos_part) {
            a.pos_part[2 * size_t(it)] = 0.0;
            a.pos_part[2 * size_t(it) + 1] = 0.0;
          }
        }
        continue;
      }
    }
    const PosInfo p = wave_position(a.pos, k, N, a.H, a.W, want_pos);
    if constexpr (PH == 1) {
      if (!p.ok) continue;  // the loss pass drops the position
    }
    if (PH == 0 && !p.ok) {
      if (tid == 0) {
        latch(a.flags, p.finite ? FLAG_BOUNDS : FLAG_NONFINITE);
        if (a.loss_part) a.loss_part[k] = 0.0;
        if (a.pos_part) {
          a.pos_part[2 * k] = 0.0;
          a.pos_part[2 * k + 1] = 0.0;
        }
        if (a.wvalid) a.wvalid[k] = 0;
      }
      if (a.w_part && tid < a.E) a.w_part[size_t(k) * a.E + tid] = 0.0;
      if (a.ipred)
        for (int i = tid; i < NN; i += T) a.ipred[size_t(k) * NN + i] = 0.f;
      if (apply_a)
        for (int i = tid; i < M * NN; i += T) a.psi_out[size_t(k) * M * NN + i] = make_float2(0.f, 0.f);
      continue;
    }
    __syncthreads();
    if (tid < a.E) wsh[tid] = a.weights ? a.weights[size_t(k) * a.E + tid] : 1.f;
    for (int i = tid; i < BIG_MAX_EIG * NW; i += T) sh.wred[i] = 0.0;
    __syncthreads();
    const float* wk = wsh;  // 1 where the call has no weights (one eigenprobe)

    // bilinear patch taps through a buffer over the (N+1) x (N+1) window; a tap of zero
    // weight re-reads the base pixel
    const BufFrame win(a.obj + size_t(p.y0) * a.W + p.x0, uint32_t((N * a.W + N + 1) * 8));
    const int wdx = p.fx > 0.f ? 8 : 0, wdy = p.fy > 0.f ? a.W * 8 : 0;
    const float w00 = (1.f - p.fy) * (1.f - p.fx), w01 = (1.f - p.fy) * p.fx;
    const float w10 = p.fy * (1.f - p.fx), w11 = p.fy * p.fx;
    // patch at the pairs i0.. of row group rg: per tap row 16-byte loads of (x, x + 1), x + 2
    // is the lane to the right (lane 15: lane 0's next pair, or one more load at the batch's end)
    const auto patch_batch = [&](int rg, int i0, float2 (&o)[BAT]) {
      const int v_win = opaque(v_win0), so = rg * 4 * a.W * 8, v_end = v_win - q * 16;
      const int x_end = i0 + BP < N2 / 2 ? (i0 + BP) * 256 : (N - 1) * 8 + wdx;
      float4 t[2][BP];
      float2 e[2];
#pragma unroll
      for (int y = 0; y < 2; ++y) {
        e[y] = win.ld(v_end, so + y * wdy + x_end);
#pragma unroll
        for (int j = 0; j < BP; ++j) t[y][j] = win.ld2(v_win + (i0 + j) * 256, so + y * wdy);
      }
#pragma unroll
      for (int j = BP - 1; j >= 0; --j) {
        float2 n[2];
#pragma unroll
        for (int y = 0; y < 2; ++y) {
          n[y] = row_dpp<0x101>(e[y], lo2(t[y][j]));
          e[y] = row_dpp<0x12f>(e[y], lo2(t[y][j]));
        }
        const float4 a0 = t[0][j], a1 = t[1][j];
        o[2 * j].x = w00 * a0.x + w01 * a0.z + w10 * a1.x + w11 * a1.z;
        o[2 * j].y = w00 * a0.y + w01 * a0.w + w10 * a1.y + w11 * a1.w;
        o[2 * j + 1].x = w00 * a0.z + w01 * n[0].x + w10 * a1.z + w11 * n[1].x;
        o[2 * j + 1].y = w00 * a0.w + w01 * n[0].y + w10 * a1.w + w11 * n[1].y;
      }
    };
    // probe P_m of this position at the pairs i0.. of row group rg, eigenprobe by
    // eigenprobe so that the loads of one eigenprobe are in flight together;
    // `each(e, u)` sees every eigenprobe's values
    const auto probe_batch = [&](int m, int rg, int i0, float2 (&P)[BAT], auto&& each) {
#pragma unroll
      for (int j = 0; j < BAT; ++j) P[j] = make_float2(0.f, 0.f);
#pragma unroll 2
      for (int e = 0; e < a.E; ++e) {
        const BufFrame ub(a.probe + (size_t(e) * M + m) * NN, NN * 8);
        const float we = wk[e];
        const int v_nat = opaque(v_nat0);
        float4 u[BP];
#pragma unroll
        for (int j = 0; j < BP; ++j) u[j] = ub.ld2(v_nat + (i0 + j) * 256, rg * 4 * N * 8);
#pragma unroll
        for (int j = 0; j < BP; ++j) {
          P[2 * j].x = fmaf(we, u[j].x, P[2 * j].x);
          P[2 * j].y = fmaf(we, u[j].y, P[2 * j].y);
          P[2 * j + 1].x = fmaf(we, u[j].z, P[2 * j + 1].x);
          P[2 * j + 1].y = fmaf(we, u[j].w, P[2 * j + 1].y);
        }
        each(e, u);
      }
    };
    // row transforms of the exit wave P_m o into the work frame
    const auto exit_rows = [&](int m) {
#pragma unroll 1
      for (int gi = 0; gi < GPW; ++gi) {
        const int rg = gi * NW + wave;
        float2 u[N2], v[N2];
#pragma unroll
        for (int i0 = 0; i0 < N2 / 2; i0 += BP) {
          float2 P[BAT], o[BAT];
          probe_batch(m, rg, i0, P, [](int, const float4(&)[BP]) {});
          patch_batch(rg, i0, o);
#pragma unroll
          for (int j = 0; j < BAT; ++j) {
            u[2 * i0 + j] = cmul(P[j], o[j]);
            pin(u[2 * i0 + j]);
          }
          __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int i = 0; i < N2; i += 2) swap_pair(u[i], u[i + 1]);
        WL::forward(ex, tws, r, n1, tr, tq, u, v);
        const int vl = opaque(v_lin0);
#pragma unroll
        for (int i = 0; i < N2; ++i) fr.st(v[i], lin_v(vl, i), lin_s(rg, i));
      }
    };

    if constexpr (PH == 1) {
      // far fields and partial intensity of the group's modes
      const BufFrame ipb(a.ipart + size_t(it) * NN, NN * 4);
      for (int m = m0; m < m1; ++m) {
        if (m > m0) __syncthreads();  // the previous mode's columns are read
        exit_rows(m);
        __syncthreads();
        const BufFrame far(a.far ? a.far + (size_t(k) * M + m) * NN : Fr, NN * 8);
#pragma unroll 1
        for (int gi = 0; gi < GPW; ++gi) {
          const int cg = gi * NW + wave;
          float2 u[N2], v[N2];
          cols_load(cg, u);
          WL::forward(ex, tws, cc, cq, cc, cq, u, v);
          const int vl = opaque(v_lin0), vf = opaque(lane * 4);
#pragma unroll
          for (int i = 0; i < N2; ++i) v[i] = cscale(v[i], inv_n);
          if (a.far) {
#pragma unroll
            for (int i = 0; i < N2; ++i) far.st(v[i], lin_v(vl, i), lin_s(cg, i));
          }
          add_intensity(ipb, vf, cg, m == m0, v);
        }
      }
      continue;
    }

    if (PH == 0 && fwd) {
      double lsum = 0.0;
      const float* im = a.imeas ? a.imeas + size_t(k) * NN : nullptr;
      for (int m = 0; m < M; ++m) {
        const bool last = m == M - 1;
        if (m > 0) __syncthreads();  // the previous mode's columns are read
        exit_rows(m);
        __syncthreads();
        // column transforms: far field and intensity; the last mode also the loss, dl/dI
        // and (forward + adjoint) its own inverse column transforms
#pragma unroll 1
        for (int gi = 0; gi < GPW; ++gi) {
          const int cg = gi * NW + wave;
          float2 u[N2], v[N2];
          cols_load(cg, u);
          if (apply_a) {
            WL::forward(ex, tws, cc, cq, cc, cq, u, v);
            float2* out = a.psi_out + (size_t(k) * M + m) * NN + cq * N + 4 * cg + cc;
#pragma unroll
            for (int i = 0; i < N2; ++i) out[i * 16 * N] = cscale(v[i], inv_n);
          } else if (!last) {
            const BufFrame pb(Ps + size_t(m) * NN, NN * 8);
            WL::forward(ex, tws, cc, cq, cc, cq, u, v);
            const int vl = opaque(v_lin0), vf = opaque(lane * 4);
#pragma unroll
            for (int i = 0; i < N2; ++i) v[i] = cscale(v[i], inv_n);
            if (fa) {
#pragma unroll
              for (int i = 0; i < N2; ++i) pb.st(v[i], lin_v(vl, i), lin_s(cg, i));
            }
            add_intensity(cfb, vf, cg, m == 0, v);
          } else {
            const BufFrame imb(im, NN * 4);
            float imv[N2];
#pragma unroll
            for (int i = 0; i < N2; ++i)
              imv[i] = imb.ldf((cq * N + cc) * 4, ((i ^ (N2 / 2)) * 16 * N + ((4 * cg + N / 2) & (N - 1))) * 4);
            WL::forward(ex, tws, cc, cq, cc, cq, u, v);
            float I[N2];
            const int vf = opaque(lane * 4);
#pragma unroll
            for (int i = 0; i < N2; ++i) I[i] = 0.f;
            if (m > 0) {
#pragma unroll
              for (int i = 0; i < N2; ++i) I[i] = cfb.ldf(linf_v(vf, i), linf_s(cg, i));
            }
#pragma unroll
            for (int i = 0; i < N2; ++i) {
              v[i] = cscale(v[i], inv_n);
              I[i] += cabs2(v[i]);
            }
            if (a.ipred) {
#pragma unroll
              for (int i = 0; i < N2; ++i) a.ipred[size_t(k) * NN + det(cg, i)] = I[i];
            }
#pragma unroll
            for (int i = 0; i < N2; ++i) {
              float l, c;
              loss_terms<LOSS>(I[i], imv[i], a.eps, l, c);
              lsum += double(l);
              I[i] = c;
              v[i] = cscale(v[i], a.gscale * c);
              if (i % 4 == 3) __builtin_amdgcn_sched_barrier(0);
            }
            if (fa && M > 1) {
#pragma unroll
              for (int i = 0; i < N2; ++i) cfb.stf(I[i], linf_v(vf, i), linf_s(cg, i));
            }
            if (fa) {
              WL::inverse(ex, tws, cc, cq, cc, cq, v, u);
              cols_store(cg, u);
            }
          }
        }
      }
      if (apply_a) continue;
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
        }
      }
      if (!fin) {
        if (a.w_part && tid < a.E) a.w_part[size_t(k) * a.E + tid] = 0.0;
        continue;
      }
      if (!fa) continue;
    }

    // adjoint, one mode at a time. Staged probe-wave gradients leave the weight gradients to
    // the contraction of the staged frames; otherwise the terms are summed in FP32 over a
    // thread's pixels of a batch, then in FP64.
    const bool want_w = (a.want & WANT_WEIGHTS) && a.weights && !a.gpstage;
    float2* gwin = a.gwin ? a.gwin + size_t(it) * WN * WN : nullptr;
    const bool want_obj = (a.want & WANT_OBJ) && gwin != nullptr;
    double gy = 0.0, gx = 0.0, gw = 0.0;
    // inverse row transforms of mode m from the work frame, conjugate multiplies,
    // probe-side gradients; the patch gradient summed over the modes so far stays in G
    // until the last one, whose rows give the window gradient and position terms
    const auto adjoint_rows = [&](int m, bool first, bool lastj) {
      const BufFrame stage(a.gpstage ? a.gpstage + (size_t(k) * M + m) * NN : Fr, NN * 8);
      // fy h of the previous group's last row (HREG; lanes 48..63)
      float2 hp[HREG ? N2 + 1 : 1];
      if constexpr (HREG) {
#pragma unroll
        for (int i = 0; i <= N2; ++i) hp[i] = make_float2(0.f, 0.f);
      }
#pragma unroll 1
      for (int gi = 0; gi < GPW; ++gi) {
        const int rg = wave * GPW + gi;
        float2 g[N2];
        {
          float2 v[N2];
          const int vl = opaque(v_lin0);
#pragma unroll
          for (int i = 0; i < N2; ++i) v[i] = fr.ld(lin_v(vl, i), lin_s(rg, i));
          WL::inverse(ex, tws, tr, tq, r, n1, v, g);
        }
#pragma unroll
        for (int i = 0; i < N2; i += 2) swap_pair(g[i], g[i + 1]);
#pragma unroll
        for (int i0 = 0; i0 < N2 / 2; i0 += BP) {
          const int b0 = 2 * i0;
          float2 gP[BAT], P[BAT];
          patch_batch(rg, i0, gP);
#pragma unroll
          for (int j = 0; j < BAT; ++j) {
            g[b0 + j] = cscale(g[b0 + j], inv_n);
            gP[j] = cmulc(gP[j], g[b0 + j]);
            pin(gP[j]);
          }
          // each eigenprobe pixel is read once, for the probe and for the weight-gradient
          // term Re<gP, U_e,m>
          probe_batch(m, rg, i0, P, [&](int e, const float4(&u)[BP]) {
            if (!want_w) return;
            float tf = 0.f;
#pragma unroll
            for (int j = 0; j < BP; ++j) tf += cdotre(gP[2 * j], lo2(u[j])) + cdotre(gP[2 * j + 1], hi2(u[j]));
            if (a.E == 1) {
              gw += double(tf);
            } else {
              const double t = wave_sum(double(tf));
              if (lane == 0) sh.wred[e * NW + wave] += t;
            }
          });
#pragma unroll
          for (int j = 0; j < BAT; ++j) {
            g[b0 + j] = cmulc(P[j], g[b0 + j]);
            pin(g[b0 + j]);
          }
          if (!first) {
            const int vl = opaque(v_lin0);
#pragma unroll
            for (int j = 0; j < BAT; ++j) P[j] = gb.ld(lin_v(vl, b0 + j), lin_s(rg, b0 + j));
#pragma unroll
            for (int j = 0; j < BAT; ++j) g[b0 + j] = cadd(g[b0 + j], P[j]);
          }
          if (!lastj) {
            const int vl = opaque(v_lin0);
#pragma unroll
            for (int j = 0; j < BAT; ++j) gb.st(g[b0 + j], lin_v(vl, b0 + j), lin_s(rg, b0 + j));
          }
          if (a.gpstage) {
            const int vn = opaque(v_nat0);
#pragma unroll
            for (int j = 0; j < BP; ++j)
              stage.st2(cat2(gP[2 * j], gP[2 * j + 1]), vn + (i0 + j) * 256, rg * 4 * N * 8);
          } else if (PH == 0 && want_probe) {
            for (int e = 0; e < a.E; ++e) {
              const BufFrame acc(pacc + (size_t(e) * M + m) * NN, NN * 8);
              const float w = wk[e];
              const int vn = opaque(v_nat0);
              float4 s[BP];
#pragma unroll
              for (int j = 0; j < BP; ++j) s[j] = make_float4(0.f, 0.f, 0.f, 0.f);
              if (!acc_fresh) {
#pragma unroll
                for (int j = 0; j < BP; ++j) s[j] = acc.ld2(vn + (i0 + j) * 256, rg * 4 * N * 8);
              }
#pragma unroll
              for (int j = 0; j < BP; ++j) {
                s[j].x = fmaf(w, gP[2 * j].x, s[j].x);
                s[j].y = fmaf(w, gP[2 * j].y, s[j].y);
                s[j].z = fmaf(w, gP[2 * j + 1].x, s[j].z);
                s[j].w = fmaf(w, gP[2 * j + 1].y, s[j].w);
                acc.st2(s[j], vn + (i0 + j) * 256, rg * 4 * N * 8);
              }
            }
          }
          __builtin_amdgcn_sched_barrier(0);
        }
        if (lastj && (want_obj || want_pos)) {
          // Window rows of this group: the transpose of the bilinear gather, along x
          // (h = (1 - fx) g[x] + fx g[x - 1], x = 0..N) and then along y
          // ((1 - fy) h[y] + fy h[y - 1]). A pair's left neighbour is the lane to the left
          // (lane 0: lane 15's previous pair), the row above another lane of the wave. fy h of
          // the group's last row belongs to the next group's first window row: it stays in
          // registers (512^2), or is written there and read back by the wave's next group (256^2:
          // 128 registers a thread, which the next transform would spill: 3.38 against 2.97 ms
          // at 2500 positions of 8 eigenprobes); after the wave's last group it is left in LDS for the
          // next wave.
          float2 left = make_float2(0.f, 0.f);
          float fy = 0.f, fx = 0.f;  // the terms of four pixels per thread in FP32, then FP64
          const int up_lane = ((lane + 48) & 63) * 4;
          // a window column of this row: position terms of h and of the difference d along x
          // against the object, then the window value
          const auto pos_terms = [&](float2 A0, float2 A1, float2 h, float2 d) {
            float2 ax;
            ax.x = fmaf(p.fy, A1.x, (1.f - p.fy) * A0.x);
            ax.y = fmaf(p.fy, A1.y, (1.f - p.fy) * A0.y);
            fy += cdotre(h, csub(A1, A0));
            fx += cdotre(d, ax);
          };
          const auto window_value = [&](int i, float2 h, float2 above) {
            float2 s = h;
            if constexpr (HREG) {
              if (lane >= 48) s = hp[i];
              hp[i] = h;
            }
            float2 up;
            up.x = __builtin_bit_cast(float, __builtin_amdgcn_ds_bpermute(up_lane, __builtin_bit_cast(int, s.x)));
            up.y = __builtin_bit_cast(float, __builtin_amdgcn_ds_bpermute(up_lane, __builtin_bit_cast(int, s.y)));
            const bool in = HREG || r > 0;
            float2 o;
            o.x = fmaf(1.f - p.fy, h.x, in ? p.fy * up.x : above.x);
            o.y = fmaf(1.f - p.fy, h.y, in ? p.fy * up.y : above.y);
            return o;
          };
          const bool carry = !HREG && gi < GPW - 1, to_lds = gi == GPW - 1;
          const BufFrame wb(want_obj ? gwin + size_t(rg) * 4 * WN : G, 5 * WN * 8);
          const int orow = opaque(v_win0), wrow = opaque((r * WN + 2 * q) * 8);
          constexpr int WB = 2;  // pairs at a time
#pragma unroll
          for (int i0 = 0; i0 < N2 / 2; i0 += WB) {
            float2 h[2 * WB], d[2 * WB];
#pragma unroll
            for (int j = 0; j < 2 * WB; j += 2) {
              const float2 x0 = g[2 * i0 + j], x1 = g[2 * i0 + j + 1];
              const float2 xl = row_dpp<0x111>(left, x1);
              left = row_dpp<0x121>(left, x1);
              h[j].x = fmaf(p.fx, xl.x, (1.f - p.fx) * x0.x);
              h[j].y = fmaf(p.fx, xl.y, (1.f - p.fx) * x0.y);
              h[j + 1].x = fmaf(p.fx, x0.x, (1.f - p.fx) * x1.x);
              h[j + 1].y = fmaf(p.fx, x0.y, (1.f - p.fx) * x1.y);
              d[j] = csub(xl, x0);
              d[j + 1] = csub(x0, x1);
            }
            if (want_pos) {
              float4 A0[WB], A1[WB];
#pragma unroll
              for (int j = 0; j < WB; ++j) {
                A0[j] = win.ld2(orow + (i0 + j) * 256, rg * 4 * a.W * 8);
                A1[j] = win.ld2(orow + (i0 + j) * 256, (rg * 4 + 1) * a.W * 8);
              }
#pragma unroll
              for (int j = 0; j < WB; ++j) {
                pos_terms(lo2(A0[j]), lo2(A1[j]), h[2 * j], d[2 * j]);
                pos_terms(hi2(A0[j]), hi2(A1[j]), h[2 * j + 1], d[2 * j + 1]);
              }
              gy += double(fy);
              gx += double(fx);
              fy = fx = 0.f;
            }
            if (want_obj) {
              float4 above[WB];
#pragma unroll
              for (int j = 0; j < WB; ++j) above[j] = make_float4(0.f, 0.f, 0.f, 0.f);
              if (!HREG && gi > 0 && r == 0) {
#pragma unroll
                for (int j = 0; j < WB; ++j) above[j] = wb.ld2(wrow + (i0 + j) * 256, 0);
              }
#pragma unroll
              for (int j = 0; j < WB; ++j)
                wb.st2(cat2(window_value(2 * (i0 + j), h[2 * j], lo2(above[j])),
                            window_value(2 * (i0 + j) + 1, h[2 * j + 1], hi2(above[j]))),
                       wrow + (i0 + j) * 256, 0);
              if (r == 3 && (carry || to_lds)) {
#pragma unroll
                for (int j = 0; j < WB; ++j) {
                  const float2 n0 = cscale(h[2 * j], p.fy), n1 = cscale(h[2 * j + 1], p.fy);
                  if (carry) {
                    wb.st2(cat2(n0, n1), wrow + (i0 + j) * 256, WN * 8);
                  } else {
                    ex[2 * q + 32 * (i0 + j)] = n0;
                    ex[2 * q + 32 * (i0 + j) + 1] = n1;
                  }
                }
              }
            }
            __builtin_amdgcn_sched_barrier(0);
          }
          // column N, held by lane 0 of each row
          const float2 h = q == 0 ? cscale(left, p.fx) : make_float2(0.f, 0.f);
          if (want_pos && q == 0)
            pos_terms(win.ld(orow + N * 8, rg * 4 * a.W * 8), win.ld(orow + N * 8, (rg * 4 + 1) * a.W * 8), h, left);
          if (want_obj) {
            float2 above = make_float2(0.f, 0.f);
            if (!HREG && gi > 0 && lane == 0) above = wb.ld(wrow + N * 8, 0);
            const float2 o = window_value(N2, h, above);
            if (q == 0) wb.st(o, wrow + N * 8, 0);
            if (lane == 48 && (carry || to_lds)) {
              if (carry) wb.st(cscale(h, p.fy), wrow + N * 8, WN * 8);
              else ex[N] = cscale(h, p.fy);
            }
          }
          gy += double(fy);
          gx += double(fx);
        }
      }
      if (lastj && want_obj) {
        // rows the waves share: fy h of a wave's last row goes to the next wave's first
        // window row (or row N of the window)
        __syncthreads();
        if (wave > 0) {
          float2* w0 = gwin + size_t(wave) * GPW * 4 * WN;
          for (int x = lane; x < WN; x += WAVE) w0[x] = cadd(w0[x], sh.ex[wave - 1][x]);
        }
        if (wave == NW - 1) {
          float2* w0 = gwin + size_t(N) * WN;
          for (int x = lane; x < WN; x += WAVE) w0[x] = ex[x];
        }
      }
    };

    if constexpr (PH == 2) {
      // per mode of the group: the stored far field scaled by 2 dl/dI / (K_norm N^2) of the
      // loss pass and transformed back, then the inverse rows
      const BufFrame cfrb(a.cfr + size_t(k) * NN, NN * 4);
      for (int m = m0; m < m1; ++m) {
        if (m > m0) __syncthreads();  // the previous mode's rows are read
        const BufFrame far(a.far + (size_t(k) * M + m) * NN, NN * 8);
#pragma unroll 1
        for (int gi = 0; gi < GPW; ++gi) {
          const int cg = gi * NW + wave;
          float2 u[N2], v[N2];
          const int vl = opaque(v_lin0), vf = opaque(lane * 4);
#pragma unroll
          for (int i = 0; i < N2; ++i)
            v[i] = cscale(far.ld(lin_v(vl, i), lin_s(cg, i)), cfrb.ldf(linf_v(vf, i), linf_s(cg, i)));
          WL::inverse(ex, tws, cc, cq, cc, cq, v, u);
          cols_store(cg, u);
        }
        __syncthreads();
        adjoint_rows(m, m == m0, m == m1 - 1);
      }
    } else {
      // forward + adjoint starts with the last mode, whose inverse column transforms the
      // column pass has already done
      for (int jm = 0; jm < M; ++jm) {
        const int m = fa ? (jm == 0 ? M - 1 : jm - 1) : jm;
        const bool first = jm == 0, lastj = jm == M - 1;
        if (!(fa && first)) {
          // inverse column transforms of the scaled far field (or of the given far field)
          const BufFrame src(Ps + size_t(m) * NN, NN * 8);
          if (!first) __syncthreads();  // the previous mode's rows are read
#pragma unroll 1
          for (int gi = 0; gi < GPW; ++gi) {
            const int cg = gi * NW + wave;
            float2 u[N2], v[N2];
            if (fa) {
              const int vl = opaque(v_lin0), vf = opaque(lane * 4);
#pragma unroll
              for (int i = 0; i < N2; ++i)
                v[i] = cscale(src.ld(lin_v(vl, i), lin_s(cg, i)), a.gscale * cfb.ldf(linf_v(vf, i), linf_s(cg, i)));
            } else {
              const float2* y = a.Y + (size_t(k) * M + m) * NN + cq * N + 4 * cg + cc;
#pragma unroll
              for (int i = 0; i < N2; ++i) v[i] = y[i * 16 * N];
            }
            WL::inverse(ex, tws, cc, cq, cc, cq, v, u);
            cols_store(cg, u);
          }
        }
        __syncthreads();
        adjoint_rows(m, first, lastj);
      }
    }
    acc_fresh = false;  // every accumulator frame holds this position's terms now

    if (want_pos && a.pos_part) {
      double v[2] = {gy, gx};
      block_sum_n<T, 2>(v, red);
      if (tid == 0) {
        a.pos_part[2 * size_t(it)] = v[0];
        a.pos_part[2 * size_t(it) + 1] = v[1];
      }
    }
    if (want_w) {
      if (a.E == 1) {
        gw = block_sum<T>(gw, red);
        if (a.w_part && tid == 0) a.w_part[it] = gw;
      } else {
        __syncthreads();
        if (a.w_part && tid < a.E) {
          double t = 0.0;
          for (int j = 0; j < NW; ++j) t += sh.wred[tid * NW + j];
          a.w_part[size_t(it) * a.E + tid] = t;
        }
      }
    }
    if (tid == 0 && a.wvalid) a.wvalid[it] = 1;
  }
  if (acc_fresh) clear_acc();
}

}  // namespace ptyhip
