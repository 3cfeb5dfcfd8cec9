// The backward walk over a window (see rglru_cg_tile.h). Per tile:
//   u -> x; x to LDS (half precision, two parts) and, in bf16 parts, to memory for the weight gradients
//   p, q (matrix cores; weights from L2); a~_t and h~_{t-1} of each step from the state entering the lane's run
//   the run's reverse map, then the adjoints, latest step first: dp, dq (bf16, two parts, to LDS and memory), the direct part of dx
//   dx += [dp | dq] W (matrix cores; transposed weights from L2), du and the tap sums, the Conv1D's adjoint
// What one step's gates give that its adjoint needs again (gates, their derivatives, 1 / m) stays in registers: no transcendental
// is formed twice.
#pragma once
#include "rglru_cg_tile.h"

namespace rglru {
namespace cgt {

template <int NCT, int HOW>
__global__ void __launch_bounds__(NCT * 64) __attribute__((amdgpu_waves_per_eu(2, 2))) cg_bwd_tile_kernel(CgTileArgs a) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  constexpr int PD = HOW % AT_ANY;
  typedef Wave<NCT, (HOW >= AT_ANY)> Wv;
  constexpr int NKS = Wv::NKS;
  const unsigned id = xcd_id();
  if (id >= a.total) return;
  Wv v(a, smem, id, a.W);
  const Problem &p = a.p;
  const int lo = v.w * a.per, end = lo + a.per < a.ntile ? lo + a.per : a.ntile, H = v.H, D = v.D;
  v.load_u(end - 1);
  v.load_dy(end - 1);
  const unsigned wbytes = (unsigned)NKS * 2 * 1024;
  const __amdgpu_buffer_rsrc_t wg_rs = buf((const char *)a.wg + (size_t)(v.g * NCT + v.wv) * wbytes, wbytes),
                               wd_rs = buf((const char *)a.wd + (size_t)(v.g * NCT + v.wv) * wbytes, wbytes);
  u32x4 wq[PD][2];
  auto load_w = [&](const __amdgpu_buffer_rsrc_t &rs, int ks) __attribute__((always_inline)) {
#pragma unroll
    for (int gt = 0; gt < 2; ++gt) wq[ks % PD][gt] = __builtin_amdgcn_raw_buffer_load_b128(rs, (unsigned)v.lane * 16, (unsigned)(ks * 2 + gt) * 1024, 0);
  };
  // the state in front of the window (lower lane half: the windows before it) and the adjoint's behind it (upper half: those after it)
  float2 h_win, eps;
  {
    float2 s = make_float2(0.f, 0.f);
    if (v.hf) s = a.init[(size_t)v.b * H + v.h];
    else if (p.h0) s = make_float2(p.h0[(size_t)v.b * D + v.h], p.h0[(size_t)v.b * D + H + v.h]);
    const int n = v.hf ? a.W - 1 - v.w : v.w, most = v.w > a.W - 1 - v.w ? v.w : a.W - 1 - v.w;
    for (int k = 0; k < most; k += 4) {
      float4 q[4];
      float2 e[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int kk = k + i < n ? k + i : 0;
        const size_t o = ((size_t)v.b * a.W + (v.hf ? a.W - 1 - kk : kk)) * H + v.h;
        q[i] = a.wagg[o];
        e[i] = a.wrev[o];
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float2 t = madd(make_float2(q[i].x, v.hf ? -q[i].y : q[i].y), s, v.hf ? e[i] : make_float2(q[i].z, q[i].w));
        if (k + i < n) s = t;
      }
    }
    both2(s, h_win, eps);
  }
  float s_ba = 0.f, s_bx = 0.f, s_lam = 0.f, s_th = 0.f, s_tap[2][4], s_cb[2], nx[2][3];
#pragma unroll
  for (int part = 0; part < 2; ++part) {
#pragma unroll
    for (int k = 0; k < 4; ++k) s_tap[part][k] = 0.f;
#pragma unroll
    for (int k = 0; k < 3; ++k) nx[part][k] = 0.f;   // first three rows of dx of the tile behind
    s_cb[part] = 0.f;
  }

  for (int tile = end - 1; tile >= lo; --tile) {
    // (the tile's loads have landed; only the stores of du behind them may still be under way)
    if (tile == end - 1) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    else asm volatile("s_waitcnt vmcnt(4)" ::: "memory");
#pragma unroll
    for (int ks = 0; ks < PD; ++ks) load_w(wg_rs, ks);
    const float4 run = a.run[(((size_t)v.b * a.ntile + tile) * 2 + v.hf) * H + v.h];
    if (tile == 0 && p.state_in) v.ring_rows();
    const int nrow = v.rows(tile);
    const bool ragged = nrow < 32;
    const int valid = nrow - v.hf * 16;   // of this lane's steps
    float x[2][16];
#pragma unroll
    for (int part = 0; part < 2; ++part) {
      unsigned hi[8], low[8];
      v.conv(part, x[part], hi, low);
      if (ragged) {   // nothing of the steps past the end
#pragma unroll
        for (int r = 0; r < 16; ++r)
          if (r >= valid) x[part][r] = 0.f;
#pragma unroll
        for (int q = 0; q < 8; ++q) {
          const unsigned keep = valid - 2 * q > 1 ? ~0u : valid - 2 * q == 1 ? 0xffffu : 0u;
          hi[q] &= keep;
          low[q] &= keep;
        }
      }
      v.put16(v.my + X + part * 2048, hi);
      v.put16(v.my + X + 4096 + part * 2048, low);
    }
    lds_barrier();   // x is there
    f32x16 ap, aq;
    {
      const f32x4 c = v.gate_consts();
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        ap[r] = c[0];
        aq[r] = c[1];
      }
      u32x4 fh[2], fl[2];
      fh[0] = v.frag_at(0, false);
      fl[0] = v.frag_at(0, true);
#pragma unroll
      for (int ks = 0; ks < NKS; ++ks) {
        if (ks + 1 < NKS) {
          fh[(ks + 1) & 1] = v.frag_at(ks + 1, false);
          fl[(ks + 1) & 1] = v.frag_at(ks + 1, true);
        }
        const f16x8 h8 = __builtin_bit_cast(f16x8, fh[ks & 1]), l8 = __builtin_bit_cast(f16x8, fl[ks & 1]);
        const f16x8 wa = __builtin_bit_cast(f16x8, wq[ks % PD][0]), wx = __builtin_bit_cast(f16x8, wq[ks % PD][1]);
        ap = __builtin_amdgcn_mfma_f32_32x32x16_f16(h8, wa, ap, 0, 0, 0);
        aq = __builtin_amdgcn_mfma_f32_32x32x16_f16(h8, wx, aq, 0, 0, 0);
        ap = __builtin_amdgcn_mfma_f32_32x32x16_f16(l8, wa, ap, 0, 0, 0);
        aq = __builtin_amdgcn_mfma_f32_32x32x16_f16(l8, wx, aq, 0, 0, 0);
        if (ks + PD < NKS) load_w(wg_rs, ks + PD);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    // Steps past the end: closed gates, a_t = 1 and m_t i_t = 0, let eps pass; with x and h_{t-1} taken as zero they add nothing
    if (ragged)
#pragma unroll
      for (int r = 0; r < 16; ++r)
        if (r >= valid) ap[r] = aq[r] = -__builtin_huge_valf();
    // (behind the loads of the weights, whose waits would take in these stores)
#pragma unroll
    for (int part = 0; part < 2; ++part) {
      unsigned hi[8], low[8];
#pragma unroll
      for (int q = 0; q < 8; ++q) split_bf16(x[part][2 * q], x[part][2 * q + 1], hi[q], low[q]);
      v.run_out(hi, a.xF[0], tile, part);
      v.run_out(low, a.xF[1], tile, part);
    }
    // ---- the gates of each step and the state in front of it
    float ax[16], ay[16], hx[16], hy[16], rg[16], rc[16], gn[16], ir[16], ic[16];
    float rsum = 0.f;
    {
      Decay dk;
      dk.l2 = v.gate_consts()[2];
      dk.rev = v.gate_consts()[3];
      float2 s = madd(make_float2(run.x, run.y), h_win, make_float2(run.z, run.w));
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const float ep = gate_exp(ap[r]), eq = gate_exp(aq[r]);
        rg[r] = __builtin_amdgcn_rcpf(1.f + ep);
        rc[r] = ep * rg[r] * rg[r];                      // r (1 - r), no cancellation when saturated
        const float ig = __builtin_amdgcn_rcpf(1.f + eq);
        ic[r] = eq * ig;                                 // 1 - i
        float l2, mod;
        const float2 c = cdecay(dk, rg[r], l2, mod);
        const float m2 = fmaxf(one_minus_mod2(mod, l2), 1e-30f), rs = __builtin_amdgcn_rsqf(m2);
        gn[r] = m2 * rs * ig;
        ir[r] = ig * rs * (mod * mod);                   // i |a~|^2 / m
        rsum += rg[r];
        ax[r] = c.x;
        ay[r] = c.y;
        hx[r] = s.x;
        hy[r] = s.y;
        s = madd(c, s, make_float2(gn[r] * x[0][r], gn[r] * x[1][r]));
        if (r % 4 == 3) __builtin_amdgcn_sched_barrier(0);
      }
      if (ragged)
#pragma unroll
        for (int r = 0; r < 16; ++r)
          if (r >= valid) hx[r] = hy[r] = 0.f;
    }
    u32x2 dq4[2];   // dy of four steps
    auto dy4 = [&](int r) __attribute__((always_inline)) {
#pragma unroll
      for (int part = 0; part < 2; ++part) dq4[part] = lds_tr(v.my + S + part * 2048 + v.r_rd + (unsigned)(r & ~3) * 64);
    };
    auto dyr = [&](int r) __attribute__((always_inline)) { return (r & 1) ? bf_hi(dq4[0][(r & 3) >> 1]) : bf_lo(dq4[0][(r & 3) >> 1]); };
    auto dyi = [&](int r) __attribute__((always_inline)) { return (r & 1) ? bf_hi(dq4[1][(r & 3) >> 1]) : bf_lo(dq4[1][(r & 3) >> 1]); };
    // ---- the run's reverse map: what the upper half hands to the lower one
    float2 e;
    {
      float2 R = make_float2(0.f, 0.f);
#pragma unroll
      for (int r = 15; r >= 0; --r) {
        if ((r & 3) == 3) dy4(r);
        R = cmul(make_float2(ax[r], -ay[r]), make_float2(dyr(r) + R.x, dyi(r) + R.y));
      }
      Decay dk;
      dk.l2 = v.gate_consts()[2];
      dk.rev = v.gate_consts()[3];
      const float2 A = conj2(run_decay(dk, rsum));
      float2 A_lo, A_up, R_lo, R_up;
      both2(A, A_lo, A_up);
      both2(R, R_lo, R_up);
      e = v.hf ? eps : madd(A_up, eps, R_up);
    }
    lds_barrier();   // (every wave has read x)
    // ---- the adjoints, latest step first
    f32x16 dx[2];
    const f32x4 more = v.con4(12);
    const float cls = more[2], cth = more[3];   // c log(sigma(Lambda)), c theta
    unsigned pk[4][8];   // dp, dq high; dp, dq low
    float dpv[2], dqv[2];
    u32x4 xh[2], xl[2];   // x of eight steps, from its two parts in LDS
    auto dot_x = [&](int part, int r, float d, float s) __attribute__((always_inline)) {   // s + d x
      const unsigned h = xh[part][(r & 7) >> 1], l = xl[part][(r & 7) >> 1];
      return (r & 1) ? fmaf(f16_hi(h), d, fmaf(f16_hi(l), d, s)) : fmaf(f16_lo(h), d, fmaf(f16_lo(l), d, s));
    };
#pragma unroll
    for (int r = 15; r >= 0; --r) {
      if ((r & 7) == 7)
#pragma unroll
        for (int part = 0; part < 2; ++part) {
          xh[part] = v.get8(v.my + X + part * 2048, r >> 3);
          xl[part] = v.get8(v.my + X + 4096 + part * 2048, r >> 3);
        }
      if ((r & 3) == 3) dy4(r);
      const float dlx = dyr(r) + e.x, dly = dyi(r) + e.y;
      const float Gr = fmaf(dlx, hx[r], dly * hy[r]), Gi = fmaf(dly, hx[r], -dlx * hy[r]);
      const float sx = dot_x(0, r, dlx, dot_x(1, r, dly, 0.f));   // dL/d(m_t i_t)
      const float dlm = fmaf(Gr, ax[r], fmaf(Gi, ay[r], -sx * ir[r]));
      const float dph = fmaf(Gi, ax[r], -Gr * ay[r]);
      dpv[r & 1] = fmaf(dlm, cls, dph * cth) * rc[r];
      dqv[r & 1] = sx * gn[r] * ic[r];
      s_ba += dpv[r & 1];
      s_bx += dqv[r & 1];
      s_lam = fmaf(dlm, rg[r], s_lam);
      s_th = fmaf(dph, rg[r], s_th);
      dx[0][r] = dlx * gn[r];
      dx[1][r] = dly * gn[r];
      e = cmul(make_float2(ax[r], -ay[r]), make_float2(dlx, dly));
      if ((r & 1) == 0) {
        split_bf16(dpv[0], dpv[1], pk[0][r >> 1], pk[2][r >> 1]);
        split_bf16(dqv[0], dqv[1], pk[1][r >> 1], pk[3][r >> 1]);
      }
      if ((r & 3) == 0) {
        asm volatile("" : "+v"(s_ba), "+v"(s_bx), "+v"(s_lam), "+v"(s_th));   // (summed here; the compiler would keep the terms for later)
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    {   // the adjoint in front of the tile: the lower half's
      float2 up;
      both2(e, eps, up);
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) v.put16(v.my + X + k * 2048, pk[k]);
#pragma unroll
    for (int ks = 0; ks < PD; ++ks) load_w(wd_rs, ks);
    lds_barrier();   // dp, dq are there
    {
      u32x4 fh[2], fl[2];
      fh[0] = v.frag_at(0, false);
      fl[0] = v.frag_at(0, true);
#pragma unroll
      for (int ks = 0; ks < NKS; ++ks) {
        if (ks + 1 < NKS) {
          fh[(ks + 1) & 1] = v.frag_at(ks + 1, false);
          fl[(ks + 1) & 1] = v.frag_at(ks + 1, true);
        }
        const bf16x8 h8 = __builtin_bit_cast(bf16x8, fh[ks & 1]), l8 = __builtin_bit_cast(bf16x8, fl[ks & 1]);
#pragma unroll
        for (int part = 0; part < 2; ++part)
          dx[part] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(h8, __builtin_bit_cast(bf16x8, wq[ks % PD][part]), dx[part], 0, 0, 0);
#pragma unroll
        for (int part = 0; part < 2; ++part)
          dx[part] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(l8, __builtin_bit_cast(bf16x8, wq[ks % PD][part]), dx[part], 0, 0, 0);
        if (ks + PD < NKS) load_w(wd_rs, ks + PD);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    unsigned ul[2][10];
#pragma unroll
    for (int part = 0; part < 2; ++part) v.template rows_of<5>(v.my + U + part * U_PART, ul[part]);
    // dp, dq for the weight gradients: behind the weights' loads, too
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      unsigned o[8];
#pragma unroll
      for (int n = 0; n < 2; ++n) {
        const u32x4 q = v.get8(v.my + X + k * 2048, n);
#pragma unroll
        for (int i = 0; i < 4; ++i) o[4 * n + i] = q[i];
      }
      v.run_out(o, a.pqF[k >> 1], tile, k & 1);
    }
    lds_barrier();   // (every wave has read dp and dq; u is in registers)
    // a window's first and last three rows: du there takes both sides
    if (a.edge && v.ok && (tile == lo || tile == end - 1)) {
      float *to = a.edge + ((size_t)v.b * a.W + v.w) * 6 * D + v.h;
#pragma unroll
      for (int part = 0; part < 2; ++part)
#pragma unroll
        for (int r = 0; r < 3; ++r) {
          if (tile == lo && !v.hf) to[(size_t)r * D + part * H] = dx[part][r];
          if (tile == end - 1 && v.hf) to[(size_t)(3 + r) * D + part * H] = dx[part][13 + r];
        }
    }
    if (tile > lo) {
      v.load_u(tile - 1);
      v.load_dy(tile - 1);
    }
    // ---- the Conv1D's adjoint
#pragma unroll
    for (int part = 0; part < 2; ++part) {
      const f32x4 tap = v.taps(part);
      float xx[19];
#pragma unroll
      for (int r = 0; r < 16; ++r) xx[r] = dx[part][r];
#pragma unroll
      for (int r = 0; r < 3; ++r) {
        float l, u;
        both_halves(dx[part][r], l, u);
        xx[16 + r] = v.hf ? nx[part][r] : u;
        nx[part][r] = l;
      }
      unsigned o[8];
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        float d[2];
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          const int r = 2 * q + i;
          d[i] = tap[0] * xx[r];
#pragma unroll
          for (int k = 1; k < 4; ++k) d[i] = fmaf(tap[k], xx[r + k], d[i]);
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            const int n = r - k + 4;
            s_tap[part][k] = fmaf(xx[r], (n & 1) ? bf_hi(ul[part][n >> 1]) : bf_lo(ul[part][n >> 1]), s_tap[part][k]);
          }
          s_cb[part] += xx[r];
        }
        o[q] = pack_bf16(d[0], d[1]);
        if (q & 1) __builtin_amdgcn_sched_barrier(0);
      }
      v.put16(v.my + X + part * 2048, o);
    }
    wave_lds_fence();
    v.rows_out(v.my + X, p.du, tile, 0);
    v.rows_out(v.my + X + 2048, p.du, tile, 1);
    wave_lds_fence();
  }
  // ---- sums of this workgroup (both lane halves hold the same channel)
  float sum[14] = {s_ba, s_bx, s_lam, s_th, s_tap[0][0], s_tap[0][1], s_tap[0][2], s_tap[0][3], s_cb[0],
                   s_tap[1][0], s_tap[1][1], s_tap[1][2], s_tap[1][3], s_cb[1]};
#pragma unroll
  for (int k = 0; k < 14; ++k) sum[k] += __shfl_xor(sum[k], 32);
  if (v.hf || !v.ok) return;
  const size_t bw = (size_t)v.b * a.W + v.w;
  float *pa = a.partA + bw * 4 * H + v.h, *pc = a.partC + bw * 5 * D + v.h;
  pa[0] = sum[0];
  pa[H] = sum[1];
  pa[2 * (size_t)H] = sum[2] * (p.c / (1.f + expf(p.Lambda[v.h])));   // c d log sigmoid(Lambda) / d Lambda
  pa[3 * (size_t)H] = sum[3] * p.c;
#pragma unroll
  for (int part = 0; part < 2; ++part)
#pragma unroll
    for (int k = 0; k < 5; ++k) pc[(size_t)k * D + part * H] = sum[4 + 5 * part + k];
  if (v.w == 0 && p.dh0) {
    p.dh0[(size_t)v.b * D + v.h] = eps.x;
    p.dh0[(size_t)v.b * D + H + v.h] = eps.y;
  }
}

}  // namespace cgt
}  // namespace rglru
