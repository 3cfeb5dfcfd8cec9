// The forward walk over a window (see rglru_cg_tile.h): its map (M_AGG), its maps in both directions and those of its runs (M_BAGG),
// or y from the true state (M_Y). The block's weights stay in registers: a wave's 32 outputs of both gates are 128 of them for 128
// channels, and two waves per SIMD have 256. (Streamed from L2, with three workgroups to a compute unit: 109, 114 and 120 us instead of
// 80, 93 and 97 at B 8 T 2048, 10 blocks of 128.)
#pragma once
#include "rglru_cg_tile.h"

namespace rglru {
namespace cgt {

constexpr int M_AGG = 0, M_BAGG = 1, M_Y = 2;

template <int NCT, int HOW>
__global__ void __launch_bounds__(NCT * 64) __attribute__((amdgpu_waves_per_eu(2, 2))) cg_tile_kernel(CgTileArgs a) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  constexpr int MODE = HOW % AT_ANY;
  typedef Wave<NCT, (HOW >= AT_ANY)> Wv;
  constexpr int NKS = Wv::NKS;
  const unsigned id = xcd_id();
  if (id >= a.total) return;
  Wv v(a, smem, id, MODE == M_AGG ? a.W - 1 : a.W);
  const Problem &p = a.p;
  const int lo = v.w * a.per, end = lo + a.per < a.ntile ? lo + a.per : a.ntile, H = v.H;
  v.load_u(lo);
  if (MODE == M_BAGG) v.load_dy(lo);
  f16x8 wq[NKS][2];
  {
    const unsigned wbytes = (unsigned)NKS * 2 * 1024;
    const __amdgpu_buffer_rsrc_t rs = buf((const char *)a.wg + (size_t)(v.g * NCT + v.wv) * wbytes, wbytes);
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks)
#pragma unroll
      for (int gt = 0; gt < 2; ++gt)
        wq[ks][gt] = __builtin_bit_cast(f16x8, __builtin_amdgcn_raw_buffer_load_b128(rs, (unsigned)v.lane * 16, (unsigned)(ks * 2 + gt) * 1024, 0));
  }
  const size_t bh = (size_t)v.b * H + v.h;
  float2 Aw = make_float2(1.f, 0.f), Ew = make_float2(0.f, 0.f), Rw = Ew;   // the window's maps; M_Y: Ew is the state
  if (MODE == M_Y) {
    float2 h0 = make_float2(0.f, 0.f);
    if (a.W > 1) h0 = a.init[bh];
    else if (p.h0) h0 = make_float2(p.h0[(size_t)v.b * v.D + v.h], p.h0[(size_t)v.b * v.D + H + v.h]);
    // the maps of the windows in front: each lane half composes half of them
    const int m = (v.w + 1) >> 1, k0 = v.hf ? m : 0, k1 = v.hf ? v.w : m;
    const float4 *ag = a.wagg + (size_t)v.b * a.W * H + v.h;
    for (int k = 0; k < m; k += 8) {
      float4 q[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) q[e] = ag[(size_t)(k0 + k + e < k1 ? k0 + k + e : k0) * H];
#pragma unroll
      for (int e = 0; e < 8; ++e)
        if (k0 + k + e < k1) cthen(Aw, Ew, make_float2(q[e].x, q[e].y), make_float2(q[e].z, q[e].w));
    }
    float2 A_lo, A_up, E_lo, E_up;
    both2(Aw, A_lo, A_up);
    both2(Ew, E_lo, E_up);
    Ew = madd(A_up, madd(A_lo, h0, E_lo), E_up);
  } else if (v.w == 0 && v.hf == 0 && v.ok) {   // (the next kernel's outputs may take their place)
    const float *from = MODE == M_BAGG ? p.dhT : p.h0;
    a.init[bh] = from ? make_float2(from[(size_t)v.b * v.D + v.h], from[(size_t)v.b * v.D + H + v.h]) : make_float2(0.f, 0.f);
  }

  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
#pragma unroll
  for (int ks = 0; ks < NKS; ++ks)
#pragma unroll
    for (int gt = 0; gt < 2; ++gt) asm volatile("" : "+v"(wq[ks][gt]));   // (resident, not loaded again in the loop)

  for (int tile = lo; tile < end; ++tile) {
    // (the tile's loads have landed; only what was stored behind them may still be under way)
    if (tile > lo) {
      if (MODE == M_Y) asm volatile("s_waitcnt vmcnt(4)" ::: "memory");
      else if (MODE == M_BAGG) asm volatile("s_waitcnt vmcnt(1)" ::: "memory");
      else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    }
    if (tile == 0 && p.state_in) v.ring_rows();
    float x[2][16];
    {
      unsigned hi[2][8], low[2][8];
#pragma unroll
      for (int part = 0; part < 2; ++part) v.conv(part, x[part], hi[part], low[part]);
      lds_barrier();   // (every wave has read the last tile's x)
#pragma unroll
      for (int part = 0; part < 2; ++part) {
        v.put16(v.my + X + part * 2048, hi[part]);
        v.put16(v.my + X + 4096 + part * 2048, low[part]);
      }
    }
    if (tile + 1 < end) v.load_u(tile + 1);
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
        ap = __builtin_amdgcn_mfma_f32_32x32x16_f16(h8, wq[ks][0], ap, 0, 0, 0);
        aq = __builtin_amdgcn_mfma_f32_32x32x16_f16(h8, wq[ks][1], aq, 0, 0, 0);
        ap = __builtin_amdgcn_mfma_f32_32x32x16_f16(l8, wq[ks][0], ap, 0, 0, 0);
        aq = __builtin_amdgcn_mfma_f32_32x32x16_f16(l8, wq[ks][1], aq, 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    if (v.rows(tile) < 32) {   // steps past the end: a closed gate, a_t = 1 and b_t = 0, leaves the state untouched
      const int valid = v.rows(tile) - v.hf * 16;
#pragma unroll
      for (int r = 0; r < 16; ++r)
        if (r >= valid) {
          ap[r] = aq[r] = -__builtin_huge_valf();
          x[0][r] = x[1][r] = 0.f;
        }
    }
    unsigned dr[8], di[8];
    if (MODE == M_BAGG) {
      v.template rows_of<4>(v.my + S, dr);
      v.template rows_of<4>(v.my + S + 2048, di);
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      if (tile + 1 < end) v.load_dy(tile + 1);
    }
    Decay dk;
    dk.l2 = v.gate_consts()[2];
    dk.rev = v.gate_consts()[3];
    float2 A = make_float2(1.f, 0.f), E = make_float2(0.f, 0.f), R = E;
    float rsum = 0.f;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      float l2, mod;
      const float rg = sigm(ap[r]);
      const float2 c = cdecay(dk, rg, l2, mod);
      const float gain = __builtin_amdgcn_sqrtf(fmaxf(one_minus_sq(mod, l2), 0.f)) * sigm(aq[r]);
      const float2 bb = make_float2(gain * x[0][r], gain * x[1][r]);
      E = madd(c, E, bb);
      if (MODE == M_BAGG) A = cmul(c, A);
      else rsum += rg;
      if (MODE == M_BAGG)   // the reverse map's end value: conj(a~ of all steps up to this one) dy
        R = madd(conj2(A), make_float2((r & 1) ? bf_hi(dr[r >> 1]) : bf_lo(dr[r >> 1]), (r & 1) ? bf_hi(di[r >> 1]) : bf_lo(di[r >> 1])), R);
      if (MODE == M_Y) {
        ap[r] = c.x;
        aq[r] = c.y;
        x[0][r] = bb.x;
        x[1][r] = bb.y;
      }
      if (r % 4 == 3) __builtin_amdgcn_sched_barrier(0);
    }
    if (MODE != M_BAGG) A = run_decay(dk, rsum);
    float2 A_lo, A_up, E_lo, E_up;
    both2(A, A_lo, A_up);
    both2(E, E_lo, E_up);
    const float2 At = cmul(A_up, A_lo), Et = madd(A_up, E_lo, E_up);
    if (MODE == M_Y) {
      float2 s = v.hf ? madd(A_lo, Ew, E_lo) : Ew;
      Ew = madd(At, Ew, Et);
      unsigned yr[8], yi[8];
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        const float2 s0 = madd(make_float2(ap[2 * q], aq[2 * q]), s, make_float2(x[0][2 * q], x[1][2 * q]));
        s = madd(make_float2(ap[2 * q + 1], aq[2 * q + 1]), s0, make_float2(x[0][2 * q + 1], x[1][2 * q + 1]));
        yr[q] = pack_bf16(s0.x, s.x);
        yi[q] = pack_bf16(s0.y, s.y);
      }
      v.put16(v.my + S, yr);
      v.put16(v.my + S + 2048, yi);
      wave_lds_fence();
      v.rows_out(v.my + S, p.y, tile, 0);
      v.rows_out(v.my + S + 2048, p.y, tile, 1);
      wave_lds_fence();
    } else {
      if (MODE == M_BAGG) {
        float2 R_lo, R_up;
        both2(R, R_lo, R_up);
        Rw = madd(conj2(Aw), madd(conj2(A_lo), R_up, R_lo), Rw);
        const float2 Ar = v.hf ? cmul(A_lo, Aw) : Aw, Er = v.hf ? madd(A_lo, Ew, E_lo) : Ew;
        if (v.ok) a.run[(((size_t)v.b * a.ntile + tile) * 2 + v.hf) * H + v.h] = make_float4(Ar.x, Ar.y, Er.x, Er.y);
      }
      Ew = madd(At, Ew, Et);
      Aw = cmul(At, Aw);
    }
  }
  if (v.hf || !v.ok) return;
  if (MODE == M_Y) {
    if (v.w == a.W - 1 && p.hT) {
      p.hT[(size_t)v.b * v.D + v.h] = Ew.x;
      p.hT[(size_t)v.b * v.D + H + v.h] = Ew.y;
    }
    return;
  }
  const size_t o = ((size_t)v.b * a.W + v.w) * H + v.h;
  a.wagg[o] = make_float4(Aw.x, Aw.y, Ew.x, Ew.y);
  if (MODE == M_BAGG) a.wrev[o] = Rw;
}

template <int NCT, bool ANY>
CgInstance fwd_instance() {
  constexpr int at = ANY ? AT_ANY : 0;
  return {(const void *)cg_tile_kernel<NCT, M_AGG + at>, (const void *)cg_tile_kernel<NCT, M_BAGG + at>, (const void *)cg_tile_kernel<NCT, M_Y + at>,
          nullptr, NCT};
}

}  // namespace cgt
}  // namespace rglru
