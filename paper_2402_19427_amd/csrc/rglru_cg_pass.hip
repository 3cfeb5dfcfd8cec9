// The complex-gated layer (Appendix B) in bf16 storage as passes that are parallel over time, for
// blocks of a multiple of 16 complex channels that the kernels in tiles (rglru_cg_tile.h) do not take (see rglru_pass.hip for the scheme and the staging):
//     h~_t = a~_t h~_{t-1} + b~_t            eps_t = conj(a~_t) (dy~_t + eps_{t+1})
// are affine with complex coefficients, so runs of steps are described by complex aggregates formed in
// the epilogue of the gate products and linked by a short chain. What travels keeps the accuracy the
// phases need (they add up over thousands of steps): x as a half-precision high + low part, both
// multiplied; pre-activations and dx in fp32; dp, dq as bf16 high + low parts (gradients have no
// bounded range), three products per pair in the weight gradients.
//   1. conv_rows_kernel   x (high, low)
//   2. cg_gates_kernel    pre-activations; aggregates of the runs (forward: 64 steps; backward: 16, in
//                         both directions)
//   3. cg_chain_kernel    states entering every run
//   4. cg_apply_kernel    y, hT          | cg_adjoint_kernel  dp, dq, direct part of dx, sums
//   5. cg_dgrad_kernel    dx += [dp | dq] W     6. conv_adjoint_kernel     7. cg_wgrad_kernel     8. sums
// The forward takes the time axis in chunks whose intermediates fit its scratch (and the last-level
// cache).
#include "rglru_cg_math.h"

#include <algorithm>

namespace rglru {
using namespace pass;

namespace {

constexpr int CST_A = PR * 64;              // one part (high or low) of a stage's 256 rows
constexpr int CST = 2 * CST_A + 128 * 64;   // stage: high | low | 128 rows of the other operand
constexpr int C_LDS = 2 * CST;
static_assert(C_LDS <= 80 * 1024, "two workgroups per CU");
constexpr int SUB = 16;                     // steps per run of the backward

__device__ __forceinline__ float2 swap_halves(float2 v) { return make_float2(__shfl_xor(v.x, 32), __shfl_xor(v.y, 32)); }

// ------------------------------------------------------------------------ preparation
// w16 [gate][nb][hs][2 hs] half precision; wt [nb][k of 2 hs][gate hs + j] bf16 (backward)
struct CgPrepArgs {
  const unsigned short *Wa, *Wx;
  unsigned short *w16, *wt;
  int nb, hs;
};
__global__ void __launch_bounds__(256) cg_prep_kernel(CgPrepArgs a) {
  const size_t per = (size_t)a.nb * a.hs * 2 * a.hs, i = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= 2 * per) return;
  const int gate = i >= per;
  const size_t o = i - (gate ? per : 0);
  const unsigned short w = (gate ? a.Wx : a.Wa)[o];
  a.w16[i] = (unsigned short)f16_bits(f16_range(__uint_as_float((unsigned)w << 16)));   // (finite weights stop at 65504)
  if (a.wt) {
    const int k = (int)(o % (2 * a.hs)), j = (int)(o / (2 * a.hs) % a.hs), g = (int)(o / (2 * a.hs) / a.hs);
    a.wt[((size_t)g * 2 * a.hs + k) * 2 * a.hs + gate * a.hs + j] = w;
  }
}

// ------------------------------------------------------------------------ 2. gates
struct CgGatesArgs {
  Problem p;                       // T: steps of the chunk in hand
  const unsigned short *xh, *xl;   // [B][T][D]
  const unsigned short *w16;
  float *pq;                       // [2][B][T][H] pre-activations
  float4 *agg;                     // forward: [B][runs of 64][H] (A, E), or null
  float4 *aggf, *aggr;             // backward: [B][runs of 16][H] in both directions
  int nct, nrt, nrun;
  unsigned total;
};
template <bool BWD>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2))) cg_gates_kernel(CgGatesArgs a) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const Problem &p = a.p;
  const unsigned id = xcd_id();
  if (id >= a.total) return;
  const int tid = threadIdx.x, lane = tid & 63, hf = lane >> 5, j = lane & 31;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int ct = (int)(id % a.nct), rt = (int)(id / a.nct % a.nrt), gb = (int)(id / a.nct / a.nrt);
  const int b = gb % p.B, g = gb / p.B;
  const int D = p.D, H = D / 2, T = p.T, hs = p.bs, t0 = rt * PR, tw = t0 + wv * RUN;
  const unsigned row_bytes = (unsigned)D * 2;
  // (every buffer starts at the tile: 32-bit offsets whatever the length of the sequence)
  const size_t row0 = (size_t)b * T + t0, first = row0 * D, nrow = T - t0 < PR ? T - t0 : PR, tile_bytes = nrow * row_bytes;
  const __amdgpu_buffer_rsrc_t xh_rs = buf(a.xh + first, tile_bytes), xl_rs = buf(a.xl + first, tile_bytes);
  const size_t wn = (size_t)hs * 2 * hs;
  const __amdgpu_buffer_rsrc_t w_rs[2] = {buf(a.w16 + (size_t)g * wn, wn * 2), buf(a.w16 + ((size_t)p.nb + g) * wn, wn * 2)};
  const int lrow = lane >> 2;
  const int ca = (lane & 3) ^ (((lrow >> 1) & 1) | ((wv & 1) << 1)), cb_ = (lane & 3) ^ ((lrow >> 1) & 3);
  const unsigned a_vo = (unsigned)lrow * row_bytes + (unsigned)(g * hs) * 2 + (unsigned)ca * 16;
  const unsigned wrow = (unsigned)hs * 4;
  const unsigned b_vo = (unsigned)(ct * 64 + lrow) * wrow + (unsigned)cb_ * 16;
  const int npc = (hs + 31) / 32, nkc = 2 * npc;   // steps per part: real inputs, then imaginary ones
  auto load_stage = [&](int kc, int st) __attribute__((always_inline)) {
    unsigned char *s = smem + st * CST;
    const int part = kc >= npc, kk = kc - (part ? npc : 0);
    const unsigned va = kk * 32 + ca * 8 < hs ? a_vo : OOB, vb = kk * 32 + cb_ * 8 < hs ? b_vo : OOB;
    const unsigned ka = (unsigned)(part * H * 2 + kk * 64), kb = (unsigned)(part * hs * 2 + kk * 64);
#pragma unroll
    for (int m = 0; m < 4; ++m) {
      const int i = wv + 4 * m;
      const unsigned so = (unsigned)(16 * i) * row_bytes + ka;
      lds16(xh_rs, s + i * 1024, va, so);
      lds16(xl_rs, s + CST_A + i * 1024, va, so);
    }
#pragma unroll
    for (int gate = 0; gate < 2; ++gate)
      lds16(w_rs[gate], s + 2 * CST_A + gate * 4096 + wv * 1024, vb, (unsigned)(16 * wv) * wrow + kb);
  };
  load_stage(0, 0);
  f32x16 acc[2][2][2];   // [gate][row block][channel block]
#pragma unroll
  for (int gt = 0; gt < 2; ++gt)
#pragma unroll
    for (int rb = 0; rb < 2; ++rb)
#pragma unroll
      for (int cb = 0; cb < 2; ++cb)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[gt][rb][cb][r] = 0.f;
  const int arow = perm_row(j);
  const unsigned a_rd = (unsigned)(wv * RUN + arow) * 64 + (unsigned)(hf ^ key_a(arow)) * 16;
  const unsigned b_rd = 2 * CST_A + (unsigned)j * 64 + (unsigned)(hf ^ key_b(j)) * 16;
  const bool rows_on = tw < T;
  const int ncb = hs - ct * 64 > 32 ? 2 : 1;
  for (int kc = 0; kc < nkc; ++kc) {
    stage_barrier();
    if (kc + 1 < nkc) load_stage(kc + 1, (kc + 1) & 1);
    if (!rows_on) continue;
    const unsigned char *s = smem + (kc & 1) * CST;
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      f16x8 fh[2], fl[2], fb[2][2];
#pragma unroll
      for (int rb = 0; rb < 2; ++rb) {
        fh[rb] = *(const f16x8 *)(s + ((a_rd + rb * 2048) ^ (ks * 32)));
        fl[rb] = *(const f16x8 *)(s + ((a_rd + CST_A + rb * 2048) ^ (ks * 32)));
      }
#pragma unroll
      for (int gt = 0; gt < 2; ++gt)
#pragma unroll
        for (int cb = 0; cb < 2; ++cb) fb[gt][cb] = *(const f16x8 *)(s + ((b_rd + gt * 4096 + cb * 2048) ^ (ks * 32)));
#pragma unroll
      for (int cb = 0; cb < 2; ++cb) {
        if (cb < ncb) {
#pragma unroll
          for (int gt = 0; gt < 2; ++gt)
#pragma unroll
            for (int rb = 0; rb < 2; ++rb)
              acc[gt][rb][cb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(fh[rb], fb[gt][cb], acc[gt][rb][cb], 0, 0, 0);
#pragma unroll
          for (int gt = 0; gt < 2; ++gt)
#pragma unroll
            for (int rb = 0; rb < 2; ++rb)
              acc[gt][rb][cb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(fl[rb], fb[gt][cb], acc[gt][rb][cb], 0, 0, 0);
        }
      }
    }
  }
  __syncthreads();   // the stages become the waves' own tiles
  if (!rows_on) return;
  // ---- aggregates. Per (channel block, row block) the wave fetches 32 rows x 32 channels of x (high,
  // low) and dy, real | imaginary in 128-byte rows, and reads them back transposed: lane (j, hf) has
  // steps 16 hf .. 16 hf + 15 of channel j
  unsigned char *tile = smem + wv * (C_LDS / 4);
  const int erow = lane >> 3, ec = (lane & 7) ^ ((erow & 3) * 2);
  const int i16 = lane & 15, q16 = (lane >> 4) & 1;
  const unsigned e_rd = (unsigned)(hf * 16 + (i16 >> 2)) * 128 +
                        (unsigned)((((q16 * 2) + ((i16 & 3) >> 1)) ^ (((i16 >> 2) & 3) * 2)) * 16) + (unsigned)(i16 & 1) * 8;
  auto e_read = [&](const unsigned char *t, int part, unsigned (&v)[8]) __attribute__((always_inline)) {
#pragma unroll
    for (int n = 0; n < 4; ++n) {
      const u32x2 w = lds_tr(t + ((e_rd + (unsigned)(4 * n) * 128) ^ (unsigned)(part * 64)));
      v[2 * n] = w[0];
      v[2 * n + 1] = w[1];
    }
  };
  const __amdgpu_buffer_rsrc_t dy_rs = buf((const unsigned short *)(BWD ? p.dy : (const void *)a.xh) + first, tile_bytes);
  const __amdgpu_buffer_rsrc_t p_rs = buf(a.pq + row0 * H, nrow * H * 4),
                               q_rs = buf(a.pq + ((size_t)p.B * T + row0) * H, nrow * H * 4);
#pragma unroll
  for (int cb = 0; cb < 2; ++cb) {
    if (cb >= ncb) break;
    const int ch = ct * 64 + cb * 32 + j;
    const bool ok = ch < hs;
    const int h = g * hs + (ok ? ch : hs - 1);
    const float ba = p.b_a[h], bx = p.b_x[h];
    const Decay dk(p, h);
    const int ecol = cb * 32 + (ec & 3) * 8;
    const unsigned e_vo = ct * 64 + ecol < hs
        ? (unsigned)erow * row_bytes + (unsigned)((ec >> 2) * H + g * hs + ct * 64 + ecol) * 2 : OOB;
    const unsigned o_vo = ok ? (unsigned)h * 4 + (unsigned)(hf * 16) * (unsigned)H * 4 : OOB;
    float2 At = make_float2(1.f, 0.f), Et = make_float2(0.f, 0.f);
#pragma unroll
    for (int rb = 0; rb < 2; ++rb) {
      const int tr = tw + rb * 32, lr = wv * RUN + rb * 32;   // first step, first row of the tile
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // the previous block's reads are done
#pragma unroll
      for (int m = 0; m < 4; ++m) {
        const unsigned so = (unsigned)(lr + 8 * m) * row_bytes;
        lds16(xh_rs, tile + m * 1024, e_vo, so);
        lds16(xl_rs, tile + 4096 + m * 1024, e_vo, so);
        if (BWD) lds16(dy_rs, tile + 8192 + m * 1024, e_vo, so);
      }
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        acc[0][rb][cb][r] += ba;
        acc[1][rb][cb][r] += bx;
        const unsigned so = (unsigned)(lr + r) * (unsigned)H * 4;
        __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(acc[0][rb][cb][r]), p_rs, o_vo, so, 0);
        __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(acc[1][rb][cb][r]), q_rs, o_vo, so, 0);
      }
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      unsigned rh[8], ih[8], rl[8], il[8], dr[8], di[8];
      e_read(tile, 0, rh);
      e_read(tile, 1, ih);
      e_read(tile + 4096, 0, rl);
      e_read(tile + 4096, 1, il);
      if (BWD) {
        e_read(tile + 8192, 0, dr);
        e_read(tile + 8192, 1, di);
      }
      const int nvalid = T - tr - hf * 16;
      float2 A = make_float2(1.f, 0.f), E = make_float2(0.f, 0.f), av[BWD ? 16 : 1];
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        float l2, mod;
        float2 c = cdecay(dk, sigm(acc[0][rb][cb][r]), l2, mod);
        const float gain = __builtin_amdgcn_sqrtf(one_minus_sq(mod, l2)) * sigm(acc[1][rb][cb][r]);
        const bool hi = r & 1;
        float2 bb = make_float2(gain * ((hi ? f16_hi(rh[r >> 1]) : f16_lo(rh[r >> 1])) + (hi ? f16_hi(rl[r >> 1]) : f16_lo(rl[r >> 1]))),
                                gain * ((hi ? f16_hi(ih[r >> 1]) : f16_lo(ih[r >> 1])) + (hi ? f16_hi(il[r >> 1]) : f16_lo(il[r >> 1]))));
        if (r >= nvalid) {   // steps past the end leave the state untouched
          c = make_float2(1.f, 0.f);
          bb = make_float2(0.f, 0.f);
        }
        if (BWD) av[r] = c;
        cthen(A, E, c, bb);
      }
      if (BWD) {
        // backwards: eps -> conj(a) (dy + eps)
        float2 R = make_float2(0.f, 0.f);
#pragma unroll
        for (int r = 15; r >= 0; --r) {
          const bool hi = r & 1;
          R.x += hi ? bf_hi(dr[r >> 1]) : bf_lo(dr[r >> 1]);   // (zero past the end)
          R.y += hi ? bf_hi(di[r >> 1]) : bf_lo(di[r >> 1]);
          R = cmul(make_float2(av[r].x, -av[r].y), R);
        }
        const int run = tr / SUB + hf;
        if (ok && run < a.nrun) {
          const size_t o = ((size_t)b * a.nrun + run) * H + h;
          a.aggf[o] = make_float4(A.x, A.y, E.x, E.y);
          a.aggr[o] = make_float4(A.x, -A.y, R.x, R.y);   // the product of the conjugates is the conjugate
        }
      } else {
        const float2 oA = swap_halves(A), oE = swap_halves(E);
        cthen(At, Et, hf ? oA : A, hf ? oE : E);
        cthen(At, Et, hf ? A : oA, hf ? E : oE);
      }
    }
    if (!BWD && a.agg && hf == 0 && ok)
      a.agg[((size_t)b * a.nrun + (t0 / RUN + wv)) * H + h] = make_float4(At.x, At.y, Et.x, Et.y);
  }
}

// ------------------------------------------------------------------------ 3. chain
// as chain_kernel, complex: eight segments of the runs per 32 channels; direction 1 walks backwards
struct CgChainArgs {
  const float4 *agg[2];
  const float *init[2];   // [B][D] or null
  float2 *in[2];
  float *fin[2];          // [B][D] or null
  int B, H, nrun, ncg;
};
__global__ void __launch_bounds__(256) cg_chain_kernel(CgChainArgs a) {
  __shared__ float4 seg[8][32];
  const int dir = blockIdx.y, hl = threadIdx.x & 31, sg = threadIdx.x >> 5;
  const int b = blockIdx.x / a.ncg, h = (blockIdx.x % a.ncg) * 32 + hl, hc = h < a.H ? h : a.H - 1;
  const int per = (a.nrun + 7) / 8, k0 = sg * per, k1 = k0 + per < a.nrun ? k0 + per : a.nrun;
  const float4 *ag = (dir ? a.agg[1] : a.agg[0]) + (size_t)b * a.nrun * a.H + hc;
  auto at = [&](int k) { return (size_t)(dir ? a.nrun - 1 - k : k) * a.H; };
  constexpr int U = 8;
  float2 A = make_float2(1.f, 0.f), E = make_float2(0.f, 0.f);
  for (int k = k0; k < k1; k += U) {
    float4 v[U];
#pragma unroll
    for (int e = 0; e < U; ++e) v[e] = ag[at(k + e < k1 ? k + e : k1 - 1)];
#pragma unroll
    for (int e = 0; e < U; ++e)
      if (k + e < k1) cthen(A, E, make_float2(v[e].x, v[e].y), make_float2(v[e].z, v[e].w));
  }
  seg[sg][hl] = make_float4(A.x, A.y, E.x, E.y);
  const float *init = dir ? a.init[1] : a.init[0];
  float2 s = make_float2(0.f, 0.f);   // (read in front of the barrier: fin may be the same array)
  if (init) s = make_float2(init[(size_t)b * 2 * a.H + hc], init[(size_t)b * 2 * a.H + a.H + hc]);
  __syncthreads();
  auto step = [&](const float4 &v) {
    const float2 t = cmul(make_float2(v.x, v.y), s);
    s = make_float2(t.x + v.z, t.y + v.w);
  };
  for (int w = 0; w < sg; ++w) step(seg[w][hl]);
  float2 *in = (dir ? a.in[1] : a.in[0]) + (size_t)b * a.nrun * a.H + hc;
  for (int k = k0; k < k1; k += U) {
    float4 v[U];
#pragma unroll
    for (int e = 0; e < U; ++e) v[e] = ag[at(k + e < k1 ? k + e : k1 - 1)];
#pragma unroll
    for (int e = 0; e < U; ++e)
      if (k + e < k1) {
        if (h < a.H) in[at(k + e)] = s;
        step(v[e]);
      }
  }
  float *fin = dir ? a.fin[1] : a.fin[0];
  if (sg == 7 && fin && h < a.H) {
    fin[(size_t)b * 2 * a.H + h] = s.x;
    fin[(size_t)b * 2 * a.H + a.H + h] = s.y;
  }
}

// ------------------------------------------------------------------------ 4. forward: y
// A thread takes two complex channels of one run of 64 steps.
struct CgApplyArgs {
  Problem p;                       // T: steps of the whole sequence (of y)
  const unsigned short *xh, *xl;   // [B][n][D]
  const float *pq;                 // [2][B][n][H]
  const float2 *in;                // [B][nrun][H], or null with a single run: init
  const float *init;               // [B][D] or null
  float *hT;                       // only with a single run
  int t_lo, n, nrun;
};
__global__ void __launch_bounds__(256) cg_apply_kernel(CgApplyArgs a) {
  const Problem &p = a.p;
  const int lane = threadIdx.x & 63, k = blockIdx.y * 4 + (threadIdx.x >> 6), b = blockIdx.z;
  const int D = p.D, H = D / 2, h = (blockIdx.x * 64 + lane) * 2;
  if (k >= a.nrun || h >= H) return;
  const Decay dk[2] = {Decay(p, h), Decay(p, h + 1)};
  const int l0 = k * RUN, n = a.n - l0 < RUN ? a.n - l0 : RUN;
  float2 s[2] = {make_float2(0.f, 0.f), make_float2(0.f, 0.f)};
  if (a.in) {
    const float4 v = *(const float4 *)(a.in + ((size_t)b * a.nrun + k) * H + h);
    s[0] = make_float2(v.x, v.y);
    s[1] = make_float2(v.z, v.w);
  } else if (a.init) {
    for (int c = 0; c < 2; ++c) s[c] = make_float2(a.init[(size_t)b * D + h + c], a.init[(size_t)b * D + H + h + c]);
  }
  const size_t row = (size_t)b * a.n + l0, rows = (size_t)p.B * a.n;
  const float *pp = a.pq + row * H + h, *qp = pp + rows * H;
  const unsigned short *xh = a.xh + row * D + h, *xl = a.xl + row * D + h;
  unsigned short *y = (unsigned short *)p.y + ((size_t)b * p.T + a.t_lo + l0) * D + h;
  constexpr int U = 4;
  float2 np[U], nq[U];
  unsigned nx[U][4];
  auto load = [&](int r0) __attribute__((always_inline)) {
#pragma unroll
    for (int e = 0; e < U; ++e) {
      const size_t r = (size_t)(r0 + e < n ? r0 + e : n - 1);
      np[e] = *(const float2 *)(pp + r * H);
      nq[e] = *(const float2 *)(qp + r * H);
      nx[e][0] = *(const unsigned *)(xh + r * D);
      nx[e][1] = *(const unsigned *)(xh + r * D + H);
      nx[e][2] = *(const unsigned *)(xl + r * D);
      nx[e][3] = *(const unsigned *)(xl + r * D + H);
    }
  };
  load(0);
  for (int r0 = 0; r0 < n; r0 += U) {
    float2 cp[U], cq[U];
    unsigned cx[U][4];
#pragma unroll
    for (int e = 0; e < U; ++e) {
      cp[e] = np[e];
      cq[e] = nq[e];
#pragma unroll
      for (int q = 0; q < 4; ++q) cx[e][q] = nx[e][q];
    }
    load(r0 + U);
#pragma unroll
    for (int e = 0; e < U; ++e) {
      if (r0 + e >= n) break;
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        float l2, mod;
        const float2 av = cdecay(dk[c], sigm(c ? cp[e].y : cp[e].x), l2, mod);
        const float gain = __builtin_amdgcn_sqrtf(one_minus_sq(mod, l2)) * sigm(c ? cq[e].y : cq[e].x);
        const float xr = c ? f16_hi(cx[e][0]) + f16_hi(cx[e][2]) : f16_lo(cx[e][0]) + f16_lo(cx[e][2]);
        const float xi = c ? f16_hi(cx[e][1]) + f16_hi(cx[e][3]) : f16_lo(cx[e][1]) + f16_lo(cx[e][3]);
        const float2 t = cmul(av, s[c]);
        s[c] = make_float2(fmaf(gain, xr, t.x), fmaf(gain, xi, t.y));
      }
      unsigned short *o = y + (size_t)(r0 + e) * D;
      *(u32_at2 *)o = pack_bf16(s[0].x, s[1].x);
      *(u32_at2 *)(o + H) = pack_bf16(s[0].y, s[1].y);
    }
  }
  if (a.hT)
    for (int c = 0; c < 2; ++c) {
      a.hT[(size_t)b * D + h + c] = s[c].x;
      a.hT[(size_t)b * D + H + h + c] = s[c].y;
    }
}

// ------------------------------------------------------------------------ 4. backward: adjoints
// A wave takes 32 complex channels x 32 steps, a lane 16 steps of a channel with the states entering
// them from both sides: forwards for h~_{t-1}, backwards for eps and the adjoints
//   G = delta~ conj(h~_{t-1}), dL/dlog|a~| = Re(conj(G) a~) - (dL/dm) |a~|^2 / m, dL/darg a~ = Im G Re a~ - Re G Im a~
// x (high, low) and dy come through LDS, transposed on the way out (as in cg_gates_kernel).
constexpr int CA_TILE = 3 * 4096;      // per wave: x high | x low | dy, 32 rows of 128 bytes each
struct CgAdjArgs {
  Problem p;
  const unsigned short *xh, *xl;
  const float *pq;
  const float2 *hin, *ein;             // [B][nsub][H]
  unsigned short *dph, *dpl;           // [B][T][nb][2][hs] bf16: dp | dq, high and low parts
  float *dx;                           // [B][T][D] direct part of dx
  float *part;                         // [B][ceil(T / 128)][4][H]
  int nsub;
};
__global__ void __launch_bounds__(256) cg_adjoint_kernel(CgAdjArgs a) {
  __shared__ __attribute__((aligned(16))) unsigned char smem[4 * CA_TILE];
  __shared__ float red[4][4][32];
  const Problem &p = a.p;
  const int tid = threadIdx.x, lane = tid & 63, hf = lane >> 5, j = lane & 31;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int D = p.D, H = D / 2, T = p.T, hs = p.bs, b = blockIdx.z, h0c = blockIdx.x * 32, tr = (blockIdx.y * 4 + wv) * 32;
  const int h = h0c + j;
  const bool ok = h < H;
  const int hc = ok ? h : H - 1, g = hc / hs;
  float s_ba = 0.f, s_bx = 0.f, s_lam = 0.f, s_th = 0.f;
  if (tr < T) {
    const unsigned row_bytes = (unsigned)D * 2;
    // (every buffer starts at the wave's rows)
    const size_t row0 = (size_t)b * T + tr, first = row0 * D, nrow = T - tr < 32 ? T - tr : 32, bytes = nrow * row_bytes;
    const __amdgpu_buffer_rsrc_t xh_rs = buf(a.xh + first, bytes), xl_rs = buf(a.xl + first, bytes),
                                 dy_rs = buf((const unsigned short *)p.dy + first, bytes),
                                 p_rs = buf(a.pq + row0 * H, nrow * H * 4),
                                 q_rs = buf(a.pq + ((size_t)p.B * T + row0) * H, nrow * H * 4),
                                 h_rs = buf(a.dph + first, bytes), l_rs = buf(a.dpl + first, bytes),
                                 x_rs = buf(a.dx + first, bytes * 2);
    unsigned char *tile = smem + wv * CA_TILE;
    const int erow = lane >> 3, ec = (lane & 7) ^ ((erow & 3) * 2), ecol = h0c + (ec & 3) * 8;
    const unsigned e_vo = ecol < H ? (unsigned)erow * row_bytes + (unsigned)((ec >> 2) * H + ecol) * 2 : OOB;
#pragma unroll
    for (int m = 0; m < 4; ++m) {
      const unsigned so = (unsigned)(8 * m) * row_bytes;
      lds16(xh_rs, tile + m * 1024, e_vo, so);
      lds16(xl_rs, tile + 4096 + m * 1024, e_vo, so);
      lds16(dy_rs, tile + 8192 + m * 1024, e_vo, so);
    }
    const unsigned g_vo = (unsigned)hc * 4 + (unsigned)(hf * 16) * (unsigned)H * 4;
    float pv[16], qv[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const unsigned so = (unsigned)r * (unsigned)H * 4;
      pv[r] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(p_rs, g_vo, so, 0));
      qv[r] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(q_rs, g_vo, so, 0));
    }
    const int sub = tr / SUB + hf, subc = sub < a.nsub ? sub : a.nsub - 1;
    float2 hst = a.hin[((size_t)b * a.nsub + subc) * H + hc], eps = a.ein[((size_t)b * a.nsub + subc) * H + hc];
    const Decay dk(p, hc);
    const float theta = p.theta[hc], log_sig = neg_c_softplus(p.Lambda[hc], 1.f);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    const int i16 = lane & 15, q16 = (lane >> 4) & 1;
    const unsigned e_rd = (unsigned)(hf * 16 + (i16 >> 2)) * 128 +
                          (unsigned)((((q16 * 2) + ((i16 & 3) >> 1)) ^ (((i16 >> 2) & 3) * 2)) * 16) + (unsigned)(i16 & 1) * 8;
    auto e_read = [&](const unsigned char *t, int part, unsigned (&v)[8]) __attribute__((always_inline)) {
#pragma unroll
      for (int n = 0; n < 4; ++n) {
        const u32x2 w = lds_tr(t + ((e_rd + (unsigned)(4 * n) * 128) ^ (unsigned)(part * 64)));
        v[2 * n] = w[0];
        v[2 * n + 1] = w[1];
      }
    };
    float2 x[16], av[16], hp[16];   // x~_t, a~_t, h~_{t-1}
    {
      unsigned rh[8], rl[8];
#pragma unroll
      for (int part = 0; part < 2; ++part) {
        e_read(tile, part, rh);
        e_read(tile + 4096, part, rl);
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const float v = (r & 1) ? f16_hi(rh[r >> 1]) + f16_hi(rl[r >> 1]) : f16_lo(rh[r >> 1]) + f16_lo(rl[r >> 1]);
          if (part) x[r].y = v;
          else x[r].x = v;
        }
      }
    }
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      float l2, mod;
      av[r] = cdecay(dk, sigm(pv[r]), l2, mod);
      const float gain = __builtin_amdgcn_sqrtf(one_minus_sq(mod, l2)) * sigm(qv[r]);
      hp[r] = hst;
      const float2 t = cmul(av[r], hst);
      hst = make_float2(fmaf(gain, x[r].x, t.x), fmaf(gain, x[r].y, t.y));
    }
    unsigned dr[8], di[8];
    e_read(tile + 8192, 0, dr);
    e_read(tile + 8192, 1, di);
    const int nvalid = T - tr - hf * 16;
    const unsigned o_vo = ok ? (unsigned)(g * 2 * hs + (h - g * hs)) * 2 + (unsigned)(hf * 16) * row_bytes : OOB;
    const unsigned x_vo = ok ? (unsigned)h * 4 + (unsigned)(hf * 16) * row_bytes * 2 : OOB;
#pragma unroll
    for (int r = 15; r >= 0; --r) {
      const bool hi = r & 1, in = r < nvalid;
      const float pl = pv[r], ql = qv[r];
      const float er = __builtin_amdgcn_exp2f(-LOG2E * fabsf(pl)), rr = __builtin_amdgcn_rcpf(1.f + er);
      const float rg = pl >= 0.f ? rr : er * rr, rrc = er * rr * rr;
      const float ei = __builtin_amdgcn_exp2f(-LOG2E * fabsf(ql)), ri = __builtin_amdgcn_rcpf(1.f + ei);
      const float ig = ql >= 0.f ? ri : ei * ri, iic = ei * ri * ri;
      const float l2 = dk.l2 * rg, mod2 = fmaf(av[r].x, av[r].x, av[r].y * av[r].y);
      const float m2 = fmaxf(one_minus_mod2(__builtin_amdgcn_exp2f(l2), l2), 1e-30f), rs = __builtin_amdgcn_rsqf(m2), m = m2 * rs;
      float2 dl = make_float2((hi ? bf_hi(dr[r >> 1]) : bf_lo(dr[r >> 1])) + eps.x, (hi ? bf_hi(di[r >> 1]) : bf_lo(di[r >> 1])) + eps.y);
      if (!in) dl = make_float2(0.f, 0.f);
      const float Gr = fmaf(dl.x, hp[r].x, dl.y * hp[r].y), Gi = fmaf(dl.y, hp[r].x, -dl.x * hp[r].y);
      const float sx = fmaf(dl.x, x[r].x, dl.y * x[r].y);   // dL/d(m_t i_t)
      const float dlm = fmaf(Gr, av[r].x, Gi * av[r].y) - sx * ig * mod2 * rs;
      const float dph = fmaf(Gi, av[r].x, -Gr * av[r].y);
      const float dpv = p.c * fmaf(dlm, log_sig, dph * theta) * rrc, dqv = sx * m * iic;
      s_ba += dpv;
      s_bx += dqv;
      s_lam = fmaf(dlm, rg, s_lam);
      s_th = fmaf(dph, rg, s_th);
      if (in) eps = cmul(make_float2(av[r].x, -av[r].y), dl);
      unsigned hi_pk, lo_pk;
      split_bf16(dpv, dqv, hi_pk, lo_pk);
      const unsigned so = (unsigned)r * row_bytes;
      __builtin_amdgcn_raw_buffer_store_b16((short)(hi_pk & 0xffffu), h_rs, o_vo, so, 0);
      __builtin_amdgcn_raw_buffer_store_b16((short)(hi_pk >> 16), h_rs, o_vo, so + (unsigned)hs * 2, 0);
      __builtin_amdgcn_raw_buffer_store_b16((short)(lo_pk & 0xffffu), l_rs, o_vo, so, 0);
      __builtin_amdgcn_raw_buffer_store_b16((short)(lo_pk >> 16), l_rs, o_vo, so + (unsigned)hs * 2, 0);
      const float gain = m * ig;
      __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(dl.x * gain), x_rs, x_vo, so * 2, 0);
      __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(dl.y * gain), x_rs, x_vo, so * 2 + (unsigned)H * 4, 0);
    }
    s_lam *= p.c / (1.f + expf(p.Lambda[hc]));   // c d log sigmoid(Lambda) / d Lambda
    s_th *= p.c;
  }
  s_ba += __shfl_xor(s_ba, 32);
  s_bx += __shfl_xor(s_bx, 32);
  s_lam += __shfl_xor(s_lam, 32);
  s_th += __shfl_xor(s_th, 32);
  if (hf == 0) {
    red[wv][0][j] = s_ba;
    red[wv][1][j] = s_bx;
    red[wv][2][j] = s_lam;
    red[wv][3][j] = s_th;
  }
  __syncthreads();
  if (tid < 128 && h0c + (tid & 31) < H) {
    const int q = tid >> 5, c = tid & 31;
    a.part[(((size_t)b * gridDim.y + blockIdx.y) * 4 + q) * H + h0c + c] = (red[0][q][c] + red[1][q][c]) + (red[2][q][c] + red[3][q][c]);
  }
}

// ------------------------------------------------------------------------ 5. dgrad
// dx[part][k] += sum_j [dp | dq][j] wt[part hs + k][j] for 256 rows x 128 input channels of one part of a
// block, high and low part of dp | dq against the same weights; fp32 in place
struct CgDgradArgs {
  Problem p;
  const unsigned short *dph, *dpl, *wt;
  float *dx;
  int nct, nrt;
  unsigned total;
};
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2))) cg_dgrad_kernel(CgDgradArgs a) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const Problem &p = a.p;
  const unsigned id = xcd_id();
  if (id >= a.total) return;
  const int tid = threadIdx.x, lane = tid & 63, hf = lane >> 5, j = lane & 31;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int pt = (int)(id % (2 * a.nct)), part = pt / a.nct, ct = pt - part * a.nct;
  const int rt = (int)(id / (2 * a.nct) % a.nrt), gb = (int)(id / (2 * a.nct) / a.nrt);
  const int b = gb % p.B, g = gb / p.B;
  const int D = p.D, H = D / 2, T = p.T, hs = p.bs, t0 = rt * PR, tw = t0 + wv * RUN;
  const unsigned row2 = (unsigned)D * 2, wrow = (unsigned)hs * 4;
  const size_t first = ((size_t)b * T + t0) * D, bytes = (size_t)(T - t0 < PR ? T - t0 : PR) * row2;
  const __amdgpu_buffer_rsrc_t h_rs = buf(a.dph + first, bytes), l_rs = buf(a.dpl + first, bytes), x_rs = buf(a.dx + first, bytes * 2),
                               w_rs = buf(a.wt + ((size_t)g * 2 * hs + part * hs) * 2 * hs, (size_t)hs * wrow);
  const int lrow = lane >> 2;
  const int ca = (lane & 3) ^ (((lrow >> 1) & 1) | ((wv & 1) << 1)), cb_ = (lane & 3) ^ ((lrow >> 1) & 3);
  const unsigned a_vo = (unsigned)lrow * row2 + (unsigned)(g * 2 * hs) * 2 + (unsigned)ca * 16;
  const unsigned b_vo = (unsigned)(ct * 128 + lrow) * wrow + (unsigned)cb_ * 16;
  const int nkc = 2 * hs / 32;
  auto load_stage = [&](int kc, int st) __attribute__((always_inline)) {
    unsigned char *s = smem + st * CST;
#pragma unroll
    for (int m = 0; m < 4; ++m) {
      const int i = wv + 4 * m;
      const unsigned so = (unsigned)(16 * i) * row2 + (unsigned)kc * 64;
      lds16(h_rs, s + i * 1024, a_vo, so);
      lds16(l_rs, s + CST_A + i * 1024, a_vo, so);
    }
#pragma unroll
    for (int m = 0; m < 2; ++m) {
      const int i = wv + 4 * m;
      lds16(w_rs, s + 2 * CST_A + i * 1024, b_vo, (unsigned)(16 * i) * wrow + (unsigned)kc * 64);
    }
  };
  load_stage(0, 0);
  f32x16 acc[2][4];
#pragma unroll
  for (int rb = 0; rb < 2; ++rb)
#pragma unroll
    for (int cb = 0; cb < 4; ++cb)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[rb][cb][r] = 0.f;
  const int arow = perm_row(j);
  const unsigned a_rd = (unsigned)(wv * RUN + arow) * 64 + (unsigned)(hf ^ key_a(arow)) * 16;
  const unsigned b_rd = 2 * CST_A + (unsigned)j * 64 + (unsigned)(hf ^ key_b(j)) * 16;
  const bool rows_on = tw < T;
  const int ncb = (hs - ct * 128 + 31) / 32;
  for (int kc = 0; kc < nkc; ++kc) {
    stage_barrier();
    if (kc + 1 < nkc) load_stage(kc + 1, (kc + 1) & 1);
    if (!rows_on) continue;
    const unsigned char *s = smem + (kc & 1) * CST;
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      bf16x8 fh[2], fl[2], fb[4];
#pragma unroll
      for (int rb = 0; rb < 2; ++rb) {
        fh[rb] = *(const bf16x8 *)(s + ((a_rd + rb * 2048) ^ (ks * 32)));
        fl[rb] = *(const bf16x8 *)(s + ((a_rd + CST_A + rb * 2048) ^ (ks * 32)));
      }
#pragma unroll
      for (int cb = 0; cb < 4; ++cb) fb[cb] = *(const bf16x8 *)(s + ((b_rd + cb * 2048) ^ (ks * 32)));
#pragma unroll
      for (int cb = 0; cb < 4; ++cb)
        if (cb < ncb) {
#pragma unroll
          for (int rb = 0; rb < 2; ++rb)
            acc[rb][cb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fh[rb], fb[cb], acc[rb][cb], 0, 0, 0);
#pragma unroll
          for (int rb = 0; rb < 2; ++rb)
            acc[rb][cb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fl[rb], fb[cb], acc[rb][cb], 0, 0, 0);
        }
    }
  }
  if (!rows_on) return;
#pragma unroll
  for (int rb = 0; rb < 2; ++rb)
#pragma unroll
    for (int cb = 0; cb < 4; ++cb) {
      const int kk = ct * 128 + cb * 32 + j;
      const unsigned vo = kk < hs ? (unsigned)(part * H + g * hs + kk) * 4 + (unsigned)(hf * 16) * row2 * 2 : OOB;
      const unsigned so = (unsigned)(wv * RUN + rb * 32) * row2 * 2;
      float v[16];
#pragma unroll
      for (int r = 0; r < 16; ++r) v[r] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(x_rs, vo, so + r * row2 * 2, 0));
#pragma unroll
      for (int r = 0; r < 16; ++r)
        __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v[r] + acc[rb][cb][r]), x_rs, vo, so + r * row2 * 2, 0);
    }
}

// ------------------------------------------------------------------------ 7. wgrad
// part[slice][g][gate hs + j][part hs + k] = sum over rows of dp|dq x: 128 x 128 outputs per workgroup.
// dp | dq (high, low) come straight into LDS; x comes through registers, where its half-precision
// parts become bf16 high + low parts (the exponent range of dp's), once per workgroup.
constexpr int WST = 4 * 8192;   // stage: dp|dq high | low | x high | low, 32 rows of 256 bytes each
constexpr int W_LDS = 2 * WST;
struct CgWgradArgs {
  const unsigned short *dph, *dpl, *xh, *xl;
  float *part;
  long long rows;
  int per, D, nb, hs, njt, nkt;   // nkt: tiles of one part of x
  unsigned total;
};
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2))) cg_wgrad_kernel(CgWgradArgs a) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const unsigned id = xcd_id();
  if (id >= a.total) return;
  const int tid = threadIdx.x, lane = tid & 63, hf = lane >> 5;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int pk = (int)(id % (2 * a.nkt)), part = pk / a.nkt, kt = pk - part * a.nkt;
  const int jt = (int)(id / (2 * a.nkt) % a.njt), g = (int)(id / (2 * a.nkt) / a.njt % a.nb),
            sl = (int)(id / (2 * a.nkt) / a.njt / a.nb);
  const int D = a.D, H = D / 2, hs = a.hs, j0 = jt * 128, k0 = kt * 128;
  const long long r_lo = (long long)sl * a.per, left = a.rows - r_lo;
  const int nrow = left < a.per ? (int)left : a.per;
  const unsigned row2 = (unsigned)D * 2;
  const size_t base = (size_t)r_lo * D, bytes = (size_t)nrow * row2;
  const __amdgpu_buffer_rsrc_t h_rs = buf(a.dph + base, bytes), l_rs = buf(a.dpl + base, bytes),
                               xh_rs = buf(a.xh + base, bytes), xl_rs = buf(a.xl + base, bytes);
  const int rq = lane >> 4, cq = (lane & 15) ^ (rq * 2);   // 4 rows of 256 bytes per instruction, pieces permuted by row & 3
  const unsigned a_vo = j0 + cq * 8 < 2 * hs ? (unsigned)rq * row2 + (unsigned)(g * 2 * hs + j0) * 2 + (unsigned)cq * 16 : OOB;
  // x: thread -> pieces tid and tid + 256 of the 32 x 16
  const int xr = tid >> 4, xc = tid & 15;
  const unsigned x_vo = k0 + xc * 8 < hs ? (unsigned)xr * row2 + (unsigned)(part * H + g * hs + k0) * 2 + (unsigned)xc * 16 : OOB;
  const unsigned x_wr = (unsigned)xr * 256 + (unsigned)(xc ^ ((xr & 3) * 2)) * 16;
  const int nst = (nrow + 31) / 32;
  u32x4 rh[2], rl[2];
  auto load_x = [&](int kc) __attribute__((always_inline)) {
#pragma unroll
    for (int m = 0; m < 2; ++m) {
      rh[m] = __builtin_amdgcn_raw_buffer_load_b128(xh_rs, x_vo, (unsigned)(kc * 32 + 16 * m) * row2, 0);
      rl[m] = __builtin_amdgcn_raw_buffer_load_b128(xl_rs, x_vo, (unsigned)(kc * 32 + 16 * m) * row2, 0);
    }
  };
  auto load_dp = [&](int kc, int st) __attribute__((always_inline)) {
    unsigned char *s = smem + st * WST;
#pragma unroll
    for (int m = 0; m < 2; ++m) {
      const int i = wv + 4 * m;
      lds16(h_rs, s + i * 1024, a_vo, (unsigned)(kc * 32 + 4 * i) * row2);
      lds16(l_rs, s + 8192 + i * 1024, a_vo, (unsigned)(kc * 32 + 4 * i) * row2);
    }
  };
  auto park_x = [&](int st) __attribute__((always_inline)) {
    unsigned char *s = smem + st * WST + 16384;
#pragma unroll
    for (int m = 0; m < 2; ++m) {
      u32x4 oh, ol;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        unsigned hp, lp;
        split_bf16(f16_lo(rh[m][e]) + f16_lo(rl[m][e]), f16_hi(rh[m][e]) + f16_hi(rl[m][e]), hp, lp);
        oh[e] = hp;
        ol[e] = lp;
      }
      *(u32x4 *)(s + m * 4096 + x_wr) = oh;
      *(u32x4 *)(s + 8192 + m * 4096 + x_wr) = ol;
    }
  };
  load_x(0);
  load_dp(0, 0);
  park_x(0);
  load_x(1 < nst ? 1 : 0);
  f32x16 acc[2][2];
#pragma unroll
  for (int m = 0; m < 2; ++m)
#pragma unroll
    for (int n = 0; n < 2; ++n)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[m][n][r] = 0.f;
  const int wj = wv >> 1, wk = wv & 1;   // the wave's 64 x 64 outputs
  const int i16 = lane & 15, q16 = (lane >> 4) & 1, key = (i16 >> 2) * 2;
  const unsigned trow = (unsigned)(hf * 8 + (i16 >> 2));
  const int tc = q16 * 2 + ((i16 & 3) >> 1);
  const unsigned sub = (unsigned)(i16 & 1) * 8;
  const unsigned a_rd = trow * 256 + (unsigned)((wj * 8 + tc) ^ key) * 16 + sub;
  const unsigned b_rd = 16384 + trow * 256 + (unsigned)((wk * 8 + tc) ^ key) * 16 + sub;
  for (int kc = 0; kc < nst; ++kc) {
    stage_barrier();
    if (kc + 1 < nst) {
      load_dp(kc + 1, (kc + 1) & 1);
      park_x((kc + 1) & 1);
      load_x(kc + 2 < nst ? kc + 2 : kc + 1);
    }
    const unsigned char *s = smem + (kc & 1) * WST;
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      bf16x8 ah[2], al[2], bh[2], bl[2];
      auto frag = [&](unsigned at) __attribute__((always_inline)) {
        const u32x2 lo = lds_tr(s + at), hi = lds_tr(s + at + 4 * 256);
        return __builtin_bit_cast(bf16x8, (u32x4){lo[0], lo[1], hi[0], hi[1]});
      };
#pragma unroll
      for (int m = 0; m < 2; ++m) {
        ah[m] = frag((a_rd ^ (unsigned)(m * 64)) + ks * 4096);
        al[m] = frag((a_rd ^ (unsigned)(m * 64)) + 8192 + ks * 4096);
        bh[m] = frag((b_rd ^ (unsigned)(m * 64)) + ks * 4096);
        bl[m] = frag((b_rd ^ (unsigned)(m * 64)) + 8192 + ks * 4096);
      }
#pragma unroll
      for (int m = 0; m < 2; ++m)
#pragma unroll
        for (int n = 0; n < 2; ++n) acc[m][n] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah[m], bh[n], acc[m][n], 0, 0, 0);
#pragma unroll
      for (int m = 0; m < 2; ++m)
#pragma unroll
        for (int n = 0; n < 2; ++n) acc[m][n] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(al[m], bh[n], acc[m][n], 0, 0, 0);
#pragma unroll
      for (int m = 0; m < 2; ++m)
#pragma unroll
        for (int n = 0; n < 2; ++n) acc[m][n] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah[m], bl[n], acc[m][n], 0, 0, 0);
    }
  }
  const int j = lane & 31;
  float *out = a.part + ((size_t)sl * a.nb + g) * 4 * hs * hs;
#pragma unroll
  for (int m = 0; m < 2; ++m)
#pragma unroll
    for (int n = 0; n < 2; ++n)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int row = j0 + wj * 64 + m * 32 + 8 * (r >> 2) + 4 * hf + (r & 3), kk = k0 + wk * 64 + n * 32 + j;
        if (row < 2 * hs && kk < hs) out[(size_t)row * 2 * hs + part * hs + kk] = acc[m][n][r];
      }
}

// ------------------------------------------------------------------------ host side
hipError_t configure() {
  static bool done = false;
  if (done) return hipSuccess;
  hipError_t e;
  if ((e = big_lds(cg_gates_kernel<false>, C_LDS)) != hipSuccess) return e;
  if ((e = big_lds(cg_gates_kernel<true>, C_LDS)) != hipSuccess) return e;
  if ((e = big_lds(cg_dgrad_kernel, C_LDS)) != hipSuccess) return e;
  if ((e = big_lds(cg_wgrad_kernel, W_LDS)) != hipSuccess) return e;
  done = true;
  return hipSuccess;
}
hipError_t launch_prep(const Problem &p, unsigned short *w16, unsigned short *wt, hipStream_t s) {
  KernelTimer kt("cg_prep_kernel", s);
  CgPrepArgs a;
  a.Wa = (const unsigned short *)p.W_a; a.Wx = (const unsigned short *)p.W_x;
  a.w16 = w16; a.wt = wt; a.nb = p.nb; a.hs = p.bs;
  const size_t n = (size_t)p.nb * p.bs * p.bs * 4;
  hipLaunchKernelGGL(cg_prep_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, a);
  return hipGetLastError();
}
CgGatesArgs gates_args(const Problem &p, int T) {
  CgGatesArgs a;
  a.p = p;
  a.p.T = T;
  a.nct = (p.bs + 63) / 64;
  a.nrt = (T + PR - 1) / PR;
  a.total = (unsigned)a.nct * a.nrt * p.B * p.nb;
  a.agg = a.aggf = a.aggr = nullptr;
  return a;
}
bool shape_ok(int B, int T, int D, int hs) {
  return hs % 16 == 0 && hs >= 16 && T >= 1 && B <= 65535 && (size_t)PR * D * 4 < ((size_t)1 << 31) &&
         (T + 127) / 128 <= 65535 && (size_t)B * ((T + PR - 1) / PR) * ((size_t)D / 16) < ((size_t)1 << 28);
}

// scratch of a chunk of n steps: weights | x high, low | pre-activations | aggregates | states; the last
// two only for more than one run. `carry`: the state between chunks.
struct FwdPlan {
  size_t off_w, off_xh, off_xl, off_pq, off_agg, off_in, off_carry, total;
};
FwdPlan plan_fwd(int B, int n, int D, int nb) {
  const int hs = D / 2 / nb, nrun = (n + RUN - 1) / RUN;
  FwdPlan q;
  size_t off = 0;
  q.off_w = off; off += al256((size_t)nb * hs * hs * 8);
  q.off_xh = off; off += al256((size_t)B * n * D * 2);
  q.off_xl = off; off += al256((size_t)B * n * D * 2);
  q.off_pq = off; off += al256((size_t)B * n * D * 4);
  q.off_agg = off; off += al256((size_t)B * nrun * (D / 2) * 16);
  q.off_in = off; off += al256((size_t)B * nrun * (D / 2) * 8);
  q.off_carry = off; off += al256((size_t)B * D * 4);
  q.total = off;
  return q;
}
// steps per chunk the size is made for: intermediates of about 128 MB, which the last-level cache holds
int chunk_steps(int B, int T, int D) {
  const size_t per = (size_t)B * D * 8;
  size_t n = ((size_t)128 << 20) / per / PR * PR;
  if (n < PR) n = PR;
  return n < (size_t)T ? (int)n : T;
}

struct BwdPlan {
  int nsub, n128, n256, S, per, njt, nkt;
  size_t off_xh, off_xl, off_pq, off_dph, off_dpl, off_dx, off_w, off_wt, off_aggf, off_aggr, off_hin, off_ein, off_partA,
      off_partC, off_partW, total;
};
BwdPlan plan_bwd(int B, int T, int D, int nb) {
  BwdPlan q;
  const int H = D / 2, hs = H / nb;
  q.nsub = (T + SUB - 1) / SUB;
  q.n128 = (T + 127) / 128;
  q.n256 = (T + 255) / 256;
  q.njt = (2 * hs + 127) / 128;
  q.nkt = (hs + 127) / 128;
  const long long rows = (long long)B * T, tiles = (long long)nb * q.njt * 2 * q.nkt;
  long long S = (2 * 256 + tiles - 1) / tiles;
  if (S > rows / 256) S = rows / 256;
  const long long most = (((long long)1 << 31) - 1) / ((long long)D * 2) - 32;
  if (S < (rows + most - 1) / most) S = (rows + most - 1) / most;
  if (S < 1) S = 1;
  q.per = (int)(((rows + S - 1) / S + 31) / 32 * 32);
  q.S = (int)((rows + q.per - 1) / q.per);
  const size_t n2 = al256((size_t)B * T * D * 2), sub = (size_t)B * q.nsub * H;
  size_t off = 0;
  q.off_xh = off; off += n2;
  q.off_xl = off; off += n2;
  q.off_dph = off; off += n2;
  q.off_dpl = off; off += n2;
  q.off_partA = off; off += al256((size_t)B * q.n128 * 4 * H * 4);
  q.off_partC = off; off += al256((size_t)B * q.n256 * 5 * D * 4);
  // from here on what the weight gradients' pass needs no more: its partial sums take the same room
  q.off_partW = off;
  q.off_pq = off; off += 2 * n2;
  q.off_dx = off; off += 2 * n2;
  q.off_w = off; off += al256((size_t)nb * hs * hs * 8);
  q.off_wt = off; off += al256((size_t)nb * hs * hs * 8);
  q.off_aggf = off; off += al256(sub * 16);
  q.off_aggr = off; off += al256(sub * 16);
  q.off_hin = off; off += al256(sub * 8);
  q.off_ein = off; off += al256(sub * 8);
  off = std::max(off, q.off_partW + al256((size_t)q.S * nb * 4 * hs * hs * 4));
  q.total = off;
  return q;
}

}  // namespace

size_t cg_forward_pass_ws_bytes(int B, int T, int D, int nb) {
  const int hs = D / 2 / nb;
  if (!shape_ok(B, T, D, hs)) return 0;
  return plan_fwd(B, chunk_steps(B, T, D), D, nb).total;
}
// With one run a sequence starts from h0 itself and three launches do; the passes are for sequences
// of more than a run (the fused and general kernels are faster on a few tiles).
bool cg_forward_pass_supported(const Problem &p) {
  return p.T > RUN && shape_ok(p.B, p.T, p.D, p.bs) && p.ws && (uintptr_t)p.ws % 256 == 0 &&
         p.ws_bytes >= plan_fwd(p.B, p.T < PR ? p.T : PR, p.D, p.nb).total;
}
hipError_t launch_cg_forward_pass(const Problem &p, hipStream_t s) {
  hipError_t e;
  if ((e = configure()) != hipSuccess) return e;
  int n = chunk_steps(p.B, p.T, p.D);
  while (n > PR && plan_fwd(p.B, n, p.D, p.nb).total > p.ws_bytes) n = (n - 1) / PR * PR;   // (a smaller workspace: shorter chunks)
  const FwdPlan q = plan_fwd(p.B, n, p.D, p.nb);
  char *ws = (char *)p.ws;
  unsigned short *w16 = (unsigned short *)(ws + q.off_w), *xh = (unsigned short *)(ws + q.off_xh), *xl = (unsigned short *)(ws + q.off_xl);
  float *pq = (float *)(ws + q.off_pq), *carry = (float *)(ws + q.off_carry);
  if ((e = launch_prep(p, w16, nullptr, s)) != hipSuccess) return e;
  for (int t_lo = 0; t_lo < p.T; t_lo += n) {
    const int m = p.T - t_lo < n ? p.T - t_lo : n;
    const bool last = t_lo + m == p.T;
    if ((e = launch_conv_rows(p, xh, xl, t_lo, m, s)) != hipSuccess) return e;
    CgGatesArgs a = gates_args(p, m);
    a.xh = xh; a.xl = xl; a.w16 = w16; a.pq = pq;
    a.nrun = (m + RUN - 1) / RUN;
    const bool chain = a.nrun > 1;
    const float *init = t_lo == 0 ? p.h0 : carry;
    float *fin = last ? p.hT : carry;
    a.agg = chain ? (float4 *)(ws + q.off_agg) : nullptr;
    {
      KernelTimer kt("cg_gates_kernel", s);
      hipLaunchKernelGGL(cg_gates_kernel<false>, dim3(grid8(a.total)), dim3(256), C_LDS, s, a);
      if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    float2 *in = (float2 *)(ws + q.off_in);
    if (chain) {
      KernelTimer kt("cg_chain_kernel", s);
      CgChainArgs c;
      c.agg[0] = c.agg[1] = a.agg; c.init[0] = c.init[1] = init; c.in[0] = c.in[1] = in; c.fin[0] = c.fin[1] = fin;
      c.B = p.B; c.H = p.D / 2; c.nrun = a.nrun; c.ncg = (c.H + 31) / 32;
      hipLaunchKernelGGL(cg_chain_kernel, dim3((unsigned)(p.B * c.ncg), 1), dim3(256), 0, s, c);
      if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    {
      KernelTimer kt("cg_apply_kernel", s);
      CgApplyArgs y;
      y.p = p; y.xh = xh; y.xl = xl; y.pq = pq;
      y.in = chain ? in : nullptr; y.init = init; y.hT = chain ? nullptr : fin;
      y.t_lo = t_lo; y.n = m; y.nrun = a.nrun;
      hipLaunchKernelGGL(cg_apply_kernel, dim3((unsigned)(p.D / 2 + 127) / 128, (unsigned)(a.nrun + 3) / 4, p.B), dim3(256), 0, s, y);
      if ((e = hipGetLastError()) != hipSuccess) return e;
    }
  }
  return hipSuccess;
}

size_t cg_backward_pass_ws_bytes(int B, int T, int D, int nb) {
  return shape_ok(B, T, D, D / 2 / nb) ? plan_bwd(B, T, D, nb).total : 0;
}
// The staging of dy wants 16-byte aligned rows: any other dy is copied first, behind the plan (the size
// reported for the call is the general kernels' where those need more, 24 bytes per element against 18).
static size_t dy_copy_bytes(const Problem &p) {
  return (uintptr_t)p.dy % 16 == 0 ? 0 : al256((size_t)p.B * p.T * p.D * 2);
}
bool cg_backward_pass_supported(const Problem &p) {
  return shape_ok(p.B, p.T, p.D, p.bs) && p.ws_bytes >= plan_bwd(p.B, p.T, p.D, p.nb).total + dy_copy_bytes(p);
}
hipError_t launch_cg_backward_pass(const Problem &call, hipStream_t s) {
  hipError_t e;
  if ((e = configure()) != hipSuccess) return e;
  Problem p = call;
  const BwdPlan q = plan_bwd(p.B, p.T, p.D, p.nb);
  char *ws = (char *)p.ws;
  if (dy_copy_bytes(p)) {
    if ((e = launch_realign(call.dy, ws + q.total, (size_t)p.B * p.T * p.D, s)) != hipSuccess) return e;
    p.dy = ws + q.total;
  }
  unsigned short *xh = (unsigned short *)(ws + q.off_xh), *xl = (unsigned short *)(ws + q.off_xl),
                 *dph = (unsigned short *)(ws + q.off_dph), *dpl = (unsigned short *)(ws + q.off_dpl),
                 *w16 = (unsigned short *)(ws + q.off_w), *wt = (unsigned short *)(ws + q.off_wt);
  float *pq = (float *)(ws + q.off_pq), *dx = (float *)(ws + q.off_dx);
  if ((e = launch_prep(p, w16, wt, s)) != hipSuccess) return e;
  if ((e = launch_conv_rows(p, xh, xl, 0, p.T, s)) != hipSuccess) return e;
  CgGatesArgs a = gates_args(p, p.T);
  a.xh = xh; a.xl = xl; a.w16 = w16; a.pq = pq;
  a.nrun = q.nsub;
  a.aggf = (float4 *)(ws + q.off_aggf); a.aggr = (float4 *)(ws + q.off_aggr);
  {
    KernelTimer kt("cg_gates_kernel", s);
    hipLaunchKernelGGL(cg_gates_kernel<true>, dim3(grid8(a.total)), dim3(256), C_LDS, s, a);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  float2 *hin = (float2 *)(ws + q.off_hin), *ein = (float2 *)(ws + q.off_ein);
  {
    KernelTimer kt("cg_chain_kernel", s);
    CgChainArgs c;
    c.agg[0] = a.aggf; c.agg[1] = a.aggr; c.init[0] = p.h0; c.init[1] = p.dhT; c.in[0] = hin; c.in[1] = ein;
    c.fin[0] = nullptr; c.fin[1] = p.dh0;
    c.B = p.B; c.H = p.D / 2; c.nrun = q.nsub; c.ncg = (c.H + 31) / 32;
    hipLaunchKernelGGL(cg_chain_kernel, dim3((unsigned)(p.B * c.ncg), 2), dim3(256), 0, s, c);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  {
    KernelTimer kt("cg_adjoint_kernel", s);
    CgAdjArgs d;
    d.p = p; d.xh = xh; d.xl = xl; d.pq = pq; d.hin = hin; d.ein = ein; d.dph = dph; d.dpl = dpl; d.dx = dx;
    d.part = (float *)(ws + q.off_partA);
    d.nsub = q.nsub;
    hipLaunchKernelGGL(cg_adjoint_kernel, dim3((unsigned)(p.D / 2 + 31) / 32, (unsigned)q.n128, p.B), dim3(256), 0, s, d);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  {
    KernelTimer kt("cg_dgrad_kernel", s);
    CgDgradArgs d;
    d.p = p; d.dph = dph; d.dpl = dpl; d.wt = wt; d.dx = dx;
    d.nct = (p.bs + 127) / 128;
    d.nrt = (p.T + PR - 1) / PR;
    d.total = (unsigned)2 * d.nct * d.nrt * p.B * p.nb;
    hipLaunchKernelGGL(cg_dgrad_kernel, dim3(grid8(d.total)), dim3(256), C_LDS, s, d);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  if ((e = launch_conv_adjoint(p, dx, (float *)(ws + q.off_partC), s)) != hipSuccess) return e;
  {
    KernelTimer kt("cg_wgrad_kernel", s);
    CgWgradArgs w;
    w.dph = dph; w.dpl = dpl; w.xh = xh; w.xl = xl; w.part = (float *)(ws + q.off_partW);
    w.rows = (long long)p.B * p.T; w.per = q.per; w.D = p.D; w.nb = p.nb; w.hs = p.bs; w.njt = q.njt; w.nkt = q.nkt;
    w.total = (unsigned)q.S * p.nb * q.njt * 2 * q.nkt;
    hipLaunchKernelGGL(cg_wgrad_kernel, dim3(grid8(w.total)), dim3(256), W_LDS, s, w);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  FinishArgs f;
  f.partW = (const float *)(ws + q.off_partW); f.partA = (const float *)(ws + q.off_partA);
  f.partC = (const float *)(ws + q.off_partC); f.sc = nullptr; f.edge = nullptr;
  f.S = q.S; f.nA = p.B * q.n128; f.nrA = 4; f.DA = p.D / 2; f.nC = p.B * q.n256; f.D = p.D; f.nb = p.nb;
  f.bb = (size_t)p.bs * 2 * p.bs;
  f.dW[0] = p.g.dW_a; f.dW[1] = p.g.dW_x;
  f.rowsA[0] = p.g.db_a; f.rowsA[1] = p.g.db_x; f.rowsA[2] = p.g.dLambda; f.rowsA[3] = p.dtheta;
  for (int k = 0; k < 4; ++k) f.rowsC[k] = p.g.dconv_w ? p.g.dconv_w + (size_t)k * p.D : nullptr;
  f.rowsC[4] = p.g.dconv_b;
  return launch_finish(f, s);
}

}  // namespace rglru
