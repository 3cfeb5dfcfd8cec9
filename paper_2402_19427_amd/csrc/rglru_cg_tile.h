// The complex-gated layer (Appendix B) in tiles, bf16 storage, blocks of 80 to 128 complex channels: counterparts of the real layer's
// kernels in tiles (rglru_bwd_fused.h: staging, layouts, helpers) on complex channels.
//
// A workgroup takes 32 steps of a gate block, a wave 32 of its complex channels, a lane 16 steps of one: u (real and imaginary
// rows) -> Conv1D -> x in registers (fp32) and in LDS (half precision, high and low part), p, q = x W_a^T, x W_x^T on the matrix
// cores, a~_t and b~_t, the recurrence. Nothing between u and y (u, dy and du) touches memory; the same layer in passes stored x
// (two parts), p, q, dp, dq (two parts) and dx and read each of them once or twice.
//
// No workgroup waits for another one. A sequence is cut into windows of tiles, as many as fill the chip. A first kernel walks every
// window but the last and leaves its map h -> A h + E; the second composes the maps in front of its window in its prologue and walks it
// with the true state. The backward's first kernel also leaves the map of eps_t = conj(a~_t) (dy~_t + eps_{t+1}) and, every 16
// steps, the map from the window's start, so that its second kernel, which walks backwards, has the state entering each run.
// The gates are formed twice for that; an exchange of records between running workgroups would form them once, but the entry
// points promise that no kernel waits on another.
// Forward + backward, us, in passes : in tiles: B 8 T 2048, 10 blocks of 128 channels 1058 : 580 (under the tracer, 4 % slower in all: first walk 76, y 93;
// first walk 92, backward 239, weight gradients 86); 16 blocks B 16 T 4096 5320 : 2830 (256 units: two windows of each sequence); 10 blocks
// B 1 T 12000 794 : 433, B 8 T 130 193 : 98, the backward of B 1 T 64 91 : 42; 10 blocks of 80, B 16 T 2048 1526 : 788.
// What bounds them: the vector unit (two waves per SIMD keep it busy 76 % of the forward walks' time and 63 % of the backward's, 165 instructions
// per complex step there, 8 of them transcendental), the matrix units next to it (24 and 18 %), and what two waves per SIMD cannot hide.
#pragma once
#include "rglru_bwd_fused.h"
#include "rglru_cg_math.h"

namespace rglru {
namespace cgt {
using namespace fused;

// A wave's region of LDS: u rows (36 of 64 bytes, real | imaginary), x as [channel][step] (high re, im, low re, im; then dp, dq,
// high and low; then du), dy rows or y as [channel][step] (re, im), constants
constexpr int U_PART = 36 * 64, U = 0, X = 2 * U_PART, S = X + 4 * 2048, C = S + 2 * 2048, CN = 20, REGION = C + 32 * CN * 4;
// constants: b_a, b_x, log2 |a~| and phase (revolutions) per r_t | taps re | taps im | conv_b re, im, log |a~| and phase per r_t
constexpr int PER_CU = 2;   // workgroups at once

struct CgTileArgs {
  Problem p;
  int ntile, W, per;            // tiles, windows per sequence, tiles per window
  unsigned total;
  const u32x4 *wg, *wd;         // weights in fragment order, [nb][wave][K-step][2][lane]: gates (half precision); transposed (bf16)
  float4 *wagg;                 // [B][W][H] maps of the windows
  float2 *wrev;                 // backward: [B][W][H] end values of the reverse maps (their factors are the conjugates)
  float2 *init;                 // [B][H]: h0 as it was (forward), dhT as it was (backward): the outputs may take their place
  float4 *run;                  // backward: [B][2 ntile][H] maps from the window's start to each run of 16 steps
  unsigned short *xF[2], *pqF[2];   // backward: x, dp | dq in bf16 high and low parts, stages of rglru_wgrad.h
  float *partA, *partC;         // [B W][4][H], [B W][5][D]
  float *edge;                  // [B][W][6][D] dx of a window's first and last three rows, or null (one window)
};

// ANY: u, dy, y and du need not lie on the 16-byte grid. Their rows then go through registers instead of straight to LDS and in 16-byte
// accesses of any alignment: the same values in the same places, so that results do not depend on where the tensors lie. What is not in
// flight while the tile in front is worked on costs 15 - 25 % (10 blocks of 128, B 8 T 2048: forward 146 us on the grid, 166 eight bytes off it,
// 186 two bytes off it, backward 394, 437 and 463; in passes 307 - 316 and 790).
// The kernels take it as AT_ANY in their second argument, so that the aligned ones' names stay as short as they are: a third argument's
// letters move their code by 256 bytes in its object, and the same instructions then take up to 1.4 % longer (forward and backward,
// 10 blocks of 128, B 8 T 2048: 581 us, 574 where they are; on one of three cards 541 either way).
constexpr int AT_ANY = 16;
template <int NCT, bool ANY>
struct Wave {
  static constexpr int NKS = 4 * NCT;
  const CgTileArgs &a;
  const Problem &p;
  unsigned char *smem, *my;
  int lane, hf, j, wv, g, b, w, hs, H, D, T, h;
  bool ok;
  unsigned row2, r_rd, t_wr[2], f_rd[2];
  size_t seq;

  __device__ __forceinline__ Wave(const CgTileArgs &a_, unsigned char *smem_, unsigned id, int W) : a(a_), p(a_.p), smem(smem_) {
    const int tid = threadIdx.x;
    lane = tid & 63; hf = lane >> 5; j = lane & 31;
    wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    w = __builtin_amdgcn_readfirstlane((int)(id % W));
    const int gb = __builtin_amdgcn_readfirstlane((int)(id / W));
    b = __builtin_amdgcn_readfirstlane(gb % p.B);
    g = __builtin_amdgcn_readfirstlane(gb / p.B);   // (neighbouring workgroups share a block's weights)
    hs = p.bs; D = p.D; H = D / 2; T = p.T;
    ok = wv * 32 + j < hs;                           // (channels past the block: zero inputs, weights and constants)
    h = g * hs + (ok ? wv * 32 + j : hs - 1);
    row2 = (unsigned)D * 2;
    my = smem + wv * REGION;
    seq = (size_t)b * T;
    if (hf == 0) {
      const float l2 = neg_c_softplus(p.Lambda[h], p.c) * LOG2E, th = p.c * p.theta[h];
      unsigned char *to = my + C + j * CN * 4;
      // (l2 finite, so that times the r_t = 0 of a closed gate it is 0 and not a NaN)
      *(f32x4 *)to = f32x4{ok ? p.b_a[h] : 0.f, ok ? p.b_x[h] : 0.f, l2 < -3e38f ? -3e38f : l2, th * 0.15915494309189535f};
#pragma unroll
      for (int part = 0; part < 2; ++part) {
        f32x4 t;
#pragma unroll
        for (int k = 0; k < 4; ++k) t[k] = !ok ? 0.f : p.conv_w ? p.conv_w[(size_t)k * D + part * H + h] : (k == 0 ? 1.f : 0.f);
        *(f32x4 *)(to + 16 + 16 * part) = t;
      }
      *(f32x4 *)(to + 48) = f32x4{ok && p.conv_b ? p.conv_b[h] : 0.f, ok && p.conv_b ? p.conv_b[H + h] : 0.f, neg_c_softplus(p.Lambda[h], p.c), th};
    }
    wave_lds_fence();
    const int i16 = lane & 15, q16 = (lane >> 4) & 1, a4 = i16 >> 2, cc = i16 & 3;
    r_rd = (unsigned)(hf * 16 + a4) * 64 + (unsigned)q16 * 32 + (unsigned)cc * 8;
#pragma unroll
    for (int n = 0; n < 2; ++n) {
      t_wr[n] = (unsigned)j * 64 + (unsigned)((hf * 2 + n) ^ key(j)) * 16;
      f_rd[n] = (unsigned)(hf * 8 + 4 * n + a4) * 64 + (unsigned)((((cc & 1) * 2 + q16) ^ key(4 * n + a4)) * 16) + (unsigned)(cc >> 1) * 8;
    }
  }
  static __device__ __forceinline__ int key(int c) { return (c >> 1) & 3; }
  __device__ __forceinline__ int lane_again() const {   // (a lane id whose uses are formed again rather than kept)
    int l = lane;
    asm volatile("" : "+v"(l));
    return l;
  }
  __device__ __forceinline__ int rows(int tile) const { return T - tile * 32 < 32 ? T - tile * 32 : 32; }
  __device__ __forceinline__ f32x4 con4(int k) const { return *(const f32x4 *)(my + C + (j * CN + k) * 4); }
  __device__ __forceinline__ f32x4 gate_consts() const { return con4(0); }
  __device__ __forceinline__ f32x4 taps(int part) const { return con4(4 + 4 * part); }

  // sixteen rows from step t on of one part, zero where there are none, to 1 KB of LDS
  __device__ __forceinline__ void rows_in(const void *from, unsigned char *to, int t, int part) const {
    const int l = lane_again(), step = t + (l >> 2), c0 = wv * 32 + (l & 3) * 8;
    u32x4 v = {0u, 0u, 0u, 0u};
    if (step >= 0 && step < T && c0 < hs) v = *(const u32x4_at2 *)((const unsigned short *)from + (seq + step) * D + part * H + g * hs + c0);
    *(u32x4 *)(to + l * 16) = v;
  }
  // six loads: u of steps -4 .. 31 of a tile
  __device__ __forceinline__ void load_u(int tile) const {
    if constexpr (ANY) {
#pragma unroll
      for (int part = 0; part < 2; ++part) {
        unsigned char *to = my + U + part * U_PART;
        rows_in(p.u, to, tile * 32 - 4, part);
        rows_in(p.u, to + 1024, tile * 32 + 12, part);
        if (lane_again() < 16) rows_in(p.u, to + 2048, tile * 32 + 28, part);
      }
      wave_lds_fence();
      return;
    }
    const int t0 = tile * 32, back = t0 > 0 ? 4 : 0;
    const int l = lane_again(), lrow = l >> 2, c0 = wv * 32 + (l & 3) * 8;
    const bool pc_ok = c0 < hs;
    const unsigned vo = pc_ok ? (unsigned)lrow * row2 + (unsigned)(g * hs + c0) * 2 : OOB;
    const unsigned lead = back ? vo : lrow >= 4 && pc_ok ? vo - 4 * row2 : OOB;
    const u32x4 rs = buf_words((const unsigned short *)p.u + (seq + t0 - back) * D, (size_t)(rows(tile) + back) * row2);
#pragma unroll
    for (int part = 0; part < 2; ++part) {
      const unsigned dst = lds_offset(my) + U + part * U_PART, po = (unsigned)(part * H) * 2;
      lds16<true>(rs, dst, lead, po);
      lds16<true>(rs, dst + 1024, vo, (unsigned)(12 + back) * row2 + po);
      if (l < 16) lds16<true>(rs, dst + 2048, vo, (unsigned)(28 + back) * row2 + po);
    }
  }
  // four loads: dy of a tile's steps
  __device__ __forceinline__ void load_dy(int tile) const {
    if constexpr (ANY) {
#pragma unroll
      for (int part = 0; part < 2; ++part)
#pragma unroll
        for (int m = 0; m < 2; ++m) rows_in(p.dy, my + S + part * 2048 + m * 1024, tile * 32 + 16 * m, part);
      wave_lds_fence();
      return;
    }
    const int l = lane_again(), lrow = l >> 2, c0 = wv * 32 + (l & 3) * 8;
    const unsigned vo = c0 < hs ? (unsigned)lrow * row2 + (unsigned)(g * hs + c0) * 2 : OOB;
    const u32x4 rs = buf_words((const unsigned short *)p.dy + (seq + tile * 32) * D, (size_t)rows(tile) * row2);
#pragma unroll
    for (int part = 0; part < 2; ++part)
#pragma unroll
      for (int m = 0; m < 2; ++m) lds16<true>(rs, lds_offset(my) + S + part * 2048 + m * 1024, vo, (unsigned)(16 * m) * row2 + (unsigned)(part * H) * 2);
  }
  // steps -3 .. -1 of a sequence from the carried ring
  __device__ __forceinline__ void ring_rows() const {
    const int l = lane_again();
    if (l >= 4 && l < 16 && wv * 32 + (l & 3) * 8 < hs)
#pragma unroll
      for (int part = 0; part < 2; ++part)
        *(u32x4 *)(my + U + part * U_PART + l * 16) = *(const u32x4_at2 *)((const unsigned short *)p.state_in +
            ((size_t)b * 3 + ring_slot(p.pos0 + (l >> 2) - 4)) * D + part * H + g * hs + wv * 32 + (l & 3) * 8);
    wave_lds_fence();
  }
  // rows 16 hf + 4 n .. + 3 of the lane's channel
  template <int N>
  __device__ __forceinline__ void rows_of(const unsigned char *t, unsigned (&v)[2 * N]) const {
#pragma unroll
    for (int n = 0; n < N; ++n) {
      const u32x2 q = lds_tr(t + r_rd + (unsigned)(4 * n) * 64);
      v[2 * n] = q[0];
      v[2 * n + 1] = q[1];
    }
  }
  __device__ __forceinline__ void put16(unsigned char *t, const unsigned (&v)[8]) const {
#pragma unroll
    for (int s = 0; s < 2; ++s) *(u32x4 *)(t + t_wr[s]) = u32x4{v[4 * s], v[4 * s + 1], v[4 * s + 2], v[4 * s + 3]};
  }
  // eight of the lane's 16 steps back (the first or the last)
  __device__ __forceinline__ u32x4 get8(const unsigned char *t, int last) const { return *(const u32x4 *)(t + t_wr[last]); }
  __device__ __forceinline__ u32x4 frag(const unsigned char *t) const {
    const u32x2 lo = lds_tr(t + f_rd[0]), hi = lds_tr(t + f_rd[1]);
    return u32x4{lo[0], lo[1], hi[0], hi[1]};
  }
  // [channel][step] tile as rows of one part of a [B][T][D] tensor: two stores
  __device__ __forceinline__ void rows_out(const unsigned char *t, void *out, int tile, int part) const {
    const __amdgpu_buffer_rsrc_t rs = buf((unsigned short *)out + (seq + tile * 32) * D, (size_t)rows(tile) * row2);
    const int l = lane_again(), r4 = (l >> 2) & 3, c4 = l & 3, c0 = wv * 32 + 8 * r4;
    const unsigned vo = c0 < hs ? (unsigned)(4 * (l >> 4) + c4) * row2 + (unsigned)(part * H + g * hs + c0) * 2 : OOB;
#pragma unroll
    for (int m = 0; m < 2; ++m) {
      u32x2 q[2];
#pragma unroll
      for (int n = 0; n < 2; ++n)
        q[n] = lds_tr(t + (unsigned)(8 * c4 + 4 * n + r4) * 64 + (unsigned)(((2 * m + (l >> 5)) ^ key(4 * n + r4)) * 16) + (unsigned)((l >> 4) & 1) * 8);
      const u32x4 v = {q[0][0], q[0][1], q[1][0], q[1][1]};
      if constexpr (ANY) {
        const int step = tile * 32 + 16 * m + 4 * (l >> 4) + c4;
        if (step < T && c0 < hs) *(u32x4_at2 *)((unsigned short *)out + (seq + step) * D + part * H + g * hs + c0) = v;
      } else {
        store16<0>(v, rs, vo, (unsigned)(16 * m) * row2);
      }
    }
  }
  // a lane's 16 steps of one part (or gate), as rglru_wgrad.h has them
  __device__ __forceinline__ void run_out(const unsigned (&v)[8], unsigned short *out, int tile, int part) const {
    const __amdgpu_buffer_rsrc_t rs = buf(out + (((size_t)b * a.ntile + tile) * p.nb + g) * 2 * hs * 32, (size_t)hs * 128);
    const int l = lane_again();
    const unsigned vo = wv * 32 + (l & 31) < hs
        ? (unsigned)(part * hs) * 64 + (unsigned)wv * 2048 + (unsigned)((l >> 4) & 1) * 1024 + (unsigned)(l >> 5) * 512 + (unsigned)(l & 15) * 16 : OOB;
    store16<RGLRU_NT>(u32x4{v[0], v[1], v[2], v[3]}, rs, vo, 0);
    store16<RGLRU_NT>(u32x4{v[4], v[5], v[6], v[7]}, rs, vo + 256, 0);
  }
  // Conv1D of one part: x, and its half-precision parts (as conv_rows_kernel splits them)
  __device__ __forceinline__ void conv(int part, float (&x)[16], unsigned (&hi)[8], unsigned (&lo)[8]) const {
    unsigned uu[10];   // steps -4 .. 15 of the lane's run
    rows_of<5>(my + U + part * U_PART, uu);
    const f32x4 tap = taps(part);
    const float bias = con4(12)[part];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      float v[8], r[8];
      unsigned o[4];
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        v[e] = bias;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const int i = 8 * q + e - k + 4;
          v[e] = fmaf(tap[k], (i & 1) ? bf_hi(uu[i >> 1]) : bf_lo(uu[i >> 1]), v[e]);
        }
        x[8 * q + e] = v[e];
      }
      cvt_f16x8(v, o);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        hi[4 * q + e] = o[e];
        r[2 * e] = fmaf(f16_lo(o[e]), -1.f, v[2 * e]);   // (a product takes half precision as it is)
        r[2 * e + 1] = fmaf(f16_hi(o[e]), -1.f, v[2 * e + 1]);
      }
      cvt_f16x8(r, o);
#pragma unroll
      for (int e = 0; e < 4; ++e) lo[4 * q + e] = o[e];
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  // K-step ks: 16 channels of part ks / 2 & 1 of wave ks / 4; low: the low part
  __device__ __forceinline__ u32x4 frag_at(int ks, bool low) const {
    return frag(smem + (ks >> 2) * REGION + X + ((ks >> 1) & 1) * 2048 + (ks & 1) * 1024 + (low ? 4096 : 0));
  }
};

__device__ __forceinline__ float2 conj2(float2 v) { return make_float2(v.x, -v.y); }
__device__ __forceinline__ void both2(float2 v, float2 &lo, float2 &up) {
  both_halves(v.x, lo.x, up.x);
  both_halves(v.y, lo.y, up.y);
}
__device__ __forceinline__ float2 madd(float2 a, float2 s, float2 e) {   // a s + e
  return make_float2(fmaf(a.x, s.x, fmaf(-a.y, s.y, e.x)), fmaf(a.x, s.y, fmaf(a.y, s.x, e.y)));
}

// The factor of a run's map: the product of a~_t over steps whose r_t sum to rsum, as |a~_t| and its phase are exponentials of r_t.
// (Up to 64 revolutions and more: the state is as far off as with the product of 16 factors, 6e-6 : 8e-6 at theta up to 0.314, 5.0e-5 : 5.3e-5
// up to pi, 4.2e-3 : 4.2e-3 up to 30, T 1000 - 2048 - each step's own phase, rounded alike in both, is what counts.)
__device__ __forceinline__ float2 run_decay(const Decay &k, float rsum) {
  float l2, mod;
  return cdecay(k, rsum, l2, mod);
}

// host side
struct CgInstance {
  const void *agg, *bagg, *y, *bwd;
  int nct;
};
CgInstance cg_instance_fwd(int nct, bool any);   // agg, y
CgInstance cg_instance_bwd(int nct, bool any);   // bagg, bwd
CgInstance cg_instance_fwd_any(int nct);
const void *cg_instance_bwd_any(int nct);

}  // namespace cgt
}  // namespace rglru
