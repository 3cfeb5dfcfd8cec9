// The forward in tiles, the counterpart of rglru_bwd_fused.h (layouts and helpers are described there): a workgroup
// takes a tile of 32 MT steps of a gate block, a wave 32 of its channels, and walks its share of a sequence
// forwards:
//   u -> Conv1D -> x (fp32 in registers, half precision in LDS)
//   p, q = x W_a^T, x W_x^T            matrix cores; x from LDS, weights from L2 in fragment order
//   a_t, b_t = m_t i_t x_t, the tile's aggregate of h_t = a_t h_{t-1} + b_t; the state entering the tile from
//   this workgroup's registers or from the records of the slices in front; y (the merge)
// Nothing but u (and branch) is read and nothing but y (and out) written. In passes the same forward stored x, log a_t
// and b_t and read them back: B 4 T 2048, 16 blocks of 352 channels, 266 us before (gates 155, decays 54, Conv1D 48), 165
// now with everything; 16 blocks of 448 channels 338 and 227.
// What bounds it: the vector unit (about 25 instructions per element, 6 of them transcendental) where workgroups
// are many, the weights' way from L2 (2 KB per K-step and wave) where a tile is 32 steps of a wide block, and the
// exchange of records where a single sequence is cut into as many slices as the chip holds.
// u lies in two places by turns: the next tile's direct-to-LDS loads start behind the products, in front of the
// gates and the wait for records, and the place of the tile in hand takes y on its way out.
#pragma once
#include "rglru_bwd_fused.h"

namespace rglru {
namespace fused {

constexpr int FWD_TILE_SLICES = 32;   // at most
struct FwdTileArgs {
  Problem p;
  int G, ntile, R;
  unsigned total;
  u64 *rec;
  int *err;
  const u32x4 *wg;            // weights in fragment order, [nb][wave][K-step][gate][lane]
  const uint4 *rmask;         // packed sequences: boundary bit masks per 32 steps, or null
  int nmask;
};

template <int MT, int VAR>
struct FwdLds {
  static constexpr bool MERGE = VAR == V_MERGE || VAR == V_MERGE_TANH;
  static constexpr int TM = 32 * MT, UROWS = TM + 16, UB = UROWS * 64;
  // two places for u, in turn (the one in hand becomes the staging tile of y); x; branch; constants
  static constexpr int U = 0, X = 2 * UB, B = X + TM * 64, C = B + (MERGE ? TM * 64 : 0), REGION = C + 32 * 48;
};

template <int NCT, int MT, int VAR, int WPE, int PD>
__global__ void __launch_bounds__(NCT * 64) __attribute__((amdgpu_waves_per_eu(WPE, WPE))) fwd_tile_kernel(FwdTileArgs a) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  typedef FwdLds<MT, VAR> L;
  constexpr bool MERGE = L::MERGE, PACKED = VAR == V_PACKED;
  constexpr int TM = L::TM, NKS = 2 * NCT;
  const Problem &p = a.p;
  const unsigned id = xcd_id();
  if (id >= a.total) return;
  const int tid = threadIdx.x, lane = tid & 63, hf = lane >> 5, j = lane & 31;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int G = a.G, w = __builtin_amdgcn_readfirstlane((int)(id % G)), gb = __builtin_amdgcn_readfirstlane((int)(id / G));
  const int b = __builtin_amdgcn_readfirstlane(gb % p.B), g = __builtin_amdgcn_readfirstlane(gb / p.B);
  const int D = p.D, T = p.T, bs = p.bs;
  const bool ok = wv * 32 + j < bs;
  const int d = g * bs + (ok ? wv * 32 + j : bs - 1);
  const unsigned row2 = (unsigned)D * 2;
  unsigned char *my = smem + wv * L::REGION;
  // per-channel constants: b_a, b_x, c log(sigma(Lambda)), conv_b | taps
  if (hf == 0) {
    f32x4 v = {0.f, 0.f, 0.f, 0.f}, t = {0.f, 0.f, 0.f, 0.f};
    if (ok) {
      v = f32x4{p.b_a[d], p.b_x[d], neg_c_softplus(p.Lambda[d], p.c), p.conv_b ? p.conv_b[d] : 0.f};
#pragma unroll
      for (int k = 0; k < 4; ++k) t[k] = p.conv_w ? p.conv_w[(size_t)k * D + d] : (k == 0 ? 1.f : 0.f);
    }
    *(f32x4 *)(my + L::C + j * 48) = v;
    *(f32x4 *)(my + L::C + j * 48 + 16) = t;
  }
  wave_lds_fence();

  auto lane_again = [&]() __attribute__((always_inline)) {
    int l = lane;
    asm volatile("" : "+v"(l));
    return l;
  };
  const size_t seq = (size_t)b * T;
  const int i16 = lane & 15, q16 = (lane >> 4) & 1, a4 = i16 >> 2, cc = i16 & 3;
  const unsigned r_rd = (unsigned)(hf * 16 + a4) * 64 + (unsigned)q16 * 32 + (unsigned)cc * 8;
  auto key = [](int c) { return (c >> 1) & 3; };
  unsigned t_wr[2], f_rd[2];
#pragma unroll
  for (int n = 0; n < 2; ++n) {
    t_wr[n] = (unsigned)j * 64 + (unsigned)((hf * 2 + n) ^ key(j)) * 16;
    f_rd[n] = (unsigned)(hf * 8 + 4 * n + a4) * 64 + (unsigned)((((cc & 1) * 2 + q16) ^ key(4 * n + a4)) * 16) + (unsigned)(cc >> 1) * 8;
  }
  const unsigned wbytes = (unsigned)NKS * 2 * 1024;
  const __amdgpu_buffer_rsrc_t w_rs = buf((const char *)a.wg + (size_t)(g * NCT + wv) * wbytes, wbytes);
  f16x8 wq[PD][2];
  auto load_w = [&](int ks) __attribute__((always_inline)) {
#pragma unroll
    for (int gt = 0; gt < 2; ++gt)
      wq[ks % PD][gt] = __builtin_bit_cast(f16x8, __builtin_amdgcn_raw_buffer_load_b128(w_rs, (unsigned)lane * 16, (unsigned)(ks * 2 + gt) * 1024, 0));
  };
  constexpr int NU = L::UROWS / 16;
  unsigned ux = 0;   // where u of the tile in hand lies
  // u into the place that is not in use (staged row s is step t0 - 4 + s), branch into its own
  auto load_tile = [&](int tile) __attribute__((always_inline)) {
    const int t0 = tile * TM, back = t0 > 0 ? 4 : 0;
    const unsigned nrow = T - t0 < TM ? T - t0 : TM, at = lds_offset(smem) + (unsigned)wv * L::REGION;
    const int l = lane_again(), lrow = l >> 2, c0 = wv * 32 + (l & 3) * 8;
    const bool pc_ok = c0 < bs;
    const unsigned vo = pc_ok ? (unsigned)lrow * row2 + (unsigned)(g * bs + c0) * 2 : OOB;
    const unsigned lead = back ? vo : lrow >= 4 && pc_ok ? vo - 4 * row2 : OOB;
    const u32x4 rs = buf_words((const unsigned short *)p.u + (seq + t0 - back) * D, (size_t)(nrow + back) * row2);
    const unsigned dst = at + L::U + (ux ^ L::UB);
    lds16<true>(rs, dst, lead, 0);
#pragma unroll
    for (int m = 1; m < NU; ++m)
      lds16<true>(rs, dst + m * 1024, m == NU - 1 && l >= 16 ? OOB : vo, (unsigned)(16 * m - 4 + back) * row2);
    if constexpr (MERGE) {
      const u32x4 b_rs = buf_words((const unsigned short *)p.branch + (seq + t0) * D, (size_t)nrow * row2);
#pragma unroll
      for (int m = 0; m < TM / 16; ++m) lds16<true>(b_rs, at + L::B + m * 1024, vo, (unsigned)(16 * m) * row2);
    }
  };
  auto rows_of = [&](const unsigned char *t, int rb, int cnt, unsigned *v) __attribute__((always_inline)) {
#pragma unroll
    for (int n = 0; n < cnt; ++n) {
      const u32x2 q = lds_tr(t + r_rd + (unsigned)(rb * 32 + 4 * n) * 64);
      v[2 * n] = q[0];
      v[2 * n + 1] = q[1];
    }
  };
  auto put16 = [&](unsigned char *t, int rb, const unsigned (&v)[8]) __attribute__((always_inline)) {
#pragma unroll
    for (int s = 0; s < 2; ++s) *(u32x4 *)(t + t_wr[s] + rb * 2048) = u32x4{v[4 * s], v[4 * s + 1], v[4 * s + 2], v[4 * s + 3]};
  };
  auto frag = [&](const unsigned char *t, int rb) __attribute__((always_inline)) {
    const u32x2 lo = lds_tr(t + f_rd[0] + rb * 2048), hi = lds_tr(t + f_rd[1] + rb * 2048);
    return __builtin_bit_cast(f16x8, (u32x4){lo[0], lo[1], hi[0], hi[1]});
  };
  auto rows_out = [&](const unsigned char *t, void *out, int t0, unsigned nrow) __attribute__((always_inline)) {
    const __amdgpu_buffer_rsrc_t rs = buf((unsigned short *)out + (seq + t0) * D, (size_t)nrow * row2);
    const int l = lane_again(), r4 = (l >> 2) & 3, c4 = l & 3, c0 = wv * 32 + 8 * r4;
    unsigned s_rd[2][2];
#pragma unroll
    for (int n = 0; n < 2; ++n)
#pragma unroll
      for (int m = 0; m < 2; ++m)
        s_rd[n][m] = (unsigned)(8 * c4 + 4 * n + r4) * 64 + (unsigned)(((2 * m + (l >> 5)) ^ key(4 * n + r4)) * 16) + (unsigned)((l >> 4) & 1) * 8;
    const unsigned s_vo = c0 < bs ? (unsigned)(4 * (l >> 4) + c4) * row2 + (unsigned)(g * bs + c0) * 2 : OOB;
#pragma unroll
    for (int m = 0; m < TM / 16; ++m) {
      const unsigned char *at = t + (m >> 1) * 2048;
      const u32x2 lo = lds_tr(at + s_rd[0][m & 1]), hi = lds_tr(at + s_rd[1][m & 1]);
      store16<0>((u32x4){lo[0], lo[1], hi[0], hi[1]}, rs, s_vo, (unsigned)(16 * m) * row2);
    }
  };

  float carry = ok && p.h0 ? p.h0[(size_t)b * D + d] : 0.f;   // the state entering this workgroup's next tile
  int spins = G > 1 && expired_before(a.err) ? SPIN_LIMIT : 0;
  int tile = w;
  if (tile < a.ntile) load_tile(tile);
  for (; tile < a.ntile; tile += G) {
    const int t0 = tile * TM;
    const unsigned nrow = T - t0 < TM ? T - t0 : TM;
    ux ^= L::UB;
    // (the tile's loads have landed; only the last stores may still be under way)
    if (tile == w) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    else asm volatile("s_waitcnt vmcnt(%0)" :: "n"(TM / 16) : "memory");
#pragma unroll
    for (int ks = 0; ks < PD; ++ks) load_w(ks);
    unsigned char *mu = my + L::U + ux;
    if (t0 == 0 && p.state_in) {   // steps -3 .. -1 from the carried ring
      const int l = lane_again();
      if (l >= 4 && l < 16 && wv * 32 + (l & 3) * 8 < bs)
        *(u32x4 *)(mu + l * 16) = *(const u32x4_at2 *)((const unsigned short *)p.state_in +
            ((size_t)b * 3 + ring_slot(p.pos0 + (l >> 2) - 4)) * D + g * bs + wv * 32 + (l & 3) * 8);
      wave_lds_fence();
    }
    unsigned st16[MT], lag[MT][4];
    if constexpr (PACKED) {
#pragma unroll
      for (int rb = 0; rb < MT; ++rb) {
        const int wd = tile * MT + rb;
        const uint4 v = wd < a.nmask ? a.rmask[(size_t)b * a.nmask + wd] : make_uint4(0u, 0u, 0u, 0u);
        st16[rb] = hf ? v.x >> 16 : v.x;
        lag[rb][1] = hf ? v.y >> 16 : v.y;
        lag[rb][2] = hf ? v.z >> 16 : v.z;
        lag[rb][3] = hf ? v.w >> 16 : v.w;
      }
    }
    // ---- Conv1D
    const bool ragged = (int)nrow < TM;
    auto left = [&]() __attribute__((always_inline)) { return (int)nrow - (lane_again() >> 5) * 16; };   // of this lane's steps (of row block 0)
    float x[MT][16];
    unsigned pk[MT][8];
    {
      const f32x4 tap = *(const f32x4 *)(my + L::C + j * 48 + 16);
      const float cbias = *(const float *)(my + L::C + j * 48 + 12);
#pragma unroll
      for (int rb = 0; rb < MT; ++rb) {
        unsigned uu[10];   // u of steps -4 .. 15 of the lane's run
        rows_of(mu, rb, 5, uu);
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          float v[8];
          unsigned o[4];
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            const int r = 8 * h + e;
            v[e] = cbias;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
              const int i = r - k + 4;
              float ui = (i & 1) ? bf_hi(uu[i >> 1]) : bf_lo(uu[i >> 1]);
              if (PACKED && k > 0) ui = ((lag[rb][k] >> r) & 1u) ? ui : 0.f;
              v[e] = fmaf(tap[k], ui, v[e]);
            }
            x[rb][r] = v[e];
          }
          cvt_f16x8(v, o);
#pragma unroll
          for (int e = 0; e < 4; ++e) pk[rb][4 * h + e] = o[e];
          __builtin_amdgcn_sched_barrier(0);
        }
        if (ragged) {   // nothing of the steps past the end
          const int valid = left();
#pragma unroll
          for (int r = 0; r < 16; ++r)
            if (r + rb * 32 >= valid) x[rb][r] = 0.f;
        }
      }
    }
    lds_barrier();   // (every wave has read the last tile's x)
#pragma unroll
    for (int rb = 0; rb < MT; ++rb) put16(my + L::X, rb, pk[rb]);
    lds_barrier();   // x is there

    // ---- gate pre-activations
    f32x16 accp[MT], accq[MT];
    const f32x4 con = *(const f32x4 *)(my + L::C + j * 48);
    // (finite, so that times the r_t = 0 of a closed gate it is 0 and not a NaN)
    const float kd = con[2] * LOG2E < -3e38f ? -3e38f : con[2] * LOG2E;
#pragma unroll
    for (int rb = 0; rb < MT; ++rb)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        accp[rb][r] = con[0];
        accq[rb][r] = con[1];
      }
    {
      f16x8 fa[2][MT];
#pragma unroll
      for (int rb = 0; rb < MT; ++rb) fa[0][rb] = frag(smem + L::X, rb);
#pragma unroll
      for (int ks = 0; ks < NKS; ++ks) {
        if (ks + 1 < NKS)
#pragma unroll
          for (int rb = 0; rb < MT; ++rb)
            fa[(ks + 1) & 1][rb] = frag(smem + L::X + ((ks + 1) >> 1) * L::REGION + ((ks + 1) & 1) * 1024, rb);
#pragma unroll
        for (int rb = 0; rb < MT; ++rb) {
          accp[rb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(fa[ks & 1][rb], wq[ks % PD][0], accp[rb], 0, 0, 0);
          accq[rb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(fa[ks & 1][rb], wq[ks % PD][1], accq[rb], 0, 0, 0);
        }
        if (ks + PD < NKS) load_w(ks + PD);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    // Steps past the end: closed gates, a_t = 1 and m_t = i_t = 0, leave the state untouched. (Set behind the products:
    // the Conv1D reaches back into the sequence there, and an infinity among its last inputs would come through.)
    if (ragged) {
      const int valid = left();
#pragma unroll
      for (int rb = 0; rb < MT; ++rb)
#pragma unroll
        for (int r = 0; r < 16; ++r)
          if (r + rb * 32 >= valid) accp[rb][r] = accq[rb][r] = -__builtin_huge_valf();
    }
    // the next tile's inputs, in front of the longest stretch that needs nothing from memory
    unsigned br[MERGE ? MT : 1][8];
    if constexpr (MERGE)
#pragma unroll
      for (int rb = 0; rb < MT; ++rb) rows_of(my + L::B, rb, 4, br[rb]);
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    if (tile + G < a.ntile) load_tile(tile + G);

    // ---- a_t, b_t (in place of p, q) and the aggregate of the tile
    float A_lo[MT], H_lo[MT], A_rb[MT], H_rb[MT];
#pragma unroll
    for (int rb = 0; rb < MT; ++rb) {
      if constexpr (PACKED) asm volatile("" : "+v"(st16[rb]));
      float A = 1.f, H = 0.f;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const float l2 = kd * __builtin_amdgcn_rcpf(1.f + __builtin_amdgcn_exp2f(-LOG2E * accp[rb][r]));
        float av = __builtin_amdgcn_exp2f(l2);
        const float ig = __builtin_amdgcn_rcpf(1.f + __builtin_amdgcn_exp2f(-LOG2E * accq[rb][r]));
        const float bv = __builtin_amdgcn_sqrtf(fmaxf(one_minus_sq(av, l2), 0.f)) * ig * x[rb][r];
        if (PACKED && ((st16[rb] >> r) & 1u)) av = 0.f;   // nothing flows into a document's first step
        accp[rb][r] = av;
        accq[rb][r] = bv;
        H = fmaf(av, H, bv);
        A *= av;
        if (r % 4 == 3) __builtin_amdgcn_sched_barrier(0);
      }
      float A_up, H_up;
      both_halves(A, A_lo[rb], A_up);
      both_halves(H, H_lo[rb], H_up);
      A_rb[rb] = A_up * A_lo[rb];
      H_rb[rb] = fmaf(A_up, H_lo[rb], H_up);
    }
    float A_t = A_rb[0], H_t = H_rb[0];
    if (MT == 2) {
      H_t = fmaf(A_rb[MT - 1], H_t, H_rb[MT - 1]);
      A_t *= A_rb[MT - 1];
    }
    float h_in = carry;
    if (G > 1) {
      const int c_ = wv * 32 + (lane_again() & 31);
      u64 *ring = a.rec + (size_t)gb * a.R * (NCT * 32) + c_;
      if (hf == 0) publish(ring + slot_of(tile, a.R) * (NCT * 32), A_t, H_t, epoch_of(tile, a.R));
      // the state behind tile - G, carried across tiles tile - G + 1 .. tile - 1: each lane half fetches and composes
      // half of the records, four per round trip
      const RecWalk<1> wk(tile - (G - 1), G - 1, hf, a.R);
      const int nrec = G >> 1;
      float rA = 1.f, rH = 0.f;
      for (int s0 = 0; s0 < nrec; s0 += 4) {
        u64 rec[4];
        unsigned want;
#pragma unroll
        for (int i = 0; i < 4; ++i) rec[i] = peek(ring + (size_t)wk.slot_at(s0 + i, want) * (NCT * 32));
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const u64 *slot = ring + (size_t)wk.slot_at(s0 + i, want) * (NCT * 32);
          const bool has = wk.has(s0 + i, a.ntile);
          while (has && rec_epoch(rec[i]) != want && spins < SPIN_LIMIT) {
            ++spins;
            __builtin_amdgcn_s_sleep(2);
            rec[i] = peek(slot);
          }
          if (spins < SPIN_LIMIT) spins = 0;   // the limit is per wait; an expired wait stays expired
          const float A = has ? rec_A(rec[i]) : 1.f, H = has ? rec_H(rec[i]) : 0.f;
          rH = fmaf(A, rH, H);
          rA *= A;
        }
      }
      const float xA = __shfl_xor(rA, 32), xH = __shfl_xor(rH, 32);
      h_in = fmaf(hf ? xA : rA, h_in, hf ? xH : rH);   // (the lower half's tiles come first)
      h_in = fmaf(hf ? rA : xA, h_in, hf ? rH : xH);
      if (spins >= SPIN_LIMIT || __shfl_xor(spins, 32) >= SPIN_LIMIT) h_in = __builtin_nanf("");
    }
    carry = fmaf(A_t, h_in, H_t);
    // ---- y, through the room of u
    float h_blk = h_in;
    unsigned yo[MT][8];
#pragma unroll
    for (int rb = 0; rb < MT; ++rb) {
      float h = hf ? fmaf(A_lo[rb], h_blk, H_lo[rb]) : h_blk;
      h_blk = fmaf(A_rb[rb], h_blk, H_rb[rb]);
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        const float h0 = fmaf(accp[rb][2 * q], h, accq[rb][2 * q]);
        h = fmaf(accp[rb][2 * q + 1], h0, accq[rb][2 * q + 1]);
        yo[rb][q] = pack_bf16(h0, h);
      }
    }
    if (!MERGE || p.y) {
#pragma unroll
      for (int rb = 0; rb < MT; ++rb) put16(mu, rb, yo[rb]);
      wave_lds_fence();
      rows_out(mu, p.y, t0, nrow);
      wave_lds_fence();
    }
    if constexpr (MERGE) {   // the product of y as stored and GeLU(branch)
#pragma unroll
      for (int rb = 0; rb < MT; ++rb) {
        unsigned o[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) {
          o[q] = pack_bf16(bf_lo(yo[rb][q]) * gelu<VAR == V_MERGE_TANH, true>(bf_lo(br[rb][q])),
                           bf_hi(yo[rb][q]) * gelu<VAR == V_MERGE_TANH, true>(bf_hi(br[rb][q])));
          if (q & 1) __builtin_amdgcn_sched_barrier(0);
        }
        put16(mu, rb, o);
      }
      wave_lds_fence();
      rows_out(mu, p.out, t0, nrow);
      wave_lds_fence();
    }
  }
  if (spins >= SPIN_LIMIT) mark_expired(a.err);
  // ---- the workgroup of the last tile hands on the state and the last three inputs (every other workgroup has read
  // the incoming ones: all tiles' records have been consumed)
  if ((a.ntile - 1) % G != w || !ok || hf) return;
  const int dd = g * bs + wv * 32 + (lane_again() & 31);
  if (p.hT) p.hT[(size_t)b * D + dd] = carry;
  if (!p.state_out) return;
  unsigned short *so = (unsigned short *)p.state_out + (size_t)b * 3 * D + dd;
  const unsigned short *si = p.state_in ? (const unsigned short *)p.state_in + (size_t)b * 3 * D + dd : nullptr;
  const long long end = p.pos0 + T;
  for (int slot = 0; slot < 3; ++slot) {   // older slots are carried over
    const long long npos = end - 1 - ring_slot(end - 1 - slot), t = npos - p.pos0;
    unsigned short v = 0;
    if (t >= 0) v = ((const unsigned short *)p.u)[(seq + t) * D + dd];
    else if (si) v = si[(size_t)slot * D];
    if (PACKED)   // an input in front of the last document's first step is not part of its history
      for (int k = t + 1 > 0 ? (int)t + 1 : 0; k < T; ++k)
        if (p.reset[seq + k]) v = 0;
    so[(size_t)slot * D] = v;
  }
}

template <int NCT, int MT, int VAR, int WPE, int PD>
Instance fwd_instance() {
  constexpr int lds = NCT * FwdLds<MT, VAR>::REGION, by_lds = 160 * 1024 / lds, by_waves = NCT == 5 ? 2 : 4 * WPE / NCT;
  // (five waves: with three workgroups to a CU the slices, not the chip, set the pace; 160 channels, B 4 T 512: 32 us, with two 25)
  if constexpr (lds <= 160 * 1024) return {(const void *)fwd_tile_kernel<NCT, MT, VAR, WPE, PD>, NCT, MT, lds, by_lds < by_waves ? by_lds : by_waves};
  else return {nullptr, 0, 0, 0, 0};
}
template <int NCT, int MT, int WPE, int PD, int MTM, int WPEM>   // (MTM, WPEM: with the merge)
Instance fwd_pick(int var) {
  if (var == V_PLAIN) return fwd_instance<NCT, MT, V_PLAIN, WPE, PD>();
  if constexpr (NCT <= 8) {   // (packed rows: 128 - 256 channels)
    if (var == V_PACKED) return fwd_instance<NCT, MT, V_PACKED, WPE, PD>();
  } else {
    if (var == V_PACKED) return {nullptr, 0, 0, 0, 0};
  }
  return var == V_MERGE ? fwd_instance<NCT, MTM, V_MERGE, WPEM, PD>() : fwd_instance<NCT, MTM, V_MERGE_TANH, WPEM, PD>();
}
Instance find_fwd_instance_a(int nct, int var);   // 4 - 6
Instance find_fwd_instance_b(int nct, int var);   // 7, 8
Instance find_fwd_short_instance(int nct, int var);   // 7, 8: tiles of 32 steps
Instance find_fwd_instance_c(int nct, int var);   // 9 - 12
Instance find_fwd_instance_d(int nct, int var);   // 13 - 15

// the weights (wd null: not transposed) in fragment order, the status word, `nrec` 16-byte words of records cleared,
// the scale (sc null: none)
hipError_t launch_tile_prep(const Problem &p, int nct, u32x4 *wg, u32x4 *wd, void *status, void *rec, size_t nrec, float *sc, hipStream_t s);
hipError_t configure(const Instance &in);
int compute_units();

}  // namespace fused
}  // namespace rglru
