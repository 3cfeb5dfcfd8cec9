// The backward in tiles: one kernel per block size for everything but the weight gradients.
// Instances are compiled in translation units of their own (rglru_bwd_fused_*.hip).
//
// A workgroup takes a tile of TM = 32 MT steps of one gate block, a wave 32 of its channels, and
// walks its share of a sequence backwards in time:
//   u -> Conv1D -> x (fp32 in registers, half precision in LDS for all waves)
//   p, q = x W_a^T, x W_x^T            matrix cores; x from LDS, weights from L2 in fragment order
//   gates, decays, the tile's aggregate of eps_t = a_t (dy_t + eps_{t+1}); the state entering the
//   tile from this workgroup's registers or, where a sequence is sliced in time, from the records of
//   the slices in front
//   S eps, the adjoints of eqs. (1)-(4): S dp, S dq (half precision, to LDS), S dxd (fp32, registers)
//   S dx = S dxd + [S dp | S dq] [W_a | W_x]      matrix cores
//   du and the tap sums, the Conv1D's adjoint
// so that logits, dxd and dx never leave the registers; what the weight gradients need (x, S dp, S dq)
// leaves from registers in the order of their matrix fragments (rglru_wgrad.h).
// B 16 T 4096, 16 blocks of 256 channels: 1.2 ms for what took two kernels 1.65 ms (gates and adjoints 1.12, products
// and Conv1D 0.54), 1.68 GB read and 2.15 GB written, which is what goes in and out, 3.9 and 2.3 GB before. Bound by the
// vector unit (busy 60 % of the time: some 60 instructions per element, 10 of them transcendental) and what two waves
// per SIMD cannot hide of the barriers around the two products. Tiles of 64 steps where registers allow two waves
// per SIMD to hold them (halves the weights' way from L2), of 32 elsewhere.
//
// Layouts. Each wave owns a region of LDS: U (u as it comes, 64 bytes a row and four rows in front; then S dq as
// [channel][step]), X (x as [channel][step]; then S dp; then du), Y, DY (y and dy as they come), with the merge B
// (branch; then dbranch). Staged rows and [channel][step] tiles are both read with the transposing LDS read
// (16 lanes x 8 bytes: 4 rows x 16 columns -> 4 rows of a column per lane): rows give a lane 16
// consecutive steps of its channel, [channel][step] tiles give a matrix fragment (a step per lane,
// 8 consecutive channels). Pieces of 16 bytes are permuted by the channel so that both sides of each
// tile spread over the banks.
#pragma once
#include "rglru_gelu.h"
#include "rglru_pass.h"

namespace rglru {
namespace fused {
using namespace pass;

struct FusedArgs {
  Problem p;
  int G, ntile, R;            // time slices per (sequence, block), tiles per sequence, slots of a record ring
  unsigned total;             // workgroups
  u64 *rec;
  int *err;
  const u32x4 *wg, *wd;       // weights in fragment order, [nb][wave][K-step][gate][lane]: as they are, transposed
  unsigned short *xT, *pqT;   // half precision x, S dp | S dq in stages of 32 steps (rglru_wgrad.h)
  const float *sc;            // sc[1] = S, sc[2] = 1 / S
  float *partA, *partC;       // [B G][3][D] sums for db_a, db_x, dLambda; [B G][5][D] for dconv_w, dconv_b
  float *edge;                // [B][ntile][6][D]: S dx of a tile's first and last three rows (sliced in time), or null
  const uint4 *rmask;         // packed sequences: boundary bit masks per 32 steps, or null
  int nmask;                  // their number per sequence
};

constexpr int V_PLAIN = 0, V_MERGE = 1, V_MERGE_TANH = 2, V_PACKED = 3;
template <int MT, int VAR, bool TIGHT = false>
struct Lds {
  static constexpr bool MERGE = VAR == V_MERGE || VAR == V_MERGE_TANH;
  static constexpr int TM = 32 * MT;
  // The loads come in sixteens; TM + 4 rows are used. TIGHT: there is no room for the others (512 channels: 16 waves in
  // 160 KB), and their lanes are switched off.
  static constexpr int UROWS = TM + (TIGHT ? 4 : 16);
  static constexpr int U = 0, X = UROWS * 64, Y = X + TM * 64, DY = Y + (MERGE ? UROWS : TM) * 64, B = DY + TM * 64,
                       C = B + (MERGE ? TM * 64 : 0);   // constants of the wave's channels: 12 floats each
  static constexpr int P = X, Q = U;     // S dp, S dq: where x and u lay
  static constexpr int REGION = C + 32 * 48;
};

// a barrier for LDS alone: loads to and stores from registers stay in flight across it
__device__ __forceinline__ void lds_barrier() {
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}
// the value of this channel's lower and of its upper lane half, in both
__device__ __forceinline__ void both_halves(float v, float &lo, float &up) {
  const unsigned w = __float_as_uint(v);
  const auto r = __builtin_amdgcn_permlane32_swap(w, w, false, false);
  lo = __uint_as_float(r[0]);
  up = __uint_as_float(r[1]);
}
// e^-v for a logit v, kept below infinity (1 / (1 + e^-v) times e^-v is then 1 where the gate is closed) but not a NaN
__device__ __forceinline__ float gate_exp(float v) {
  return __builtin_amdgcn_exp2f(__builtin_elementwise_minimum(-LOG2E * v, 126.f));
}
// Eight values to half precision, to nearest; finite ones stop at 65504, infinities and NaNs stay: MODE.FP16_OVFL
// does that in the conversion itself. It is set around the conversions only, because the matrix
// instructions heed it too (a NaN in their third operand is lost under it).
__device__ __forceinline__ void cvt_f16x8(const float (&v)[8], unsigned (&o)[4]) {
  asm("s_setreg_imm32_b32 hwreg(HW_REG_MODE, 23, 1), 1\n\t"
      "v_cvt_pk_f16_f32 %0, %4, %5\n\t"
      "v_cvt_pk_f16_f32 %1, %6, %7\n\t"
      "v_cvt_pk_f16_f32 %2, %8, %9\n\t"
      "v_cvt_pk_f16_f32 %3, %10, %11\n\t"
      "s_setreg_imm32_b32 hwreg(HW_REG_MODE, 23, 1), 0"
      : "=&v"(o[0]), "=&v"(o[1]), "=&v"(o[2]), "=&v"(o[3])
      : "v"(v[0]), "v"(v[1]), "v"(v[2]), "v"(v[3]), "v"(v[4]), "v"(v[5]), "v"(v[6]), "v"(v[7]));
}

// NCT: waves = 32-channel tiles of the block; MT: 32-step tiles; WPE: waves per SIMD; PD: K-steps of weights in flight; K: what stays in registers
// until the adjoints instead of being formed again (1: x, 2: a, too)
template <int NCT, int MT, int VAR, int WPE, int PD, int K>
__global__ void __launch_bounds__(NCT * 64) __attribute__((amdgpu_waves_per_eu(WPE, WPE))) bwd_tile_kernel(FusedArgs a) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  constexpr bool TIGHT = NCT == 16;
  typedef Lds<MT, VAR, TIGHT> L;
  constexpr bool MERGE = L::MERGE, PACKED = VAR == V_PACKED, KEEP = K >= 1, KEEPA = K >= 2;
  constexpr int TM = L::TM, NKS = 2 * NCT;
  const Problem &p = a.p;
  const unsigned id = xcd_id();
  if (id >= a.total) return;
  const int tid = threadIdx.x, lane = tid & 63, hf = lane >> 5, j = lane & 31;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int G = a.G, w = __builtin_amdgcn_readfirstlane((int)(id % G)), gb = __builtin_amdgcn_readfirstlane((int)(id / G));
  const int b = __builtin_amdgcn_readfirstlane(gb % p.B), g = __builtin_amdgcn_readfirstlane(gb / p.B);   // (neighbouring workgroups share a block's weights)
  const int D = p.D, T = p.T, bs = p.bs;
  const int ch = wv * 32 + j;
  const bool ok = ch < bs;                         // (channels past the block: zero inputs, weights and constants)
  const int d = g * bs + (ok ? ch : bs - 1);
  const unsigned row2 = (unsigned)D * 2;
  unsigned char *my = smem + wv * L::REGION;

  // ---- per-channel constants
  const float S = a.sc[1], invS = a.sc[2];
  // (in LDS: registers are what this kernel is short of) b_a, b_x, c log(sigma(Lambda)), conv_b | taps
  if (hf == 0) {
    f32x4 v = {0.f, 0.f, 0.f, 0.f}, t = {0.f, 0.f, 0.f, 0.f};
    if (ok) {
      v = f32x4{p.b_a[d], p.b_x[d], neg_c_softplus(p.Lambda[d], p.c), p.conv_b ? p.conv_b[d] : 0.f};
#pragma unroll
      for (int k = 0; k < 4; ++k) t[k] = p.conv_w ? p.conv_w[(size_t)k * D + d] : (k == 0 ? 1.f : 0.f);
    }
    *(f32x4 *)(my + L::C + j * 48) = v;
    *(f32x4 *)(my + L::C + j * 48 + 16) = t;
    *(float *)(my + L::C + j * 48 + 32) = ok && p.h0 ? p.h0[(size_t)b * D + d] : 0.f;   // h_{-1}
  }
  wave_lds_fence();

  // ---- addresses (those that are used once a tile are formed again there, from a lane id the compiler cannot see
  // through: it would keep them in registers across the loop)
  auto lane_again = [&]() __attribute__((always_inline)) {
    int l = lane;
    asm volatile("" : "+v"(l));
    return l;
  };
  const size_t seq = (size_t)b * T;
  // transposing reads of staged rows: lane (j, hf) gets rows 16 hf + 4 n .. + 3 of channel j
  const int i16 = lane & 15, q16 = (lane >> 4) & 1, a4 = i16 >> 2, cc = i16 & 3;
  const unsigned r_rd = (unsigned)(hf * 16 + a4) * 64 + (unsigned)q16 * 32 + (unsigned)cc * 8;
  // [channel][step] tiles, 32 steps each (64 bytes a row, 2 KB): the 16-byte piece i of channel c lies at piece i ^ key(c)
  auto key = [](int c) { return (c >> 1) & 3; };
  unsigned t_wr[2], f_rd[2];
#pragma unroll
  for (int n = 0; n < 2; ++n) {
    // a lane's own 16 steps
    t_wr[n] = (unsigned)j * 64 + (unsigned)((hf * 2 + n) ^ key(j)) * 16;
    // fragments: lane -> step perm_row(lane & 31), channels 8 hf .. + 7 of a K-step's 16 in two reads
    f_rd[n] = (unsigned)(hf * 8 + 4 * n + a4) * 64 + (unsigned)((((cc & 1) * 2 + q16) ^ key(4 * n + a4)) * 16) + (unsigned)(cc >> 1) * 8;
  }

  // ---- weights: fragments of this wave's 32 columns, a kilobyte each
  const unsigned wbytes = (unsigned)NKS * 2 * 1024;
  const __amdgpu_buffer_rsrc_t wg_rs = buf((const char *)a.wg + (size_t)(g * NCT + wv) * wbytes, wbytes),
                               wd_rs = buf((const char *)a.wd + (size_t)(g * NCT + wv) * wbytes, wbytes);
  f16x8 wq[PD][2];
  auto load_w = [&](const __amdgpu_buffer_rsrc_t &rs, int ks) __attribute__((always_inline)) {
#pragma unroll
    for (int gt = 0; gt < 2; ++gt)
      wq[ks % PD][gt] = __builtin_bit_cast(f16x8, __builtin_amdgcn_raw_buffer_load_b128(rs, (unsigned)lane * 16,
                                                                                       (unsigned)(ks * 2 + gt) * 1024, 0));
  };

  // ---- a tile's inputs, straight into the wave's own rows of LDS (nothing else reads them, so that a wave waits for
  // its own loads only). NU loads of u, NY of y, TM / 16 of dy, as many of the other branch.
  constexpr int NU = TM / 16 + 1, NY = MERGE ? NU : TM / 16;
  constexpr int LOAD_U = 1, LOAD_Y = 2;
  auto load_tile = [&](int tile, int which) __attribute__((always_inline)) {
    const int t0 = tile * TM, back = t0 > 0 ? 4 : 0;
    const unsigned nrow = T - t0 < TM ? T - t0 : TM;
    // 16 rows of the wave's 64 bytes per instruction (lane -> row lane / 4, piece lane & 3)
    const int l = lane_again(), lrow = l >> 2, c0 = wv * 32 + (l & 3) * 8;
    const bool pc_ok = c0 < bs;
    const unsigned ld_vo = pc_ok ? (unsigned)lrow * row2 + (unsigned)(g * bs + c0) * 2 : OOB;
    // staged row s of u (and of y with the merge) is step t0 - 4 + s
    const unsigned lead = back ? ld_vo : lrow >= 4 && pc_ok ? ld_vo - 4 * row2 : OOB;
    auto rows4 = [&](const void *src, unsigned dst) __attribute__((always_inline)) {
      const u32x4 rs = buf_words((const unsigned short *)src + (seq + t0 - back) * D, (size_t)(nrow + back) * row2);
      lds16<true>(rs, dst, lead, 0);
#pragma unroll
      for (int m = 1; m < NU; ++m)
        if (!TIGHT || m < NU - 1) lds16<true>(rs, dst + m * 1024, m == NU - 1 && l >= 16 ? OOB : ld_vo, (unsigned)(16 * m - 4 + back) * row2);
        else if (l < 16) lds16<true>(rs, dst + m * 1024, ld_vo, (unsigned)(16 * m - 4 + back) * row2);
    };
    auto rows = [&](const void *src, unsigned dst) __attribute__((always_inline)) {
      const u32x4 rs = buf_words((const unsigned short *)src + (seq + t0) * D, (size_t)nrow * row2);
#pragma unroll
      for (int m = 0; m < TM / 16; ++m) lds16<true>(rs, dst + m * 1024, ld_vo, (unsigned)(16 * m) * row2);
    };
    const unsigned at = lds_offset(smem) + (unsigned)wv * L::REGION;
    if (which & LOAD_U) rows4(p.u, at + L::U);
    if (!(which & LOAD_Y)) return;
    if constexpr (MERGE) {
      rows4(p.y_in, at + L::Y);
      rows(p.branch, at + L::B);
    } else {   // staged row s of y is step t0 - 1 + s
      const int yb = t0 > 0 ? 1 : 0;
      const u32x4 rs = buf_words((const unsigned short *)p.y_in + (seq + t0 - yb) * D, (size_t)(nrow + yb) * row2);
      lds16<true>(rs, at + L::Y, yb ? ld_vo : lrow >= 1 && pc_ok ? ld_vo - row2 : OOB, 0);
#pragma unroll
      for (int m = 1; m < NY; ++m) lds16<true>(rs, at + L::Y + m * 1024, ld_vo, (unsigned)(16 * m - 1 + yb) * row2);
    }
    rows(p.dy, at + L::DY);
  };
  auto rows_of = [&](const unsigned char *t, int rb, int n0, int cnt, unsigned *v) __attribute__((always_inline)) {
#pragma unroll
    for (int n = 0; n < cnt; ++n) {
      const u32x2 q = lds_tr(t + r_rd + (unsigned)(rb * 32 + 4 * (n0 + n)) * 64);
      v[2 * n] = q[0];
      v[2 * n + 1] = q[1];
    }
  };
  auto put16 = [&](unsigned char *t, int rb, const unsigned (&v)[8]) __attribute__((always_inline)) {   // a lane's 16 steps
#pragma unroll
    for (int s = 0; s < 2; ++s)
      *(u32x4 *)(t + t_wr[s] + rb * 2048) = u32x4{v[4 * s], v[4 * s + 1], v[4 * s + 2], v[4 * s + 3]};
  };
  auto frag = [&](const unsigned char *t, int rb) __attribute__((always_inline)) {
    const u32x2 lo = lds_tr(t + f_rd[0] + rb * 2048), hi = lds_tr(t + f_rd[1] + rb * 2048);
    return __builtin_bit_cast(f16x8, (u32x4){lo[0], lo[1], hi[0], hi[1]});
  };
  // a lane's 16 steps, for the weight gradients (rglru_wgrad.h); `per` bytes of all blocks per 32 steps
  auto run_out = [&](const unsigned (&v)[8], int rb, const unsigned short *out, size_t per) __attribute__((always_inline)) {
    const __amdgpu_buffer_rsrc_t rs = buf((const char *)out + rb * per, (size_t)bs * 64);   // (channels past the block: past its range)
    const int l = lane_again();
    const unsigned vo = (unsigned)wv * 2048 + (unsigned)((l >> 4) & 1) * 1024 + (unsigned)(l >> 5) * 512 + (unsigned)(l & 15) * 16;
    store16<RGLRU_NT>(u32x4{v[0], v[1], v[2], v[3]}, rs, vo, 0);
    store16<RGLRU_NT>(u32x4{v[4], v[5], v[6], v[7]}, rs, vo + 256, 0);
  };
  // [channel][step] tiles as rows of a [B][T][D] tensor
  auto rows_out = [&](const unsigned char *t, void *out, int t0, unsigned nrow) __attribute__((always_inline)) {
    const __amdgpu_buffer_rsrc_t rs = buf((unsigned short *)out + (seq + t0) * D, (size_t)nrow * row2);
    // lane -> row 16 m + 4 (lane / 16) + (lane & 3), channels 8 ((lane & 15) / 4) .. + 7 in two reads
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

  float s_ba = 0.f, s_bx = 0.f, s_lam = 0.f, s_tap[4] = {0.f, 0.f, 0.f, 0.f}, s_cb = 0.f;
  float carry = ok && p.dhT ? S * p.dhT[(size_t)b * D + d] : 0.f;   // S eps entering this workgroup's next tile
  float nx[3] = {0.f, 0.f, 0.f};                     // first three rows of dx of the tile behind (unsliced)
  int spins = G > 1 && expired_before(a.err) ? SPIN_LIMIT : 0;

  int tile = a.ntile - 1 - w;
  if (tile >= 0) load_tile(tile, LOAD_U | LOAD_Y);
  for (; tile >= 0; tile -= G) {
    const int t0 = tile * TM;
    const unsigned nrow = T - t0 < TM ? T - t0 : TM;
    // (the tile's loads have landed; only the stores of du behind them may still be under way)
    if (tile == a.ntile - 1 - w) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    else asm volatile("s_waitcnt vmcnt(%0)" :: "n"(TM / 16) : "memory");
#pragma unroll
    for (int ks = 0; ks < PD; ++ks) load_w(wg_rs, ks);
    if (t0 == 0 && p.state_in) {   // steps -3 .. -1 from the carried ring
      const int l = lane_again();
      if (l >= 4 && l < 16 && wv * 32 + (l & 3) * 8 < bs)
        *(u32x4 *)(my + L::U + l * 16) = *(const u32x4_at2 *)((const unsigned short *)p.state_in +
            ((size_t)b * 3 + ring_slot(p.pos0 + (l >> 2) - 4)) * D + g * bs + wv * 32 + (l & 3) * 8);
      wave_lds_fence();
    }
    // document boundaries (scalar words): bit i of [0]: step 32 rb + i starts a document, of [k]: lag k stays inside
    unsigned st16[MT];
    unsigned mk[MT][4];
    if constexpr (PACKED) {
#pragma unroll
      for (int rb = 0; rb < MT; ++rb) {
        const int wd = tile * MT + rb;
        const uint4 v = wd < a.nmask ? a.rmask[(size_t)b * a.nmask + wd] : make_uint4(0u, 0u, 0u, 0u);
        mk[rb][0] = v.x; mk[rb][1] = v.y; mk[rb][2] = v.z; mk[rb][3] = v.w;
        st16[rb] = hf ? v.x >> 16 : v.x;
      }
    }
    // ---- Conv1D: x of a lane's run, from u of its steps -4 .. 15
    auto u_rows = [&](int rb, unsigned (&uu)[10]) __attribute__((always_inline)) { rows_of(my + L::U, rb, 0, 5, uu); };
    auto u_at = [](const unsigned (&uu)[10], int i) __attribute__((always_inline)) {
      const unsigned v = uu[(i + 4) >> 1];
      return (i & 1) ? bf_hi(v) : bf_lo(v);
    };
    auto conv = [&](const unsigned (&uu)[10], const f32x4 &tap, float cbias, int rb, int r) __attribute__((always_inline)) {
      float v = cbias;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        float ui = u_at(uu, r - k);
        if (PACKED && k > 0) ui = ((hf ? mk[rb][k] >> 16 : mk[rb][k]) >> r) & 1u ? ui : 0.f;
        v = fmaf(tap[k], ui, v);
      }
      return v;
    };
    float xk[KEEP ? MT : 1][16];
    const bool ragged = (int)nrow < TM;
    auto left = [&]() __attribute__((always_inline)) { return (int)nrow - (lane_again() >> 5) * 16; };   // of this lane's steps (of row block 0)
    // pairs of 16-bit values of a lane's steps: nothing of those past the end
    auto cut = [&](unsigned (&v)[8], int rb) __attribute__((always_inline)) {
      const int valid = left() - rb * 32;
#pragma unroll
      for (int e = 0; e < 8; ++e) v[e] = valid - 2 * e > 1 ? v[e] : valid - 2 * e == 1 ? v[e] & 0xffffu : 0u;
    };
#pragma unroll
    for (int rb = 0; rb < MT; ++rb) {
      unsigned uu[10], pk[8];
      u_rows(rb, uu);
      const f32x4 tap = *(const f32x4 *)(my + L::C + j * 48 + 16);
      const float cbias = *(const float *)(my + L::C + j * 48 + 12);
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        float v[8];
        unsigned o[4];
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = conv(uu, tap, cbias, rb, 8 * h + e);
        if constexpr (KEEP)
#pragma unroll
          for (int e = 0; e < 8; ++e) xk[rb][8 * h + e] = v[e];
        cvt_f16x8(v, o);
#pragma unroll
        for (int e = 0; e < 4; ++e) pk[4 * h + e] = o[e];
        __builtin_amdgcn_sched_barrier(0);
      }
      if (ragged) {
        cut(pk, rb);
        if constexpr (KEEP) {
          const int valid = left();
#pragma unroll
          for (int r = 0; r < 16; ++r)
            if (r + rb * 32 >= valid) xk[rb][r] = 0.f;
        }
      }
      put16(my + L::X, rb, pk);
      run_out(pk, rb, a.xT + (((size_t)b * a.ntile + tile) * MT * D + g * bs) * 32, (size_t)D * 64);
    }
    // ---- the upstream gradient (with the merge: dy = dout GeLU(branch) in fp32, dbranch = dout y GeLU'(branch))
    float dym[MERGE ? MT : 1][16];
    auto dy_at = [&](const unsigned (&dyv)[8], int rb, int r) __attribute__((always_inline)) {
      if constexpr (MERGE) return dym[rb][r];
      else return (r & 1) ? bf_hi(dyv[r >> 1]) : bf_lo(dyv[r >> 1]);
    };
    if constexpr (MERGE) {
      unsigned bo[MT][8];
#pragma unroll
      for (int rb = 0; rb < MT; ++rb) {
        unsigned dv[8], bv[8], yv[10];
        rows_of(my + L::DY, rb, 0, 4, dv);
        rows_of(my + L::B, rb, 0, 4, bv);
        rows_of(my + L::Y, rb, 0, 5, yv);
#pragma unroll
        for (int q = 0; q < 8; ++q) {
          float db[2];
#pragma unroll
          for (int e = 0; e < 2; ++e) {
            float val, grad;
            gelu_and_grad<VAR == V_MERGE_TANH, true>(e ? bf_hi(bv[q]) : bf_lo(bv[q]), val, grad);
            const float go = e ? bf_hi(dv[q]) : bf_lo(dv[q]);
            db[e] = go * (e ? bf_hi(yv[q + 2]) : bf_lo(yv[q + 2])) * grad;
            dym[rb][2 * q + e] = go * val;
          }
          bo[rb][q] = pack_bf16(db[0], db[1]);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
      wave_lds_fence();
#pragma unroll
      for (int rb = 0; rb < MT; ++rb) put16(my + L::B, rb, bo[rb]);
    }
    lds_barrier();   // x is there
    if constexpr (MERGE) rows_out(my + L::B, p.dbranch, t0, nrow);

    // ---- gate pre-activations
    f32x16 accp[MT], accq[MT];
    const f32x4 con = *(const f32x4 *)(my + L::C + j * 48);
    // (kd: within what the 2^-126 of a gate held closed still takes to nothing)
    const float bp = con[0], bq = con[1], kdn = con[2], kd = kdn * LOG2E < -1e30f ? -1e30f : kdn * LOG2E;
#pragma unroll
    for (int rb = 0; rb < MT; ++rb)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        accp[rb][r] = bp;
        accq[rb][r] = bq;
      }
    // Steps past the end: a closed gate, a_t = 1 and m_t = 0, lets eps pass; with x and h_{t-1} taken as zero there they add
    // nothing, whatever the sequence's last inputs (which the Conv1D reaches back to) and its last state are
    if (ragged) {
      const int valid = left();
#pragma unroll
      for (int rb = 0; rb < MT; ++rb)
#pragma unroll
        for (int r = 0; r < 16; ++r)
          if (r + rb * 32 >= valid) accp[rb][r] = -__builtin_huge_valf();
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
        if (ks + PD < NKS) load_w(wg_rs, ks + PD);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    // ---- r_t, a_t and the aggregate of the tile, latest step first
    float ak[KEEPA ? MT : 1][16];
    float ep[MT][16];   // e^-p: r = 1 / (1 + e^-p), 1 - r = e^-p r
    float A_up[MT], E_up[MT], A_rb[MT], E_rb[MT];
#pragma unroll
    for (int rb = MT - 1; rb >= 0; --rb) {
      if constexpr (PACKED) asm volatile("" : "+v"(st16[rb]));
      float A = 1.f, E = 0.f;
      unsigned dyv[8];
      if constexpr (!MERGE) rows_of(my + L::DY, rb, 0, 4, dyv);
#pragma unroll
      for (int r = 15; r >= 0; --r) {
        // (1 - r as a product: no cancellation when saturated)
        ep[rb][r] = gate_exp(accp[rb][r]);
        float av = __builtin_amdgcn_exp2f(kd * __builtin_amdgcn_rcpf(1.f + ep[rb][r]));
        if constexpr (KEEPA) ak[rb][r] = av;
        if (PACKED && ((st16[rb] >> r) & 1u)) av = 0.f;   // nothing flows out of a document's first step
        E = av * fmaf(S, dy_at(dyv, rb, r), E);
        A *= av;
        if (r % 4 == 0) __builtin_amdgcn_sched_barrier(0);
      }
      float A_lo, E_lo;
      both_halves(A, A_lo, A_up[rb]);
      both_halves(E, E_lo, E_up[rb]);
      A_rb[rb] = A_lo * A_up[rb];
      E_rb[rb] = fmaf(A_lo, E_up[rb], E_lo);
    }
    float A_t = A_rb[MT - 1], E_t = E_rb[MT - 1];
    if (MT == 2) {
      E_t = fmaf(A_rb[0], E_t, E_rb[0]);
      A_t *= A_rb[0];
    }
    float e_in = carry;
    if (G > 1) {
      int c_ = wv * 32 + j;
      asm volatile("" : "+v"(c_));
      u64 *ring = a.rec + (size_t)gb * a.R * (NCT * 32) + c_;
      if (hf == 0) publish(ring + slot_of(tile, a.R) * (NCT * 32), A_t, E_t, epoch_of(tile, a.R));
      // the state behind tile + G, carried across tiles tile + G - 1 .. tile + 1: each lane half fetches and composes
      // half of the records, four per round trip
      const RecWalk<-1> wk(tile + G - 1, G - 1, hf, a.R);
      const int nrec = G >> 1;
      float rA = 1.f, rE = 0.f;
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
          const float A = has ? rec_A(rec[i]) : 1.f, E = has ? rec_H(rec[i]) : 0.f;
          rE = fmaf(A, rE, E);
          rA *= A;
        }
      }
      const float xA = __shfl_xor(rA, 32), xE = __shfl_xor(rE, 32);
      e_in = fmaf(hf ? xA : rA, e_in, hf ? xE : rE);
      e_in = fmaf(hf ? rA : xA, e_in, hf ? rE : xE);
      // a wait that expired: this channel's results are NaN from here on, visibly invalid
      if (spins >= SPIN_LIMIT || __shfl_xor(spins, 32) >= SPIN_LIMIT) e_in = __builtin_nanf("");
    }
    carry = fmaf(A_t, e_in, E_t);

    // ---- the adjoints, latest step first
    unsigned ul[MT][10];
#pragma unroll
    for (int rb = 0; rb < MT; ++rb) u_rows(rb, ul[rb]);
    lds_barrier();   // (every wave has read x)
    f32x16 dx[MT];
    float e_blk = e_in;
    const f32x4 tap2 = *(const f32x4 *)(my + L::C + j * 48 + 16);
    const float cbias2 = *(const float *)(my + L::C + j * 48 + 12);
    const float h_first = *(const float *)(my + L::C + j * 48 + 32);
#pragma unroll
    for (int rb = MT - 1; rb >= 0; --rb) {
      if constexpr (PACKED) asm volatile("" : "+v"(st16[rb]));   // (tested bit by bit, not expanded for all steps at once)
      float e = hf ? e_blk : fmaf(A_up[rb], e_blk, E_up[rb]);   // eps_{t+1} for the last step of this run
      e_blk = fmaf(A_rb[rb], e_blk, E_rb[rb]);
      unsigned yv[8], dyv[8], pk[8], qk[8];   // h_{t-1}, dy
      if constexpr (MERGE) {
        unsigned v[10];
        rows_of(my + L::Y, rb, 0, 5, v);
#pragma unroll
        for (int q = 0; q < 8; ++q) yv[q] = __builtin_amdgcn_alignbit(v[q + 2], v[q + 1], 16);
      } else {
        rows_of(my + L::Y, rb, 0, 4, yv);
        rows_of(my + L::DY, rb, 0, 4, dyv);
      }
      if (ragged) cut(yv, rb);
      int valid = 0;
      if constexpr (!KEEP) valid = left();
      if (rb == 0) {   // the next tile's y and dy (and branch): in front of a stretch that needs nothing from memory
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        if (tile - G >= 0) load_tile(tile - G, LOAD_Y);
      }
      float dpq[8];   // dp of four steps, dq
#pragma unroll
      for (int r = 0; r < 16; ++r) asm volatile("" : "+v"(ep[rb][r]));   // (r and a are formed again rather than kept)
#pragma unroll
      for (int r = 15; r >= 0; --r) {
        float xv;
        if constexpr (KEEP) xv = xk[rb][r];
        else xv = r + rb * 32 < valid ? conv(ul[rb], tap2, cbias2, rb, r) : 0.f;
        const float rv = __builtin_amdgcn_rcpf(1.f + ep[rb][r]), l2 = kd * rv;
        float av;
        if constexpr (KEEPA) av = ak[rb][r];
        else av = __builtin_amdgcn_exp2f(l2);
        const float eq = gate_exp(accq[rb][r]), ig = __builtin_amdgcn_rcpf(1.f + eq);
        // (a gate closed so far that r_t = 0 gives m = 0: the floor keeps 1/m finite, and the terms
        // it scales carry the factor r_t (1 - r_t))
        const float m2 = fmaxf(one_minus_sq(av, l2), 1e-30f), rs = __builtin_amdgcn_rsqf(m2);
        const float delta = fmaf(S, dy_at(dyv, rb, r), e), gin = ig * xv;
        const bool fresh = PACKED && ((st16[rb] >> r) & 1u);   // a document's first step: h_{t-1} = 0
        float hp = (r & 1) ? bf_hi(yv[r >> 1]) : bf_lo(yv[r >> 1]);
        if (rb == 0 && r == 0) hp = tile == 0 && hf == 0 ? h_first : hp;
        if (fresh) hp = 0.f;
        const float t = delta * av;
        const float dla = t * fmaf(-av * gin, rs, hp);   // delta a (h_{t-1} - a g / m)
        const float dxd = delta * (m2 * rs) * ig, dlr = dla * rv;
        const float dqv = dxd * xv * (eq * ig), dpv = kdn * dlr * (ep[rb][r] * rv);
        dx[rb][r] = dxd;
        s_ba += dpv;
        s_bx += dqv;
        s_lam += dlr;
        e = fresh ? 0.f : t;
        dpq[r & 3] = dpv;
        dpq[4 + (r & 3)] = dqv;
        if ((r & 3) == 0) {
          unsigned o[4];
          cvt_f16x8(dpq, o);
          pk[r >> 1] = o[0];
          pk[(r >> 1) + 1] = o[1];
          qk[r >> 1] = o[2];
          qk[(r >> 1) + 1] = o[3];
          asm volatile("" : "+v"(s_ba), "+v"(s_bx), "+v"(s_lam));   // (summed here; the compiler would keep the terms for later)
          __builtin_amdgcn_sched_barrier(0);
        }
      }
      put16(my + L::P, rb, pk);
      put16(my + L::Q, rb, qk);
      const unsigned short *o = a.pqT + (((size_t)b * a.ntile + tile) * MT * D + g * bs) * 64;
      run_out(pk, rb, o, (size_t)D * 128);
      run_out(qk, rb, o + (size_t)bs * 32, (size_t)D * 128);
    }
#pragma unroll
    for (int ks = 0; ks < PD; ++ks) load_w(wd_rs, ks);
    lds_barrier();   // dp, dq are there
    // ---- dx: the products with the transposed weights on top of the direct part
    {
      f16x8 fa[2][2][MT];
      auto fetch = [&](int ks) __attribute__((always_inline)) {
#pragma unroll
        for (int gt = 0; gt < 2; ++gt)
#pragma unroll
          for (int rb = 0; rb < MT; ++rb)
            fa[ks & 1][gt][rb] = frag(smem + (gt ? L::Q : L::P) + (ks >> 1) * L::REGION + (ks & 1) * 1024, rb);
      };
      fetch(0);
#pragma unroll
      for (int ks = 0; ks < NKS; ++ks) {
        if (ks + 1 < NKS) fetch(ks + 1);
#pragma unroll
        for (int gt = 0; gt < 2; ++gt)
#pragma unroll
          for (int rb = 0; rb < MT; ++rb)
            dx[rb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(fa[ks & 1][gt][rb], wq[ks % PD][gt], dx[rb], 0, 0, 0);
        if (ks + PD < NKS) load_w(wd_rs, ks + PD);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    lds_barrier();   // (every wave has read dp and dq)

    // ---- the Conv1D's adjoint; dx carries the factor S
    float lo[MT][3], up[MT][3];
#pragma unroll
    for (int rb = 0; rb < MT; ++rb)
#pragma unroll
      for (int r = 0; r < 3; ++r) both_halves(dx[rb][r], lo[rb][r], up[rb][r]);
    if (a.edge && ok) {
      int d_ = g * bs + wv * 32 + j;
      asm volatile("" : "+v"(d_));
      float *e = a.edge + (((size_t)b * a.ntile + tile) * 6 + hf * 3) * D + d_;
#pragma unroll
      for (int r = 0; r < 3; ++r) e[(size_t)r * D] = hf ? dx[MT - 1][13 + r] : dx[0][r];
    }
    // the next tile's u: behind the last weights, in front of work that needs nothing from memory
    f32x4 tap = *(const f32x4 *)(my + L::C + j * 48 + 16);
#pragma unroll
    for (int k = 0; k < 4; ++k) tap[k] *= invS;
    if (tile - G >= 0) load_tile(tile - G, LOAD_U);
#pragma unroll
    for (int rb = 0; rb < MT; ++rb)   // (u is kept as it came, not as the fp32 values the adjoints made of it)
#pragma unroll
      for (int q = 0; q < 10; ++q) asm volatile("" : "+v"(ul[rb][q]));
#pragma unroll
    for (int rb = 0; rb < MT; ++rb) {
      float xx[19];
#pragma unroll
      for (int r = 0; r < 16; ++r) xx[r] = dx[rb][r];
#pragma unroll
      for (int r = 0; r < 3; ++r) xx[16 + r] = hf ? (rb + 1 < MT ? lo[MT - 1][r] : nx[r]) : up[rb][r];
      unsigned lag[4] = {0u, 0u, 0u, 0u};   // lag masks of the 19 steps from this lane's first
      if constexpr (PACKED) {
#pragma unroll
        for (int k = 1; k < 4; ++k) {
          const int wd = tile * MT + rb + 1;
          unsigned nxt;
          if (rb + 1 < MT) nxt = mk[MT - 1][k];
          else {
            const uint4 v = wd < a.nmask ? a.rmask[(size_t)b * a.nmask + wd] : make_uint4(0u, 0u, 0u, 0u);
            nxt = k == 1 ? v.y : k == 2 ? v.z : v.w;
          }
          lag[k] = hf ? (mk[rb][k] >> 16) | (nxt << 16) : mk[rb][k];
        }
      }
      unsigned pk[8];
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        float o[2];
#pragma unroll
        for (int e = 0; e < 2; ++e) {
          const int r = 2 * q + e;
          float v = tap[0] * xx[r];
#pragma unroll
          for (int k = 1; k < 4; ++k) v = fmaf(tap[k], !PACKED || ((lag[k] >> (r + k)) & 1u) ? xx[r + k] : 0.f, v);
          o[e] = v;
        }
        pk[q] = pack_bf16(o[0], o[1]);
      }
      put16(my + L::X, rb, pk);
#pragma unroll
      for (int r = 0; r < 16; ++r) {
#pragma unroll
        for (int k = 0; k < 4; ++k)
          s_tap[k] = fmaf(!PACKED || k == 0 || ((lag[k] >> r) & 1u) ? xx[r] : 0.f, u_at(ul[rb], r - k), s_tap[k]);
        s_cb += xx[r];
        if (r % 4 == 3) __builtin_amdgcn_sched_barrier(0);
      }
    }
    if (G == 1)
#pragma unroll
      for (int r = 0; r < 3; ++r) nx[r] = lo[0][r];
    wave_lds_fence();
    rows_out(my + L::X, p.du, t0, nrow);
    wave_lds_fence();
  }
  if (spins >= SPIN_LIMIT) mark_expired(a.err);

  // ---- per-channel sums of this workgroup (both lane halves hold the same channel)
  float sum[8] = {s_ba * invS, s_bx * invS, s_lam * invS, s_tap[0] * invS, s_tap[1] * invS, s_tap[2] * invS, s_tap[3] * invS, s_cb * invS};
#pragma unroll
  for (int k = 0; k < 8; ++k) sum[k] += __shfl_xor(sum[k], 32);
  if (hf == 0 && ok) {
    int d = g * bs + wv * 32 + j;
    asm volatile("" : "+v"(d));
    float *pa = a.partA + (size_t)(b * G + w) * 3 * D + d, *pc = a.partC + (size_t)(b * G + w) * 5 * D + d;
    pa[0] = sum[0];
    pa[D] = sum[1];
    pa[2 * (size_t)D] = sum[2] * (p.c / (1.f + expf(p.Lambda[d])));   // c sigmoid(-Lambda)
#pragma unroll
    for (int k = 0; k < 5; ++k) pc[(size_t)k * D] = sum[3 + k];
    // the workgroup that ran tile 0 holds eps_0 = dL/dh0
    if (p.dh0 && (a.ntile - 1 - w) % G == 0) p.dh0[(size_t)b * D + d] = carry * invS;
  }
}

// ---- host side: what the dispatch knows of an instance
struct Instance {
  const void *kernel;
  int waves, mt, lds, per_cu;   // per_cu: workgroups that run at once on a compute unit
};
template <int NCT, int MT, int VAR, int WPE, int PD, int K>
Instance instance() {
  constexpr int lds = NCT * Lds<MT, VAR, NCT == 16>::REGION, by_lds = 160 * 1024 / lds, by_waves = 4 * WPE / NCT;
  if constexpr (lds <= 160 * 1024) return {(const void *)bwd_tile_kernel<NCT, MT, VAR, WPE, PD, K>, NCT, MT, lds, by_lds < by_waves ? by_lds : by_waves};
  else return {nullptr, 0, 0, 0, 0};   // (the widest blocks with the merge)
}
template <int NCT, int MT, int WPE, int PD, int K>
Instance pick_merge(int var) {
  return var == V_MERGE ? instance<NCT, MT, V_MERGE, WPE, PD, K>() : instance<NCT, MT, V_MERGE_TANH, WPE, PD, K>();
}
template <int NCT, int MT, int WPE, int PD, int K>
Instance pick(int var) {
  if (var == V_PLAIN) return instance<NCT, MT, V_PLAIN, WPE, PD, K>();
  if constexpr (NCT == 8) {   // (packed rows: 256 channels only)
    if (var == V_PACKED) return instance<NCT, MT, V_PACKED, WPE, PD, K>();
  } else {
    if (var == V_PACKED) return {nullptr, 0, 0, 0, 0};
  }
  if constexpr (MT == 1) return pick_merge<NCT, MT, WPE, PD, K>(var);
  else return {nullptr, 0, 0, 0, 0};
}
// by the number of 32-channel tiles of a block; kernel null: none for that size. var: V_PLAIN ...
Instance find_instance_a(int nct, int var);   // 4 - 6
Instance find_instance_b(int nct, int var);   // 7, 8
Instance find_instance_c(int nct, int var);   // 9 - 12
Instance find_instance_d(int nct, int var);   // 13 - 16

}  // namespace fused
}  // namespace rglru
