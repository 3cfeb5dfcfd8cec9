// Decode step (Section 5; states of Appendix F) for few sequences, bf16 storage, gate blocks of 128 to
// 512 channels: one workgroup per (gate block, sequence), the gate products on the vector unit.
//
// With one to a few dozen sequences the step is a chain of latencies around 256 KB of weights per
// block. The kernel for full tiles of 32 sequences turns the weights into matrix-core fragments
// through LDS, four phases of which two are in flight; here a wave asks for all of its 32 output
// channels' rows at once (32 loads of 16 bytes per lane: half a wave reads a row of W_a, the other
// half the same row of W_x), multiplies them as they arrive against eight inputs per lane
// (v_dot2_f32_bf16, x as bf16 high + low part: 16 significant bits where the fragments carry 8), and
// sums over the 32 lanes by a butterfly that leaves lane l with output l. A block's Conv1D ring has
// one reader, which also replaces the oldest slot - unless the block is wider than the 256 outputs a
// workgroup has (8 waves of 32): then several workgroups share it and the ring is written by a
// kernel of its own. With the merge at B1 D2560 in 10 blocks a call takes 6.2 us against 8.9 on the kernel
// for tiles (a launch of nothing takes 3.9), at B1 D5632 in 16 blocks 7.5 against 10.9.
#include "rglru_gelu.h"
#include "rglru_mfma.h"

namespace rglru {
using namespace mfma;

namespace {

typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

struct SmallArgs {
  Problem p;   // u = u_t [B][D], hT = h [B][D] (in place), state_out = ring (in place), y = y_t
  int nout;    // output channels per workgroup (32 per wave)
  int nob;     // workgroups per block
};

// One halving step of the transposed sum below: a lane keeps the values of the half its bit S names and
// takes the partner's share of them (the partner, by a DPP permutation, is a lane with the other bit S)
template <int S, int DPP>
__device__ __forceinline__ void half_sum(float (&v)[32], int lane) {
  const bool up = lane & S;
#pragma unroll
  for (int i = 0; i < S; ++i) {
    const float keep = up ? v[i + S] : v[i], give = up ? v[i] : v[i + S];
    v[i] = keep + __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, give), DPP, 0xf, 0xf, true));
  }
}
// sums of 32 values over 32 lanes: lane l of each half ends with the sum of v[l]
__device__ __forceinline__ float sum_transposed(float (&v)[32], int lane) {
#pragma unroll
  for (int i = 0; i < 16; ++i) {   // odd rows of 16 lanes of v[i] change places with even rows of v[i + 16]
    const auto t = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(unsigned, v[i]),
                                                    __builtin_bit_cast(unsigned, v[i + 16]), false, false);
    const unsigned t0 = t[0], t1 = t[1];
    v[i] = __builtin_bit_cast(float, t0) + __builtin_bit_cast(float, t1);
  }
  half_sum<8, 0x128>(v, lane);   // row_ror:8
  half_sum<4, 0x141>(v, lane);   // row_half_mirror
  half_sum<2, 0x4e>(v, lane);    // quad_perm:[2,3,0,1]
  half_sum<1, 0xb1>(v, lane);    // quad_perm:[1,0,3,2]
  return v[0];
}

// LPR: lanes that share a weight row (32: blocks up to 256 channels, 64: up to 512)
// MERGE: 1 / 2 = the block's merge as epilogue. RING: the workgroup replaces the ring slot itself.
template <int LPR, int MERGE, bool RING>
__global__ void __launch_bounds__(512) decode_small_kernel(SmallArgs a) {
  constexpr int MAXC = LPR * 8;                    // channels of a block, padded
  __shared__ __attribute__((aligned(16))) unsigned xh[MAXC / 2], xl[MAXC / 2];   // bf16 pairs: high, low part of x
  __shared__ float xf[MAXC];
  const Problem &p = a.p;
  const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int g = blockIdx.x / a.nob, ob = blockIdx.x - g * a.nob, b = blockIdx.y;
  const int D = p.D, bs = p.bs, c0 = ob * a.nout + wv * 32;   // this wave's first output channel
  const long long pos = p.pos_rows ? p.pos_rows[b] : p.pos0;
  // ---- Conv1D inputs: a channel pair per thread (bs is even)
  const int c2 = 2 * tid < bs ? 2 * tid : bs - 2, dc = g * bs + c2;
  const int s1 = ring_slot(pos - 1), s2 = ring_slot(pos - 2), s3 = ring_slot(pos - 3);
  unsigned short *ring = (unsigned short *)p.state_out + (size_t)b * 3 * D + dc;
  const unsigned u0 = *(const unsigned *)((const unsigned short *)p.u + (size_t)b * D + dc);
  const unsigned u1 = *(const unsigned *)(ring + (size_t)s1 * D), u2 = *(const unsigned *)(ring + (size_t)s2 * D),
                 u3 = *(const unsigned *)(ring + (size_t)s3 * D);
  float2 w[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) w[k] = *(const float2 *)(p.conv_w + (size_t)k * D + dc);
  const float2 cb = p.conv_b ? *(const float2 *)(p.conv_b + dc) : make_float2(0.f, 0.f);
  // ---- this lane's output channel
  const int ch = c0 + (lane & 31), d = g * bs + (ch < bs ? ch : bs - 1);
  const bool mine = ch < bs && c0 < ob * a.nout + a.nout;
  const float h0 = p.hT[(size_t)b * D + d];
  const float ba = p.b_a[d], bx = p.b_x[d], lam = p.Lambda[d];
  float br = 0.f;
  if (MERGE) br = bf_lo((unsigned)((const unsigned short *)p.branch)[(size_t)b * D + d]);
  // ---- weights: row i of both gates (channel c0 + i; rows past the block are read from its last)
  const int piece = lane & (LPR - 1), pc = piece * 8 < bs ? piece : 0;   // this lane's eight input channels
  const unsigned short *wa = (const unsigned short *)p.W_a + (size_t)g * bs * bs + pc * 8;
  const unsigned short *wx = (const unsigned short *)p.W_x + (size_t)g * bs * bs + pc * 8;
  const unsigned short *wrow = LPR == 32 && lane >= 32 ? wx : wa;
  u32x4 wq[32];
#pragma unroll
  for (int i = 0; i < 32; ++i) wq[i] = *(const u32x4 *)(wrow + (size_t)(c0 + i < bs ? c0 + i : bs - 1) * bs);
  __builtin_amdgcn_sched_barrier(0);
  {
    float x0 = cb.x, x1 = cb.y;
    x0 = fmaf(w[0].x, bf_lo(u0), x0); x1 = fmaf(w[0].y, bf_hi(u0), x1);
    x0 = fmaf(w[1].x, bf_lo(u1), x0); x1 = fmaf(w[1].y, bf_hi(u1), x1);
    x0 = fmaf(w[2].x, bf_lo(u2), x0); x1 = fmaf(w[2].y, bf_hi(u2), x1);
    x0 = fmaf(w[3].x, bf_lo(u3), x0); x1 = fmaf(w[3].y, bf_hi(u3), x1);
    if (2 * tid < MAXC) {
      const bool in = 2 * tid < bs;
      unsigned hi = 0u, lo = 0u;
      if (in) split_bf16(x0, x1, hi, lo);
      xh[tid] = hi;
      xl[tid] = lo;
      *(float2 *)(xf + 2 * tid) = make_float2(in ? x0 : 0.f, in ? x1 : 0.f);
      // slot pos mod 3 == slot (pos - 3) mod 3
      if (RING && in) *(unsigned *)(ring + (size_t)s3 * D) = u0;
    }
  }
  const float gl = MERGE ? gelu<MERGE == 2, true>(br) : 0.f;
  float kd;
  {
    const float z = -lam, sp = z > 0.f ? z + log1pf(expf(-z)) : log1pf(expf(z));
    kd = -p.c * sp * LOG2E;
  }
  __syncthreads();
  if (c0 >= bs) return;   // (a wave past the block)
  typedef __bf16 bf16x2v __attribute__((ext_vector_type(2)));
  const u32x4 vh = *(const u32x4 *)(xh + piece * 4), vl = *(const u32x4 *)(xl + piece * 4);
  auto dots = [&](float (&acc)[32]) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < 32; ++i) {
      float s = 0.f;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const unsigned q = wq[i][e], xhe = vh[e], xle = vl[e];   // (bit_cast of a vector element takes the first)
        s = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2v, q), __builtin_bit_cast(bf16x2v, xhe), s, false);
        s = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2v, q), __builtin_bit_cast(bf16x2v, xle), s, false);
      }
      acc[i] = s;
    }
  };
  float acc[32], pp, qq;
  dots(acc);
  if (LPR == 32) {
    const float r = sum_transposed(acc, lane), o = __shfl_xor(r, 32);
    pp = lane < 32 ? r : o;
    qq = lane < 32 ? o : r;
  } else {
#pragma unroll
    for (int i = 0; i < 32; ++i) wq[i] = *(const u32x4 *)(wx + (size_t)(c0 + i < bs ? c0 + i : bs - 1) * bs);
    float r = sum_transposed(acc, lane);
    pp = r + __shfl_xor(r, 32);
    dots(acc);
    r = sum_transposed(acc, lane);
    qq = r + __shfl_xor(r, 32);
  }
  // ---- eqs. (1)-(4)
  const float rg = __builtin_amdgcn_rcpf(1.f + __builtin_amdgcn_exp2f(-LOG2E * (pp + ba)));
  const float ig = __builtin_amdgcn_rcpf(1.f + __builtin_amdgcn_exp2f(-LOG2E * (qq + bx)));
  const float l2 = kd * rg, av = __builtin_amdgcn_exp2f(l2);
  const float hn = fmaf(av, h0, __builtin_amdgcn_sqrtf(one_minus_sq(av, l2)) * ig * xf[ch < MAXC ? ch : 0]);
  if (lane < 32 && mine) {
    p.hT[(size_t)b * D + d] = hn;
    const unsigned yb = pack_bf16(hn, 0.f) & 0xffffu;
    ((unsigned short *)p.y)[(size_t)b * D + d] =
        (unsigned short)(MERGE ? pack_bf16(bf_lo(yb) * gl, 0.f) & 0xffffu : yb);
  }
}

// the new token into its ring slot, after every reader of the ring (blocks shared by several workgroups)
__global__ void __launch_bounds__(256) ring_put_kernel(const uint4 *u, uint4 *ring, int B, int chunks, int slot,
                                                       const long long *pos_rows) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= B * chunks) return;
  const int b = i / chunks, c = i - b * chunks;
  if (pos_rows) slot = ring_slot(pos_rows[b]);
  ring[((size_t)b * 3 + slot) * chunks + c] = u[i];
}

template <int LPR, bool RING>
void launch_t(const SmallArgs &a, dim3 grid, int threads, hipStream_t s) {
  if (a.p.merge == 0) hipLaunchKernelGGL((decode_small_kernel<LPR, 0, RING>), grid, dim3(threads), 0, s, a);
  else if (a.p.merge == 1) hipLaunchKernelGGL((decode_small_kernel<LPR, 1, RING>), grid, dim3(threads), 0, s, a);
  else hipLaunchKernelGGL((decode_small_kernel<LPR, 2, RING>), grid, dim3(threads), 0, s, a);
}

}  // namespace

// A block of up to 256 channels takes one workgroup of 8 waves and about 160 registers per sequence, one
// per CU: up to 256 of them run at once (B16 D4096 in 16 blocks, 256 workgroups: 6.3 us against 8.1 on the
// kernel for tiles, with the merge 6.8 against 8.9), with more the second round costs more than it saves
// (B20, 320 workgroups: 10.2 against 8.1, with the merge 10.6 against 8.9).
// A wider block's four-wave workgroups go two to a CU: 10.3 us with 480 workgroups (B10, 352 channels)
// against 10.9 on the kernel for tiles, 11.0 with 512 (B8, 512 channels) against 11.3; 12.7 against 10.9 with 528
// (B11) and 13.7 against 11.2 with 576 (B9).
bool decode_small_supported(const Problem &p, bool bf) {
  const uintptr_t all = (uintptr_t)p.W_a | (uintptr_t)p.W_x | (uintptr_t)p.u | (uintptr_t)p.state_out |
                        (uintptr_t)p.hT | (uintptr_t)p.y | (uintptr_t)p.conv_w | (uintptr_t)p.conv_b |
                        (uintptr_t)(p.merge ? p.branch : nullptr);
  if (!bf || !p.conv_w || p.bs % 16 != 0 || p.bs < 128 || p.bs > 512 || all % 16 != 0) return false;
  const long long wgs = (long long)p.nb * p.B;
  return p.bs <= 256 ? wgs <= 256 : wgs * ((p.bs + 127) / 128) <= 512;
}

hipError_t launch_ring_put(const Problem &p, hipStream_t s) {
  const int chunks = p.D / 8;
  hipLaunchKernelGGL(ring_put_kernel, dim3((p.B * chunks + 255) / 256), dim3(256), 0, s, (const uint4 *)p.u,
                     (uint4 *)p.state_out, p.B, chunks, ring_slot(p.pos0), p.pos_rows);
  return hipGetLastError();
}

hipError_t launch_decode_small(const Problem &p, hipStream_t s) {
  SmallArgs a;
  a.p = p;
  if (p.bs <= 256) {
    a.nout = 256;
    a.nob = 1;
    KernelTimer kt("decode_small_kernel", s);
    launch_t<32, true>(a, dim3(p.nb, p.B), 64 * ((p.bs + 31) / 32), s);
    return hipGetLastError();
  }
  a.nout = 128;
  a.nob = (p.bs + 127) / 128;
  {
    KernelTimer kt("decode_small_kernel", s);
    launch_t<64, false>(a, dim3(p.nb * a.nob, p.B), 256, s);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return launch_ring_put(p, s);
}

}  // namespace rglru
