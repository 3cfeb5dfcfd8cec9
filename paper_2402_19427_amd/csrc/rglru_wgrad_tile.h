// The weight gradients' kernel (layouts: rglru_wgrad.h); its instances are spread over two files.
#pragma once
#include "rglru_wgrad.h"

#include <atomic>

namespace rglru {
namespace wgrad {
using namespace pass;

// 256 rows x 32 N columns per workgroup of four waves, one wave per SIMD: 128 x 16 N outputs each, or 64 x 32 N where N is odd. Where
// stages are many, all of a block's columns up to 256 are in one workgroup: rows are read once (in tiles of 256 x 128 twice: as much again
// as memory delivers beside the products), and a pair of fragments from LDS serves 2 N products instead of 8 for 6 of 128 columns,
// for which LDS was as busy as the matrix units. Where they are few, its start and end are what it takes, and half of the columns start and
// end faster (see cost).
// What goes round is a unit of two planes of 16 steps: both halves of a stage, or the two parts of one half. Rows and columns
// come to LDS by direct-to-LDS loads, P units ahead (a counted wait and one barrier per unit); the fragments of a plane
// arrive while the other's products run. Bound by memory where the chip is full: B 16 T 4096, 16 blocks of 256 channels 303 us, 1.6 GB
// (346 in tiles of 256 x 128); B 8 T 2048, 10 blocks of 256 66 (90), 16 of 160 72 (77), B 4 16 of 352 in two slices 105 (117; in five 99, but
// 6 us more in the final sums).
template <int PARTS, int N>
struct Wg {
  static constexpr int WC = N % 2 ? 1 : 2, WR = 4 / WC, M = 8 / WR, NW = N / WC;   // waves along columns, rows; 32-blocks of a wave
  static constexpr int LB = (2 * N + 3) / 4;                           // column loads of a wave and unit, a kilobyte each; 4 of rows
  static constexpr int A = 16 * 1024, UNIT = A + 4 * LB * 1024;
  static constexpr int FIT = 160 * 1024 / UNIT, P = FIT > 6 ? 5 : FIT - 1, LDS = (P + 1) * UNIT;
};
struct WgradArgs {
  TileWgrad w;
  int njt, nkt;
  unsigned total;
};
template <int PARTS, int N>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 1))) tile_wgrad_kernel(WgradArgs a) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  typedef Wg<PARTS, N> K;
  constexpr int P = K::P, M = K::M, NW = K::NW;
  const unsigned id = xcd_id();
  if (id >= a.total) return;
  const int tid = threadIdx.x, lane = tid & 63, hf = lane >> 5, j = lane & 31;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6), wr = wv / K::WC, wc = wv % K::WC;
  // the tiles of one (slice, block) are neighbours: they share rows and columns
  // (divisions leave scalars in vector registers)
  const auto scalar = [](unsigned v) { return __builtin_amdgcn_readfirstlane((int)v); };
  const int kt = scalar(id % a.nkt), jt = scalar(id / a.nkt % a.njt), g = scalar(id / a.nkt / a.njt % a.w.nb), sl = scalar(id / a.nkt / a.njt / a.w.nb);
  const int ra = a.w.ra, cb = a.w.cb, j0 = jt * 256, k0 = kt * N * 32;
  const int s_lo = sl * a.w.per, s_hi = s_lo + a.w.per < a.w.nst ? s_lo + a.w.per : a.w.nst, nu = (s_hi - s_lo) * PARTS;
  const unsigned vo = (unsigned)(lane >> 5) * 1024 + (unsigned)(lane & 31) * 16;   // a plane of two groups of 16 channels
  const unsigned lds0 = lds_offset(smem);
  auto half_of = [](int v, int q) { return (unsigned)(PARTS == 1 ? q : v & 1) * 512; };
  auto load = [&](int v, int at) __attribute__((always_inline)) {
    const int s = s_lo + (PARTS == 1 ? v : v >> 1);
    const unsigned on = v < nu ? vo : OOB, dst = lds0 + (unsigned)at * K::UNIT;
#pragma unroll
    for (int m = 0; m < 4; ++m) {
      const int q = m >> 1;
      const u32x4 rs = buf_words(a.w.A[PARTS == 1 ? 0 : q] + ((size_t)s * a.w.nb + g) * ra * 32, (size_t)ra * 64);
      lds16<false>(rs, dst + (unsigned)(wv + 4 * m) * 1024, on, (unsigned)(j0 * 64 + (wv + 4 * (m & 1)) * 2048) + half_of(v, q));
    }
#pragma unroll
    for (int m = 0; m < K::LB; ++m) {
      const int i = wv + 4 * m, q = i >= N;   // (i past 2 N: room that nothing reads)
      const u32x4 rs = buf_words((PARTS == 2 && q ? a.w.B[1] : a.w.B[0]) + ((size_t)s * a.w.nb + g) * cb * 32, (size_t)cb * 64);
      lds16<false>(rs, dst + K::A + (unsigned)i * 1024, i < 2 * N ? on : OOB, (unsigned)(k0 * 64 + (i - q * N) * 2048) + half_of(v, q));
    }
  };
  f32x16 acc[M][NW];
#pragma unroll
  for (int m = 0; m < M; ++m)
#pragma unroll
    for (int n = 0; n < NW; ++n)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[m][n][r] = 0.f;
  auto mul = [](const u32x4 &x, const u32x4 &y, const f32x16 &c) __attribute__((always_inline)) {
    if constexpr (PARTS == 1) return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, x), __builtin_bit_cast(f16x8, y), c, 0, 0, 0);
    else return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, x), __builtin_bit_cast(bf16x8, y), c, 0, 0, 0);
  };
  const unsigned piece = (unsigned)(j >> 4) * 512 + (unsigned)hf * 256 + (unsigned)(j & 15) * 16;   // of a block of 32 channels in a plane
  const unsigned a_rd = (unsigned)wr * M * 1024 + piece, b_rd = K::A + (unsigned)wc * NW * 1024 + piece;
  u32x4 fa[2][M], fb[2][NW];
  auto fetch = [&](int q, int at) __attribute__((always_inline)) {
    const unsigned char *st = smem + at * K::UNIT;
#pragma unroll
    for (int m = 0; m < M; ++m) fa[q][m] = *(const u32x4 *)(st + a_rd + q * 8192 + m * 1024);
#pragma unroll
    for (int n = 0; n < NW; ++n) fb[q][n] = *(const u32x4 *)(st + b_rd + (q * N + n) * 1024);
  };
  auto mul_all = [&](int qa, int qb) __attribute__((always_inline)) {
#pragma unroll
    for (int n = 0; n < NW; ++n)
#pragma unroll
      for (int m = 0; m < M; ++m) acc[m][n] = mul(fa[qa][m], fb[qb][n], acc[m][n]);
    __builtin_amdgcn_sched_barrier(0);
  };
#pragma unroll
  for (int q = 0; q < P; ++q) load(q, q);
  const bool rows_on = j0 + wr * M * 32 < ra;
  int at = 0;   // the buffer of the unit in hand
  // one plane's fragments arrive under the other's products: a unit is waited for in the middle of the one in front of it
  asm volatile("s_waitcnt vmcnt(%0)" :: "n"((P - 1) * (4 + K::LB)) : "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
  fetch(0, 0);
  load(P, P);
  for (int v = 0; v < nu; ++v) {
    const int nx = at == P ? 0 : at + 1;
    fetch(1, at);
    __builtin_amdgcn_sched_barrier(0);
    if (rows_on) mul_all(0, 0);
    if (PARTS == 2 && rows_on) {
      mul_all(1, 0);
      mul_all(0, 1);
    }
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" :: "n"((P - 1) * (4 + K::LB)) : "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    fetch(0, nx);
    load(v + P + 1, at);   // (into the buffer everyone has just left)
    __builtin_amdgcn_sched_barrier(0);
    if (PARTS == 1 && rows_on) mul_all(1, 1);
    at = nx;
  }
  int l = lane;   // (nothing of the following is worth a register in the loop)
  asm volatile("" : "+v"(l));
  // rows past the block: past the buffer's range
  const __amdgpu_buffer_rsrc_t rs = buf(a.w.part + ((size_t)sl * a.w.nb + g) * ra * cb, (size_t)ra * cb * 4);
  const unsigned row = (unsigned)(j0 + wr * M * 32 + 4 * (l >> 5));
#pragma unroll
  for (int n = 0; n < NW; ++n) {   // (whole lines of 32 columns: the transposed product's 16-byte stores took 4 us longer per workgroup)
    const int col = k0 + (wc * NW + n) * 32 + (l & 31);
    const unsigned o = col < cb ? (row * (unsigned)cb + (unsigned)col) * 4 : OOB;
#pragma unroll
    for (int m = 0; m < M; ++m)
#pragma unroll
      for (int r = 0; r < 16; ++r)
        __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(acc[m][n][r]), rs, o, (unsigned)(m * 32 + 8 * (r >> 2) + (r & 3)) * (unsigned)cb * 4, 0);
  }
}

template <int PARTS, int N>
hipError_t launch(const WgradArgs &a, hipStream_t s) {
  static std::atomic<bool> configured{false};
  if (!configured.load()) {
    const hipError_t e = big_lds(tile_wgrad_kernel<PARTS, N>, Wg<PARTS, N>::LDS);
    if (e != hipSuccess) return e;
    configured.store(true);
  }
  hipLaunchKernelGGL((tile_wgrad_kernel<PARTS, N>), dim3(grid8(a.total)), dim3(256), (Wg<PARTS, N>::LDS), s, a);
  return hipGetLastError();
}
// Tiles of 2 and 3 column blocks, in an object of their own (rglru_wgrad_b.hip): in one with the others they move those, and the complex-gated
// forward and backward, whose own instructions are the same, took 214 us instead of 212 (16 blocks of 128, B 1 T 2771; 210 and 204 on another
// card, 197 either way on a third).
hipError_t launch_small(int n, const WgradArgs &a, hipStream_t s);

}  // namespace wgrad
}  // namespace rglru
