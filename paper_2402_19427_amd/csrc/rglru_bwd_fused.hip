// The backward in tiles (see rglru_bwd_fused.h): preparation, weight gradients, dispatch.
#include "rglru_fwd_tile.h"

#include <algorithm>
#include <atomic>

namespace rglru {
using namespace fused;

namespace {

// ------------------------------------------------------------------------ preparation
// Weights in half precision (exact for bf16 weights from 6.1e-5 up, finite ones stop at 65504) in matrix-fragment order,
// [nb][wave][K-step][gate][lane][8]: as they are (rows of W, for the gates) and transposed (for dx), zero
// past the block; the status word and the record rings cleared; the last workgroup forms the scale.
struct PrepArgs {
  const unsigned short *W[2];
  u32x4 *wg, *wd;
  uint4 *zero, *rec;    // the status word's 256 bytes; the record rings
  size_t n16, nrec;     // 16-byte words of both
  float *sc;
  int nb, bs, nct;
};
__global__ void __launch_bounds__(256) tile_prep_kernel(PrepArgs a) {
  if (a.sc && blockIdx.x == gridDim.x - 1) {
    scale_from_parts(a.sc, 4);
    return;
  }
  const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (i < a.n16) a.zero[i] = cleared_word(a.zero, i, true);
  if (i < a.nrec) a.rec[i] = make_uint4(0u, 0u, 0u, 0u);
  const int nks = 2 * a.nct;
  const size_t per = (size_t)a.nb * a.nct * nks * 2 * 64;
  if (i >= (a.wd ? 2 * per : per)) return;
  const bool tr = i >= per;
  size_t f = tr ? i - per : i;
  const int lane = (int)(f & 63);
  f >>= 6;
  const int gate = (int)(f & 1), ks = (int)((f >> 1) % nks), wv = (int)((f >> 1) / nks % a.nct), g = (int)((f >> 1) / nks / a.nct);
  const unsigned short *src = a.W[gate] + (size_t)g * a.bs * a.bs;
  const int c = wv * 32 + (lane & 31), k0 = ks * 16 + (lane >> 5) * 8;   // column of the product, first of its eight K
  u32x4 o = {0u, 0u, 0u, 0u};
  if (c < a.bs && k0 < a.bs) {
    unsigned short v[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = tr ? src[(size_t)(k0 + e) * a.bs + c] : src[(size_t)c * a.bs + k0 + e];
#pragma unroll
    for (int e = 0; e < 4; ++e)
      o[e] = pack_sat(__uint_as_float((unsigned)v[2 * e] << 16), __uint_as_float((unsigned)v[2 * e + 1] << 16));
  }
  (tr ? a.wd : a.wg)[tr ? i - per : i] = o;
}

// Partial maxima of |dout GeLU(branch)| and |dhT|, one per workgroup of SCALE_PARTS (as absmax_kernel
// leaves them for a dy handed in): 16 bytes of both per lane, four pairs in flight. Read at the rate of memory
// (B 8 T 2048, 2560 channels: 39 us, 168 MB, 4.3 TB/s).
template <bool TANH>
__global__ void __launch_bounds__(256) absmax_merge_kernel(const u32x4 *dout, const u32x4 *branch, size_t n8, const float *w, size_t nw,
                                                           unsigned *parts) {
  float m = 0.f;
  auto take = [&](float v) {   // (NaNs are left out of the range estimate)
    const unsigned b = __float_as_uint(v) & 0x7fffffffu;
    m = b <= 0x7f800000u ? fmaxf(m, __uint_as_float(b)) : m;
  };
  const size_t stride = (size_t)SCALE_PARTS * 256;
  constexpr int U = 4;
  for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n8; i += U * stride) {
    u32x4 d[U], z[U];
#pragma unroll
    for (int k = 0; k < U; ++k) {
      const size_t q = i + k * stride < n8 ? i + k * stride : i;
      d[k] = dout[q];
      z[k] = branch[q];
    }
#pragma unroll
    for (int k = 0; k < U; ++k)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        take(bf_lo(d[k][e]) * gelu<TANH, true>(bf_lo(z[k][e])));
        take(bf_hi(d[k][e]) * gelu<TANH, true>(bf_hi(z[k][e])));
      }
  }
  if (w)
    for (size_t k = (size_t)blockIdx.x * 256 + threadIdx.x; k < nw; k += stride) take(w[k]);
  for (int o = 32; o > 0; o >>= 1) m = fmaxf(m, __shfl_xor(m, o));
  __shared__ float wm[4];
  if ((threadIdx.x & 63) == 0) wm[threadIdx.x >> 6] = m;
  __syncthreads();
  if (threadIdx.x == 0) parts[blockIdx.x] = __float_as_uint(fmaxf(fmaxf(wm[0], wm[1]), fmaxf(wm[2], wm[3])));
}

// ------------------------------------------------------------------------ weight gradients
// part[slice][g][gate bs + j][k] = sum over the slice's steps of S dp|dq[j][t] x[k][t]: 256 x 128 outputs per
// workgroup of four waves, 64 x 128 each. Both operands lie time fastest, so that a fragment is one 16-byte
// read; stages of 32 steps (256 + 128 rows of 64 bytes, pieces permuted by the row) by direct-to-LDS loads,
// three buffers, two stages in flight (a counted wait: each wave loads six pieces of 16 rows per stage).
// Bound by the operands' way into LDS: 24 KB per stage for 32 products of a wave. B 16 T 4096, 16 blocks of 256
// channels: 346 us (0.79 PFLOP/s; 490 as it was, with x formed again from u); twice that with the loads marked streaming:
// neighbouring workgroups share rows and want them in L2. Blocks that do not fill 256 x 128 pay for the rest: 160
// channels use 39 % of their products.
constexpr int WT_A = 256 * 64, WT_B = 128 * 64, WT_STAGE = WT_A + WT_B, WT_LDS = 3 * WT_STAGE;
static_assert(WT_LDS <= 80 * 1024, "two workgroups per CU");
struct WgradArgs {
  const unsigned short *pqT, *xT;
  float *part;
  int nst, per;                 // stages in all, per slice
  int D, nb, bs, njt, nkt;
  unsigned total;
};
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2))) tile_wgrad_kernel(WgradArgs a) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const unsigned id = xcd_id();
  if (id >= a.total) return;
  const int tid = threadIdx.x, lane = tid & 63, hf = lane >> 5, j = lane & 31;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  // the tiles of one (slice, block) are neighbours: they share rows
  const int kt = (int)(id % a.nkt), jt = (int)(id / a.nkt % a.njt), g = (int)(id / a.nkt / a.njt % a.nb),
            sl = (int)(id / a.nkt / a.njt / a.nb);
  const int D = a.D, bs = a.bs, j0 = jt * 256, k0 = kt * 128;
  const int s_lo = sl * a.per, s_hi = s_lo + a.per < a.nst ? s_lo + a.per : a.nst;
  const unsigned vo = (unsigned)(lane >> 2) * 64 + (unsigned)((lane & 3) ^ ((lane >> 3) & 3)) * 16;   // key: (row >> 1) & 3
  auto load_stage = [&](int s) __attribute__((always_inline)) {
    const size_t at = ((size_t)s * D + (size_t)g * bs) * 32;
    const u32x4 q_rs = buf_words(a.pqT + 2 * at, (size_t)2 * bs * 64), x_rs = buf_words(a.xT + at, (size_t)bs * 64);
    const unsigned st = lds_offset(smem) + (unsigned)(s - s_lo) % 3u * WT_STAGE;
#pragma unroll
    for (int m = 0; m < 4; ++m) {
      const int i = wv + 4 * m;
      lds16<false>(q_rs, st + i * 1024, vo, (unsigned)(j0 + 16 * i) * 64);
    }
#pragma unroll
    for (int m = 0; m < 2; ++m) {
      const int i = wv + 4 * m;
      lds16<false>(x_rs, st + WT_A + i * 1024, vo, (unsigned)(k0 + 16 * i) * 64);
    }
  };
  f32x16 acc[2][4];
#pragma unroll
  for (int m = 0; m < 2; ++m)
#pragma unroll
    for (int n = 0; n < 4; ++n)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[m][n][r] = 0.f;
  const unsigned a_rd = (unsigned)(wv * 64 + j) * 64 + (unsigned)(hf ^ key_b(j)) * 16, b_rd = WT_A + (unsigned)j * 64 + (unsigned)(hf ^ key_b(j)) * 16;
  const int njb = (2 * bs - j0 - wv * 64 + 31) / 32, nkb = (bs - k0 + 31) / 32;   // 32-blocks that exist
  if (s_lo < s_hi) load_stage(s_lo);
  if (s_lo + 1 < s_hi) load_stage(s_lo + 1);
  for (int s = s_lo; s < s_hi; ++s) {
    if (s + 1 < s_hi) asm volatile("s_waitcnt vmcnt(6)" ::: "memory");   // this stage is there, the next may be under way
    else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    lds_barrier();
    if (s + 2 < s_hi) load_stage(s + 2);   // (into the buffer everyone has just left)
    if (njb <= 0) continue;
    const unsigned char *st = smem + (unsigned)(s - s_lo) % 3u * WT_STAGE;
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      f16x8 fa[2], fb[4];
#pragma unroll
      for (int m = 0; m < 2; ++m) fa[m] = *(const f16x8 *)(st + ((a_rd + m * 2048) ^ (ks * 32)));
#pragma unroll
      for (int n = 0; n < 4; ++n) fb[n] = *(const f16x8 *)(st + ((b_rd + n * 2048) ^ (ks * 32)));
#pragma unroll
      for (int n = 0; n < 4; ++n)
        if (n < nkb)
#pragma unroll
          for (int m = 0; m < 2; ++m)
            acc[m][n] = __builtin_amdgcn_mfma_f32_32x32x16_f16(fa[m], fb[n], acc[m][n], 0, 0, 0);
    }
  }
  float *out = a.part + ((size_t)sl * a.nb + g) * 2 * bs * bs;
#pragma unroll
  for (int m = 0; m < 2; ++m)
#pragma unroll
    for (int n = 0; n < 4; ++n)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int row = j0 + wv * 64 + m * 32 + 8 * (r >> 2) + 4 * hf + (r & 3), col = k0 + n * 32 + j;
        if (row < 2 * bs && col < bs) out[(size_t)row * bs + col] = acc[m][n][r];
      }
}

// ------------------------------------------------------------------------ host side
Instance find_instance(int bs, int var) {
  const int nct = (bs + 31) / 32;
  return nct <= 6 ? find_instance_a(nct, var) : nct <= 8 ? find_instance_b(nct, var) : nct <= 12 ? find_instance_c(nct, var) : find_instance_d(nct, var);
}
int variant(const Problem &p) { return p.reset ? V_PACKED : p.merge == 2 ? V_MERGE_TANH : p.merge ? V_MERGE : V_PLAIN; }

struct Plan {
  int nct, TM, ntile, G, R, S, per, nst, njt, nkt;
  size_t off_sc, off_partA, off_partC, off_edge, off_masks, off_rec, off_x, off_pq, off_w, off_partW, wbytes, total;
};
// have: bytes there are (the weight gradients take as many slices as fit); ncu: compute units
Plan make_plan(int B, int T, int D, int nb, bool packed, const Instance &in, size_t have, int ncu) {
  Plan q;
  const int bs = D / nb, units = B * nb;
  q.nct = (bs + 31) / 32;
  q.TM = 32 * in.mt;
  q.ntile = (T + q.TM - 1) / q.TM;
  q.G = pick_slices(units, q.ntile, in.per_cu * ncu, 16);   // (slices wait for each other: all run at once)
  q.R = ring_depth(q.G);
  q.nst = B * q.ntile * in.mt;
  q.njt = (2 * bs + 255) / 256;
  q.nkt = (bs + 127) / 128;
  const size_t n2 = (size_t)B * q.ntile * q.TM * D * 2;
  size_t off = 256;   // the status word
  q.off_sc = off; off += al256(SCALE_CELL_BYTES);
  q.off_partA = off; off += al256((size_t)B * q.G * 3 * D * 4);
  q.off_partC = off; off += al256((size_t)B * q.G * 5 * D * 4);
  q.off_edge = off; off += q.G > 1 ? al256((size_t)B * q.ntile * 6 * D * 4) : 0;
  q.off_masks = off; off += packed ? al256((size_t)B * ((T + 31) / 32) * sizeof(uint4)) : 0;
  q.off_x = off; off += al256(n2);
  q.off_pq = off; off += al256(2 * n2);
  // from here on what the weight gradients need no more: their partial sums take the same room
  q.wbytes = (size_t)nb * q.nct * q.nct * 2 * 2 * 1024;
  q.off_partW = q.off_w = off;
  q.off_rec = off + 2 * q.wbytes;
  const size_t first = 2 * q.wbytes + (q.G > 1 ? (size_t)units * q.R * q.nct * 32 * sizeof(u64) : 0);
  const size_t one = (size_t)nb * 2 * bs * bs * 4;
  // slices of the weight gradients: two workgroups per CU, none shorter than 8 stages, as many as there is room for
  const long long tiles = (long long)nb * q.njt * q.nkt;
  long long S = (2 * 256 + tiles - 1) / tiles;
  if (S > q.nst / 8) S = q.nst / 8;
  const long long fit = have > off ? (long long)((have - off) / one) : 0;
  if (S > fit) S = fit;
  if (S < 1) S = 1;
  q.per = (int)((q.nst + S - 1) / S);
  q.S = (q.nst + q.per - 1) / q.per;
  q.total = off + std::max(first, q.S * one);
  return q;
}

// What is staged 16 bytes at a time lies on that grid or is copied there first, behind the plan; blocks of other sizes
// than the fused kernels' bring the room for that whatever their tensors' alignment is, so that results do not
// depend on it.
constexpr int COPIES = 4;   // u; y; dy or du (a tile's rows of dy are read before its rows of du are written, and by nobody else); branch or dbranch
size_t room(int B, int T, int D, int bs, bool merge) {
  return bs == BS ? 0 : (merge ? COPIES : COPIES - 1) * al256((size_t)B * T * D * 2) + 16;
}
bool on_grid(const Problem &p) {
  return ((uintptr_t)p.u | (uintptr_t)p.y_in | (uintptr_t)p.dy | (uintptr_t)p.branch | (uintptr_t)p.du | (uintptr_t)p.dbranch) % 16 == 0;
}
// (Sequences of 2^32 bytes of fp32 and more of 256 channels, and packed rows of other blocks, ran on the general kernels in plain fp32
// arithmetic before there were tiles, and do so: dW_x of packed rows of 128 channels is 3e-7 off, 2e-4 in tiles.)
bool shape_ok(int B, int T, int D, int nb, bool packed) {
  if (D / nb == BS ? (size_t)T * D * 4 >= ((size_t)1 << 32) : packed) return false;
  return D / nb % 16 == 0 && T >= 1 && (long long)B * ((T + 31) / 32) < ((long long)1 << 30) && (size_t)D * 2 * 64 < ((size_t)1 << 31);
}

// Where tiles are the faster backward: everywhere but for a few sequences' blocks of many steps, where 16 slices each leave most of
// the chip idle while what runs instead (the passes; at 256 channels three kernels) is parallel over all of time. What decides is how
// many workgroups there are (16 per unit of sequence and block) and how often each goes round. us, tiles : passes, over block sizes, units
// and T from 300 to 32768 (4506 calls):
// - 112 to 192 channels: up to 8 units (9 up to 128 channels), from 9 - 12 rounds on, more for more units (160, one block: T 4096
//   97 : 120, T 16384 322 : 141; 8 units, T 4096 108 : 129, T 16384 337 : 347, with the merge 411 : 386).
// - 208 to 240: from 8 rounds of 32 steps on, without the merge (tiles of 64 steps) up to 4 units, with it up to 8 (240, 3 blocks: T 4096
//   106 : 126, T 8192 186 : 149).
// - 256: with the merge, up to 3 units of 32 rounds and more (one block: T 8192 246 : 280, T 32768 879 : 762).
// - 272 to 384: up to 7 units (8 with the merge, or above 320 channels from 16 rounds on), from 5 - 6 rounds on (352, one block: T 2048 104 : 123, T 4096 174 : 127; 384, 7
//   blocks, T 4096 211 : 228, T 8192 388 : 382).
// - 400 to 512, whose tiles spill: up to 10 units from 4 rounds on, 3 above 448 channels (512, 4 blocks: T 1024 115 : 141, T 2048
//   179 : 155, T 4096 318 : 183; 10 blocks, T 6144 620 : 581); 11 from 8 on.
// Calls past these lines gave up to five times their time away to the tiles (512, one block, T 16384).
bool worth(int B, int T, int nb, int bs, int var, const Instance &in) {
  const bool merge = var == V_MERGE || var == V_MERGE_TANH;
  if (T <= 256) return true;   // (even a single slice's 8 rounds take no longer than the launches of the passes)
  // (for 256 compute units: the same rule where no card is visible)
  const int ntile = (T + 32 * in.mt - 1) / (32 * in.mt), G = pick_slices(B * nb, ntile, in.per_cu * 256, 16);
  const long long w = (long long)B * nb * G, rounds = (long long)((ntile + G - 1) / G) * in.mt;   // workgroups; rounds of 32 steps
  const auto units = [&](int n) { return w <= 16 * n; };
  if (bs <= 192) return !units(bs <= 128 ? 9 : 8) || 32 * rounds <= 256 + w;
  if (bs < BS) return !units(merge ? 8 : 4) || rounds <= (merge ? 7 : 7 + w / 16);
  if (bs == BS) return !merge || !units(3) || rounds < 32;
  if (bs <= 384) return !units(merge || (bs > 320 && rounds >= 16) ? 8 : 7) || 64 * rounds <= (bs <= 320 ? 320 : 256) + w;
  if (units(10)) return rounds <= (bs <= 448 ? 3 : 2);
  return !units(11) || rounds <= 7;
}

}  // namespace

// these kernels ask for more than the default LDS limit; told once per instance
hipError_t fused::configure(const Instance &in) {
  static std::atomic<const void *> done[128];
  for (auto &d : done) {
    const void *k = d.load();
    if (k == in.kernel) return hipSuccess;
    if (k) continue;
    hipError_t e = hipFuncSetAttribute(in.kernel, hipFuncAttributeMaxDynamicSharedMemorySize, in.lds);
    if (e != hipSuccess) return e;
    const void *none = nullptr;
    if (d.compare_exchange_strong(none, in.kernel)) return hipSuccess;
    if (none == in.kernel) return hipSuccess;
  }
  return hipFuncSetAttribute(in.kernel, hipFuncAttributeMaxDynamicSharedMemorySize, in.lds);
}
int fused::compute_units() { return std::min(num_cu(), 256); }

hipError_t fused::launch_tile_prep(const Problem &p, int nct, u32x4 *wg, u32x4 *wd, void *status, void *rec, size_t nrec, float *sc, hipStream_t s) {
  KernelTimer kt("tile_prep_kernel", s);
  PrepArgs a;
  a.W[0] = (const unsigned short *)p.W_a; a.W[1] = (const unsigned short *)p.W_x;
  a.wg = wg; a.wd = wd;
  a.zero = (uint4 *)status; a.n16 = 16;
  a.rec = (uint4 *)rec; a.nrec = nrec;
  a.sc = sc; a.nb = p.nb; a.bs = p.bs; a.nct = nct;
  const size_t frags = (size_t)p.nb * nct * nct * 4 * 64 * (wd ? 2 : 1), m = std::max(std::max(frags, nrec), (size_t)16);
  hipLaunchKernelGGL(tile_prep_kernel, dim3((unsigned)((m + 255) / 256 + (sc ? 1 : 0))), dim3(256), 0, s, a);
  return hipGetLastError();
}

bool backward_tile_supported(const Problem &p, bool bf) {
  if (!bf || p.dy_lo || !shape_ok(p.B, p.T, p.D, p.nb, p.reset != nullptr) || (uintptr_t)p.ws % 16 != 0) return false;
  const Instance in = find_instance(p.bs, variant(p));
  if (!in.kernel || (p.bs == BS && !on_grid(p))) return false;
  if (!worth(p.B, p.T, p.nb, p.bs, variant(p), in) && (p.bs == BS ? backward_mfma_supported(p, true) : backward_pass_supported(p, true))) return false;
  const size_t r = room(p.B, p.T, p.D, p.bs, p.merge != 0), have = p.ws_bytes > r ? p.ws_bytes - r : 0;
  return have >= make_plan(p.B, p.T, p.D, p.nb, p.reset != nullptr, in, have, compute_units()).total;
}
// the least it runs in, for 256 compute units; 0: not for this shape
size_t backward_tile_ws_bytes(int B, int T, int D, int nb, bool packed, bool merge) {
  if (!shape_ok(B, T, D, nb, packed)) return 0;
  const Instance in = find_instance(D / nb, packed ? V_PACKED : merge ? V_MERGE : V_PLAIN);
  return in.kernel ? al256(make_plan(B, T, D, nb, packed, in, 0, 256).total + room(B, T, D, D / nb, merge)) : 0;
}

hipError_t launch_backward_tile(const Problem &call, hipStream_t s) {
  Problem p = call;
  const Instance in = find_instance(p.bs, variant(p));
  const size_t n2 = al256((size_t)p.B * p.T * p.D * 2), r = room(p.B, p.T, p.D, p.bs, p.merge != 0), have = p.ws_bytes - r;
  const Plan q = make_plan(p.B, p.T, p.D, p.nb, p.reset != nullptr, in, have, compute_units());
  char *ws = (char *)p.ws, *copy = ws + (have + 15) / 16 * 16;
  hipError_t e;
  const void **src[] = {&p.u, &p.y_in, &p.dy, &p.branch};
  void *none = nullptr, **dst[] = {&none, &none, &p.du, &p.dbranch};
  for (int k = 0; k < COPIES; ++k, copy += n2) {   // (no merge: branch and dbranch are null)
    if ((uintptr_t)*src[k] % 16 != 0) {
      if ((e = launch_realign(*src[k], copy, (size_t)p.B * p.T * p.D, s)) != hipSuccess) return e;
      *src[k] = copy;
    }
    if ((uintptr_t)*dst[k] % 16 != 0) *dst[k] = copy;
  }
  if ((e = configure(in)) != hipSuccess) return e;
  float *sc = (float *)(ws + q.off_sc);
  const size_t n = (size_t)p.B * p.T * p.D;
  if (p.merge) {
    KernelTimer kt("absmax_merge_kernel", s);
    const auto kernel = p.merge == 2 ? absmax_merge_kernel<true> : absmax_merge_kernel<false>;
    hipLaunchKernelGGL(kernel, dim3(SCALE_PARTS), dim3(256), 0, s, (const u32x4 *)p.dy, (const u32x4 *)p.branch, n / 8, p.dhT,
                       (size_t)p.B * p.D, (unsigned *)sc + 64);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  } else if ((e = launch_absmax(p.dy, n, p.dhT, (size_t)p.B * p.D, sc, s)) != hipSuccess) {
    return e;
  }
  uint4 *masks = (uint4 *)(ws + q.off_masks);
  if (p.reset && (e = launch_reset_masks(p.reset, masks, nullptr, p.B, p.T, s)) != hipSuccess) return e;
  u32x4 *wg = (u32x4 *)(ws + q.off_w), *wd = (u32x4 *)(ws + q.off_w + q.wbytes);
  const size_t nrec = q.G > 1 ? (size_t)p.B * p.nb * q.R * q.nct * 32 * sizeof(u64) / 16 : 0;
  if ((e = launch_tile_prep(p, q.nct, wg, wd, ws, ws + q.off_rec, nrec, sc, s)) != hipSuccess) return e;
  FusedArgs a;
  a.p = p;
  a.G = q.G; a.ntile = q.ntile; a.R = q.R;
  a.total = (unsigned)(p.B * p.nb * q.G);
  a.rec = (u64 *)(ws + q.off_rec);
  a.err = (int *)ws;
  a.wg = wg; a.wd = wd;
  a.xT = (unsigned short *)(ws + q.off_x); a.pqT = (unsigned short *)(ws + q.off_pq);
  a.sc = sc;
  a.partA = (float *)(ws + q.off_partA); a.partC = (float *)(ws + q.off_partC);
  a.edge = q.G > 1 ? (float *)(ws + q.off_edge) : nullptr;
  a.rmask = p.reset ? masks : nullptr;
  a.nmask = (p.T + 31) / 32;
  {
    KernelTimer kt("bwd_tile_kernel", s);
    void *args[] = {&a};
    if ((e = hipLaunchKernel(in.kernel, dim3(grid8(a.total)), dim3(in.waves * 64), args, in.lds, s)) != hipSuccess) return e;
  }
  {
    static std::atomic<bool> configured{false};
    if (!configured.load()) {
      if ((e = big_lds(tile_wgrad_kernel, WT_LDS)) != hipSuccess) return e;
      configured.store(true);
    }
    KernelTimer kt("tile_wgrad_kernel", s);
    WgradArgs w;
    w.pqT = a.pqT; w.xT = a.xT; w.part = (float *)(ws + q.off_partW);
    w.nst = q.nst; w.per = q.per;
    w.D = p.D; w.nb = p.nb; w.bs = p.bs; w.njt = q.njt; w.nkt = q.nkt;
    w.total = (unsigned)q.S * p.nb * q.njt * q.nkt;
    hipLaunchKernelGGL(tile_wgrad_kernel, dim3(grid8(w.total)), dim3(256), WT_LDS, s, w);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  FinishArgs f;
  f.partW = (const float *)(ws + q.off_partW);
  f.partA = a.partA; f.partC = a.partC; f.sc = sc;
  f.S = q.S; f.nA = f.nC = p.B * q.G; f.nrA = 3; f.DA = f.D = p.D; f.nb = p.nb;
  f.bb = (size_t)p.bs * p.bs;
  f.dW[0] = p.g.dW_a; f.dW[1] = p.g.dW_x;
  f.rowsA[0] = p.g.db_a; f.rowsA[1] = p.g.db_x; f.rowsA[2] = p.g.dLambda; f.rowsA[3] = nullptr;
  for (int k = 0; k < 4; ++k) f.rowsC[k] = p.g.dconv_w ? p.g.dconv_w + (size_t)k * p.D : nullptr;
  f.rowsC[4] = p.g.dconv_b;
  f.edge = a.edge; f.conv_w = p.conv_w; f.du = (unsigned short *)p.du;
  f.B = p.B; f.T = p.T; f.nrt = q.ntile; f.rows = q.TM;
  f.rmask = a.rmask; f.nmask = a.nmask;
  if ((e = launch_finish(f, s)) != hipSuccess) return e;
  for (const auto &[to, from] : {std::make_pair(call.du, p.du), std::make_pair(call.dbranch, p.dbranch)})
    if (to != from && (e = launch_realign(from, to, (size_t)p.B * p.T * p.D, s)) != hipSuccess) return e;
  return hipSuccess;
}

}  // namespace rglru
