// The backward in tiles (see rglru_bwd_fused.h): preparation, weight gradients, dispatch.
#include "rglru_fwd_tile.h"
#include "rglru_wgrad.h"

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
// A thread forms one lane's eight weights from 16 bytes of a row, or, transposed, those of four neighbouring columns from 8 bytes of
// eight rows (a lane's by itself, two bytes at a time: 16 blocks of 352 channels 14 us instead of 9, 10 of 256 6.8 instead of 4.9).
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
  const auto half = [](unsigned v) { return pack_sat(bf_lo(v), bf_hi(v)); };
  if (i < per) {
    size_t f = i;
    const int lane = (int)(f & 63);
    f >>= 6;
    const int gate = (int)(f & 1), ks = (int)((f >> 1) % nks), wv = (int)((f >> 1) / nks % a.nct), g = (int)((f >> 1) / nks / a.nct);
    const int c = wv * 32 + (lane & 31), k0 = ks * 16 + (lane >> 5) * 8;   // column of the product, first of its eight K
    u32x4 o = {0u, 0u, 0u, 0u};
    if (c < a.bs && k0 < a.bs) {
      const u32x4 v = *(const u32x4_at2 *)(a.W[gate] + ((size_t)g * a.bs + c) * a.bs + k0);
#pragma unroll
      for (int e = 0; e < 4; ++e) o[e] = half(v[e]);
    }
    a.wg[i] = o;
  } else if (a.wd && i < per + per / 4) {
    size_t f = i - per;
    const int q = (int)(f & 15);   // K half, four columns
    f >>= 4;
    const int gate = (int)(f & 1), ks = (int)((f >> 1) % nks), wv = (int)((f >> 1) / nks % a.nct), g = (int)((f >> 1) / nks / a.nct);
    const int c = wv * 32 + (q & 7) * 4, k0 = ks * 16 + (q >> 3) * 8;
    u32x2 v[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = u32x2{0u, 0u};
    if (c < a.bs && k0 < a.bs)
#pragma unroll
      for (int e = 0; e < 8; ++e) v[e] = *(const u32x2_at2 *)(a.W[gate] + ((size_t)g * a.bs + k0 + e) * a.bs + c);
    u32x4 *to = a.wd + f * 64 + (q >> 3) * 32 + (q & 7) * 4;
#pragma unroll
    for (int n = 0; n < 4; ++n) {
      u32x4 o;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const unsigned x = v[2 * e][n >> 1], y = v[2 * e + 1][n >> 1];
        o[e] = half(n & 1 ? x >> 16 | (y & 0xffff0000u) : (x & 0xffffu) | y << 16);
      }
      to[n] = o;
    }
  }
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

// ------------------------------------------------------------------------ host side
Instance find_instance(int bs, int var) {
  const int nct = (bs + 31) / 32;
  return nct <= 6 ? find_instance_a(nct, var) : nct <= 8 ? find_instance_b(nct, var) : nct <= 12 ? find_instance_c(nct, var) : find_instance_d(nct, var);
}
int variant(const Problem &p) { return p.reset ? V_PACKED : p.merge == 2 ? V_MERGE_TANH : p.merge ? V_MERGE : V_PLAIN; }

struct Plan {
  int nct, TM, ntile, G, R, S, per, nst;
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
  const int S = tile_wgrad_slices(q.nst, nb, 2 * bs, bs, 1, have > off ? (long long)((have - off) / one) : 1);
  q.per = (q.nst + S - 1) / S;
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
  const size_t frags = (size_t)p.nb * nct * nct * 4 * 64, m = std::max(std::max(wd ? frags + frags / 4 : frags, nrec), (size_t)16);
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
// what it runs best in, for 256 compute units (less makes the slices of the weight gradients fewer); 0: not for this shape
size_t backward_tile_ws_bytes(int B, int T, int D, int nb, bool packed, bool merge) {
  if (!shape_ok(B, T, D, nb, packed)) return 0;
  const Instance in = find_instance(D / nb, packed ? V_PACKED : merge ? V_MERGE : V_PLAIN);
  return in.kernel ? al256(make_plan(B, T, D, nb, packed, in, ~(size_t)0, 256).total + room(B, T, D, D / nb, merge)) : 0;
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
  TileWgrad w;
  w.A[0] = a.pqT; w.B[0] = a.xT; w.A[1] = w.B[1] = nullptr;
  w.part = (float *)(ws + q.off_partW);
  w.nst = q.nst; w.S = q.S; w.per = q.per;
  w.nb = p.nb; w.ra = 2 * p.bs; w.cb = p.bs;
  if ((e = launch_tile_wgrad(w, 1, s)) != hipSuccess) return e;
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
