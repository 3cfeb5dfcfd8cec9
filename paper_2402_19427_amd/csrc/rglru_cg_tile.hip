// The complex-gated layer in tiles (see rglru_cg_tile.h): preparation, dispatch.
#include "rglru_cg_tile.h"
#include "rglru_fwd_tile.h"
#include "rglru_wgrad.h"

#include <algorithm>

namespace rglru {
using namespace cgt;

namespace {

// Weights in fragment order, [nb][wave][K-step][2][lane][8]: for the gates as half precision (exact for bf16 weights from 6.1e-5 up, finite
// ones stop at 65504), K-step = 16 inputs of (wave, part); transposed, as they are, for dx: K-step = 16 channels of (wave, gate), the two
// being the parts of the input. Zero past the block.
struct CgPrepArgs {
  const unsigned short *W[2];
  u32x4 *wg, *wd;
  int nb, hs, nct;
};
__global__ void __launch_bounds__(256) cg_tile_prep_kernel(CgPrepArgs a) {
  const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
  const int nks = 4 * a.nct, hs = a.hs;
  const size_t per = (size_t)a.nb * a.nct * nks * 2 * 64, wn = (size_t)hs * 2 * hs;
  const bool tr = i >= per;   // (then a thread forms four lanes, from eight rows)
  if (i >= (a.wd ? per + per / 4 : per)) return;
  size_t f = tr ? i - per : i;
  const int q = (int)(tr ? f & 15 : f & 63);
  f >>= tr ? 4 : 6;
  const int two = (int)(f & 1), ks = (int)((f >> 1) % nks), wv = (int)((f >> 1) / nks % a.nct), g = (int)((f >> 1) / nks / a.nct);
  const int mid = (ks >> 1) & 1, k0 = (ks >> 2) * 32 + (ks & 1) * 16;
  if (!tr) {
    const int c = wv * 32 + (q & 31), k = k0 + (q >> 5) * 8;
    u32x4 o = {0u, 0u, 0u, 0u};
    if (c < hs && k < hs) {
      const u32x4 v = *(const u32x4_at2 *)(a.W[two] + g * wn + (size_t)c * 2 * hs + mid * hs + k);
#pragma unroll
      for (int e = 0; e < 4; ++e) o[e] = pack_sat(bf_lo(v[e]), bf_hi(v[e]));
    }
    a.wg[i] = o;
    return;
  }
  const int c = wv * 32 + (q & 7) * 4, k = k0 + (q >> 3) * 8;
  u32x2 v[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) v[e] = u32x2{0u, 0u};
  if (c < hs && k < hs)
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = *(const u32x2_at2 *)(a.W[mid] + g * wn + (size_t)(k + e) * 2 * hs + two * hs + c);
  u32x4 *to = a.wd + f * 64 + (q >> 3) * 32 + (q & 7) * 4;
#pragma unroll
  for (int n = 0; n < 4; ++n) {
    u32x4 o;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const unsigned x = v[2 * e][n >> 1], y = v[2 * e + 1][n >> 1];
      o[e] = n & 1 ? x >> 16 | (y & 0xffff0000u) : (x & 0xffffu) | y << 16;
    }
    to[n] = o;
  }
}
hipError_t launch_prep(const Problem &p, int nct, u32x4 *wg, u32x4 *wd, hipStream_t s) {
  KernelTimer kt("cg_tile_prep_kernel", s);
  CgPrepArgs a;
  a.W[0] = (const unsigned short *)p.W_a; a.W[1] = (const unsigned short *)p.W_x;
  a.wg = wg; a.wd = wd; a.nb = p.nb; a.hs = p.bs; a.nct = nct;
  const size_t frags = (size_t)p.nb * nct * nct * 8 * 64, n = wd ? frags + frags / 4 : frags;
  hipLaunchKernelGGL(cg_tile_prep_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, a);
  return hipGetLastError();
}

int tiles_of(int hs) { return (hs + 31) / 32; }
// Blocks of 80 to 128 channels, for which there are instances, at any alignment. Sequences of 2^31 bytes in fp32 and more run in passes as they did
// before there were tiles, though nothing here stands against them: 16 blocks of 128, T 131072, forward 1.62 ms in tiles and 3.45 in passes,
// backward 4.26 and 8.46.
bool shape_ok(int B, int T, int D, int hs) {
  return (size_t)T * D * 4 < ((size_t)1 << 31) && hs % 16 == 0 && hs > 64 && hs <= 128 && T >= 1 && (size_t)D * 2 * 64 < ((size_t)1 << 31) && (long long)B * ((T + 31) / 32) < ((long long)1 << 28);
}
size_t weight_bytes(int nb, int nct) { return (size_t)nb * nct * nct * 8 * 1024; }

// As many windows as fill the chip, of whole tiles; none is empty. (From 257 units on one, whose second round of workgroups is nearly empty up to
// 511: 260 units of 128 channels, T 2048 398 us, 256 in two windows 291; in the fused kernel, which rounds the same way, 1075 and 520.)
struct Windows {
  int ntile, W, per;
};
Windows windows(int B, int T, int nb) {
  Windows q;
  q.ntile = (T + 31) / 32;
  const int most = std::min(std::max(PER_CU * 256 / std::max(B * nb, 1), 1), q.ntile);
  q.per = (q.ntile + most - 1) / most;
  q.W = (q.ntile + q.per - 1) / q.per;
  return q;
}

struct FwdPlan {
  Windows w;
  size_t off_w, off_agg, off_init, total;
};
FwdPlan plan_fwd(int B, int T, int D, int nb) {
  FwdPlan q;
  q.w = windows(B, T, nb);
  size_t off = 0;
  q.off_w = off; off += weight_bytes(nb, tiles_of(D / 2 / nb));
  q.off_agg = off; off += al256((size_t)B * q.w.W * (D / 2) * 16);
  q.off_init = off; off += al256((size_t)B * (D / 2) * 8);
  q.total = off;
  return q;
}
struct BwdPlan {
  Windows w;
  int nst, S, per;
  size_t off_x, off_pq, n2, off_partA, off_partC, off_edge, off_w, off_agg, off_rev, off_init, off_run, off_partW, total;
};
// have: bytes there are (the weight gradients take as many slices as fit)
BwdPlan plan_bwd(int B, int T, int D, int nb, size_t have) {
  BwdPlan q;
  const int H = D / 2, hs = H / nb;
  q.w = windows(B, T, nb);
  q.nst = B * q.w.ntile;
  q.n2 = al256((size_t)q.nst * D * 64);
  size_t off = 0;
  q.off_x = off; off += 2 * q.n2;
  q.off_pq = off; off += 2 * q.n2;
  q.off_partA = off; off += al256((size_t)B * q.w.W * 4 * H * 4);
  q.off_partC = off; off += al256((size_t)B * q.w.W * 5 * D * 4);
  q.off_edge = off; off += q.w.W > 1 ? al256((size_t)B * q.w.W * 6 * D * 4) : 0;
  // from here on what the weight gradients need no more: their partial sums take the same room
  q.off_partW = q.off_w = off;
  size_t first = off + 2 * weight_bytes(nb, tiles_of(hs));
  q.off_agg = first; first += al256((size_t)B * q.w.W * H * 16);
  q.off_rev = first; first += al256((size_t)B * q.w.W * H * 8);
  q.off_init = first; first += al256((size_t)B * H * 8);
  q.off_run = first; first += al256((size_t)q.nst * 2 * H * 16);
  const size_t one = (size_t)nb * 4 * hs * hs * 4;
  const int S = tile_wgrad_slices(q.nst, nb, 2 * hs, 2 * hs, 2, have > off ? (long long)((have - off) / one) : 1);
  q.per = (q.nst + S - 1) / S;
  q.S = (q.nst + q.per - 1) / q.per;
  q.total = std::max(first, off + q.S * one);
  return q;
}

hipError_t launch(const void *kernel, const char *name, int nct, CgTileArgs &a, int per_unit, hipStream_t s) {
  hipError_t e;
  Instance in;
  in.kernel = kernel; in.lds = nct * REGION;
  if ((e = configure(in)) != hipSuccess) return e;
  a.total = (unsigned)(a.p.B * a.p.nb * per_unit);
  KernelTimer kt(name, s);
  void *args[] = {&a};
  return hipLaunchKernel(kernel, dim3(grid8(a.total)), dim3(nct * 64), args, in.lds, s);
}

}  // namespace

size_t cg_forward_tile_ws_bytes(int B, int T, int D, int nb) {
  return shape_ok(B, T, D, D / 2 / nb) ? plan_fwd(B, T, D, nb).total : 0;
}
// (short sequences: the fused kernel's single launch)
bool cg_forward_tile_supported(const Problem &p) {
  return p.T > pass::RUN && shape_ok(p.B, p.T, p.D, p.bs) && p.ws && (uintptr_t)p.ws % 16 == 0 && p.ws_bytes >= plan_fwd(p.B, p.T, p.D, p.nb).total;
}
hipError_t launch_cg_forward_tile(const Problem &p, hipStream_t s) {
  const FwdPlan q = plan_fwd(p.B, p.T, p.D, p.nb);
  const int nct = tiles_of(p.bs);
  const CgInstance in = cg_instance_fwd(nct, ((uintptr_t)p.u | (uintptr_t)p.y) % 16 != 0);
  char *ws = (char *)p.ws;
  hipError_t e;
  CgTileArgs a = {};
  a.p = p;
  a.ntile = q.w.ntile; a.W = q.w.W; a.per = q.w.per;
  a.wg = (const u32x4 *)(ws + q.off_w);
  a.wagg = (float4 *)(ws + q.off_agg); a.init = (float2 *)(ws + q.off_init);
  if ((e = launch_prep(p, nct, (u32x4 *)(ws + q.off_w), nullptr, s)) != hipSuccess) return e;
  if (a.W > 1 && (e = launch(in.agg, "cg_tile_kernel", nct, a, a.W - 1, s)) != hipSuccess) return e;
  return launch(in.y, "cg_tile_kernel", nct, a, a.W, s);
}

size_t cg_backward_tile_ws_bytes(int B, int T, int D, int nb) {
  return shape_ok(B, T, D, D / 2 / nb) ? al256(plan_bwd(B, T, D, nb, ~(size_t)0).total) : 0;
}
bool cg_backward_tile_supported(const Problem &p) {
  return shape_ok(p.B, p.T, p.D, p.bs) && (uintptr_t)p.ws % 16 == 0 && p.ws_bytes >= plan_bwd(p.B, p.T, p.D, p.nb, p.ws_bytes).total;
}
hipError_t launch_cg_backward_tile(const Problem &p, hipStream_t s) {
  const BwdPlan q = plan_bwd(p.B, p.T, p.D, p.nb, p.ws_bytes);
  const int nct = tiles_of(p.bs);
  const CgInstance in = cg_instance_bwd(nct, ((uintptr_t)p.u | (uintptr_t)p.dy | (uintptr_t)p.du) % 16 != 0);
  char *ws = (char *)p.ws;
  hipError_t e;
  CgTileArgs a = {};
  a.p = p;
  a.ntile = q.w.ntile; a.W = q.w.W; a.per = q.w.per;
  u32x4 *wg = (u32x4 *)(ws + q.off_w), *wd = (u32x4 *)(ws + q.off_w + weight_bytes(p.nb, nct));
  a.wg = wg; a.wd = wd;
  a.wagg = (float4 *)(ws + q.off_agg); a.wrev = (float2 *)(ws + q.off_rev); a.init = (float2 *)(ws + q.off_init);
  a.run = (float4 *)(ws + q.off_run);
  for (int k = 0; k < 2; ++k) {
    a.xF[k] = (unsigned short *)(ws + q.off_x + k * q.n2);
    a.pqF[k] = (unsigned short *)(ws + q.off_pq + k * q.n2);
  }
  a.partA = (float *)(ws + q.off_partA); a.partC = (float *)(ws + q.off_partC);
  a.edge = a.W > 1 ? (float *)(ws + q.off_edge) : nullptr;
  if ((e = launch_prep(p, nct, wg, wd, s)) != hipSuccess) return e;
  if ((e = launch(in.bagg, "cg_tile_kernel", nct, a, a.W, s)) != hipSuccess) return e;
  if ((e = launch(in.bwd, "cg_bwd_tile_kernel", nct, a, a.W, s)) != hipSuccess) return e;
  TileWgrad w;
  for (int k = 0; k < 2; ++k) {
    w.A[k] = a.pqF[k];
    w.B[k] = a.xF[k];
  }
  w.part = (float *)(ws + q.off_partW);
  w.nst = q.nst; w.S = q.S; w.per = q.per;
  w.nb = p.nb; w.ra = w.cb = 2 * p.bs;
  if ((e = launch_tile_wgrad(w, 2, s)) != hipSuccess) return e;
  FinishArgs f = {};
  f.partW = w.part; f.partA = a.partA; f.partC = a.partC; f.sc = nullptr;
  f.S = q.S; f.nA = f.nC = p.B * a.W; f.nrA = 4; f.DA = p.D / 2; f.D = p.D; f.nb = p.nb;
  f.bb = (size_t)p.bs * 2 * p.bs;
  f.dW[0] = p.g.dW_a; f.dW[1] = p.g.dW_x;
  f.rowsA[0] = p.g.db_a; f.rowsA[1] = p.g.db_x; f.rowsA[2] = p.g.dLambda; f.rowsA[3] = p.dtheta;
  for (int k = 0; k < 4; ++k) f.rowsC[k] = p.g.dconv_w ? p.g.dconv_w + (size_t)k * p.D : nullptr;
  f.rowsC[4] = p.g.dconv_b;
  f.edge = a.edge; f.conv_w = p.conv_w; f.du = (unsigned short *)p.du;
  f.B = p.B; f.T = p.T; f.nrt = a.W; f.rows = a.per * 32;
  return launch_finish(f, s);
}

}  // namespace rglru
