// Forward for fp32 storage and gate blocks of a multiple of 16 channels, parallel over time, in two
// launches (three beyond 64 runs):
//   1. f32_coeff_kernel  Conv1D, gate products on the fp32 matrix cores (true fp32 products and sums:
//                        the contract is 1e-5), eqs. (1)-(3) with accurate math -> a_t, b_t, and the
//                        affine aggregate of every run of 16 steps
//   2. f32_apply_kernel  a run's incoming state out of the aggregates in front of it, y, the merge, hT,
//                        the new Conv1D ring
// A small layer (256 channels, 256 steps) is bound by launches and by the latency of one workgroup's
// chain, so a workgroup takes 16 steps of one gate block and every wave 16 x 16 outputs: weights and
// inputs are requested together, 32 input channels of the weights at a time pass through LDS, and the
// local scan runs on the accumulators (lane: four consecutive steps of a channel). It replaces a pass
// with one thread per output and 16 steps, a thread per channel walking the sequence, a clear and a
// ring update: 31 -> 13 us at B1 T256 D256 in four blocks.
// Where there are enough workgroups to fill the chip without it, one takes four runs: every run
// re-stages the block's weights otherwise (B4 T1000 D1024 in 8 blocks: 262 MB from L2).
#include "rglru_gelu.h"
#include "rglru_generic.h"
#include "rglru_mfma.h"
#include "rglru_pass.h"

namespace rglru {
namespace {

constexpr int FT = 16;        // steps per run
constexpr int KC = 32;        // input channels of the weights in LDS at a time
constexpr int WS = KC + 4;    // row stride of the weight tile: rows 16 bytes apart in the banks
constexpr int MAX_DIRECT = 64;   // runs whose aggregates every run reads itself
typedef float f32x4 __attribute__((ext_vector_type(4)));

struct CoeffArgs {
  Problem p;
  int t_lo, n, nrun;     // the chunk of steps in hand
  float *A, *Bv;         // [B][n][D]
  float2 *agg;           // [B][nrun][D]
  const float *h0;       // first piece: copied into `cell`, or null
  float *cell;
};

// MAXT: column tiles of 16 outputs per wave (a block of up to 64 MAXT channels); RT: runs per workgroup
template <int MAXT, int RT>
__global__ void __launch_bounds__(NTHREADS) f32_coeff_kernel(CoeffArgs a) {
  extern __shared__ __attribute__((aligned(16))) float smem[];
  const Problem &p = a.p;
  const int g = blockIdx.x, run = blockIdx.y * RT, b = blockIdx.z, bs = p.bs, D = p.D, tid = threadIdx.x;
  const int lane = tid & 63, wv = tid >> 6, j = lane & 15, kq = lane >> 4;
  const int l0 = run * FT, t0 = a.t_lo + l0, nt = a.n - l0 < RT * FT ? a.n - l0 : RT * FT;
  const int xst = bs + 4;
  float *xs = smem, *wl = smem + RT * FT * xst;   // x tile; weights [2][bs][WS]
  // ---- weights of the first chunk, requested in front of everything else
  const int npiece = 2 * bs * (KC / 4);      // 16-byte pieces of a chunk
  constexpr int NP = 8;                      // pieces in flight per thread
  const int nkc = (bs + KC - 1) / KC;
  f32x4 pw[NP];
  auto piece = [&](int kc, int i) __attribute__((always_inline)) -> const float * {
    const int c = i % (KC / 4), r = i / (KC / 4) % bs, gate = i / (KC / 4) / bs;
    const int k = kc * KC + c * 4;
    return (const float *)(gate ? p.W_x : p.W_a) + ((size_t)g * bs + r) * bs + (k < bs ? k : bs - 4);
  };
  auto fetch = [&](int kc, int from) __attribute__((always_inline)) {
#pragma unroll
    for (int q = 0; q < NP; ++q) {
      const int i = from + q * NTHREADS + tid;
      pw[q] = *(const f32x4 *)piece(kc, i < npiece ? i : npiece - 1);
    }
  };
  auto park = [&](int from) __attribute__((always_inline)) {
#pragma unroll
    for (int q = 0; q < NP; ++q) {
      const int i = from + q * NTHREADS + tid;
      if (i < npiece) *(f32x4 *)(wl + (i / (KC / 4)) * WS + (i % (KC / 4)) * 4) = pw[q];
    }
  };
  fetch(0, 0);
  // ---- Conv1D: a thread takes four steps of a channel
  for (int i = tid; i < (RT * FT / 4) * bs; i += NTHREADS) {
    const int c = i % bs, r0 = (i / bs) * 4, d = g * bs + c;
    float in[7], w[4];
    const float *u = (const float *)p.u + (size_t)b * p.T * D + d;
#pragma unroll
    for (int q = 0; q < 7; ++q) {
      const int t = t0 + r0 - 3 + q;
      const int tc = t < 0 ? 0 : (t < p.T ? t : p.T - 1);
      in[q] = u[(size_t)tc * D];
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) w[k] = p.conv_w ? p.conv_w[(size_t)k * D + d] : (k == 0 ? 1.f : 0.f);
    const float bias = p.conv_w && p.conv_b ? p.conv_b[d] : 0.f;
    if (t0 + r0 < 3) {   // inputs in front of the sequence
#pragma unroll
      for (int q = 0; q < 3; ++q)
        if (t0 + r0 - 3 + q < 0) in[q] = p.conv_w ? input_at<float>(p, b, t0 + r0 - 3 + q, d) : 0.f;
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      float x = bias;
#pragma unroll
      for (int k = 0; k < 4; ++k) x = fmaf(w[k], in[r + 3 - k], x);
      xs[(r0 + r) * xst + c] = p.conv_w ? x : in[r + 3];
    }
  }
  // ---- products: a wave's column tiles wv, wv + 4, ... of 16 outputs
  const int ntile = bs / 16;
  f32x4 accp[MAXT][RT], accq[MAXT][RT];
#pragma unroll
  for (int q = 0; q < MAXT; ++q)
#pragma unroll
    for (int m = 0; m < RT; ++m) accp[q][m] = accq[q][m] = f32x4{0.f, 0.f, 0.f, 0.f};
  for (int kc = 0; kc < nkc; ++kc) {
    if (kc > 0) __syncthreads();
    park(0);
    for (int from = NP * NTHREADS; from < npiece; from += NP * NTHREADS) {
      fetch(kc, from);
      park(from);
    }
    __syncthreads();
    if (kc + 1 < nkc) fetch(kc + 1, 0);
    const int nk = bs - kc * KC < KC ? bs - kc * KC : KC;   // 16 or 32
    for (int k0 = 0; k0 < nk; k0 += 16) {
      // lane (j, kq): four consecutive k of row / column j; product e contracts k = 4 kq + e
      f32x4 xa[RT];
#pragma unroll
      for (int m = 0; m < RT; ++m) xa[m] = *(const f32x4 *)(xs + (m * FT + j) * xst + kc * KC + k0 + kq * 4);
#pragma unroll
      for (int q = 0; q < MAXT; ++q) {
        const int ct = wv + 4 * q;
        if (ct < ntile) {
          const f32x4 wa = *(const f32x4 *)(wl + (ct * 16 + j) * WS + k0 + kq * 4);
          const f32x4 wx = *(const f32x4 *)(wl + (bs + ct * 16 + j) * WS + k0 + kq * 4);
#pragma unroll
          for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int m = 0; m < RT; ++m) {
              accp[q][m] = __builtin_amdgcn_mfma_f32_16x16x4f32(xa[m][e], wa[e], accp[q][m], 0, 0, 0);
              accq[q][m] = __builtin_amdgcn_mfma_f32_16x16x4f32(xa[m][e], wx[e], accq[q][m], 0, 0, 0);
            }
        }
      }
    }
  }
  // ---- eqs. (1)-(3): lane (j, kq) holds steps 4 kq .. 4 kq + 3 of channel 16 ct + j
#pragma unroll
  for (int q = 0; q < MAXT; ++q) {
    const int ct = wv + 4 * q;
    if (ct >= ntile) break;
    const int c = ct * 16 + j, d = g * bs + c;
    if (a.h0 && run == 0 && kq == 0) a.cell[(size_t)b * D + d] = a.h0[(size_t)b * D + d];
    const float ba = p.b_a[d], bx = p.b_x[d], neg_cs = -p.c * softplus_f(-p.Lambda[d]);
#pragma unroll
    for (int m = 0; m < RT; ++m) {
      if (m * FT >= nt) break;
      float Ar = 1.f, Er = 0.f;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int tt = m * FT + kq * 4 + r;
        const float rg = sigmoid_f(accp[q][m][r] + ba), ig = sigmoid_f(accq[q][m][r] + bx), la = neg_cs * rg;
        float av = expf(la), bv = sqrtf(-expm1f(2.f * la)) * (ig * xs[tt * xst + c]);
        if (tt < nt) {
          const size_t o = ((size_t)b * a.n + l0 + tt) * D + d;
          a.A[o] = av;
          a.Bv[o] = bv;
        } else {   // steps past the end leave the state untouched
          av = 1.f;
          bv = 0.f;
        }
        Er = fmaf(av, Er, bv);
        Ar *= av;
      }
      // four lanes' groups of four steps: neighbours first, then the pairs
      {
        const float oA = __shfl_xor(Ar, 16), oE = __shfl_xor(Er, 16);
        const bool lo = (kq & 1) == 0;
        Er = lo ? fmaf(oA, Er, oE) : fmaf(Ar, oE, Er);
        Ar *= oA;
      }
      {
        const float oA = __shfl_xor(Ar, 32), oE = __shfl_xor(Er, 32);
        const bool lo = (kq & 2) == 0;
        Er = lo ? fmaf(oA, Er, oE) : fmaf(Ar, oE, Er);
        Ar *= oA;
      }
      if (kq == 0) a.agg[((size_t)b * a.nrun + run + m) * D + d] = make_float2(Ar, Er);
    }
  }
}

struct ApplyArgs {
  Problem p;
  int t_lo, n, nrun, last;
  const float *A, *Bv;
  const float2 *agg;
  const float *in;       // states entering the runs (chain_kernel), or null: from `agg` and `init`
  const float *init;     // [B][D] or null
  float *fin;            // [B][D] or null: the state after the chunk's last step
};
// MERGE: 0, or the merge as epilogue (1: exact GeLU, 2: tanh form). A workgroup: 64 channels x 4 runs;
// with `last`, one more row of workgroups writes the Conv1D ring. Every run reads `init` while the last
// one writes `fin`, in no order: the two are never the same memory (launch_forward_f32).
template <int MERGE>
__global__ void __launch_bounds__(NTHREADS) f32_apply_kernel(ApplyArgs a) {
  const Problem &p = a.p;
  const int D = p.D, b = blockIdx.z, d = blockIdx.x * 64 + (threadIdx.x & 63);
  if ((int)blockIdx.y == (a.nrun + 3) / 4) {   // ring slots of the last inputs (older ones are carried over)
    const int slot = threadIdx.x >> 6;
    if (slot > 2 || d >= D) return;
    const long long end = p.pos0 + p.T, npos = end - 1 - ring_slot(end - 1 - slot);
    const size_t o = ((size_t)b * 3 + slot) * D + d;
    float v = 0.f;
    if (npos >= p.pos0) v = ((const float *)p.u)[((size_t)b * p.T + (size_t)(npos - p.pos0)) * D + d];
    else if (p.state_in) v = ((const float *)p.state_in)[o];
    ((float *)p.state_out)[o] = v;
    return;
  }
  const int run = blockIdx.y * 4 + (threadIdx.x >> 6);
  if (run >= a.nrun || d >= D) return;
  const int l0 = run * FT, nt = a.n - l0 < FT ? a.n - l0 : FT;
  const size_t base = ((size_t)b * a.n + l0) * D + d, yb = ((size_t)b * p.T + a.t_lo + l0) * D + d;
  float av[FT], bv[FT], br[MERGE ? FT : 1];
#pragma unroll
  for (int r = 0; r < FT; ++r) {
    const size_t o = (size_t)(r < nt ? r : nt - 1) * D;
    av[r] = a.A[base + o];
    bv[r] = a.Bv[base + o];
    if (MERGE) br[r] = ((const float *)p.branch)[yb + o];
  }
  float h;
  if (a.in) {
    h = a.in[((size_t)b * a.nrun + run) * D + d];
  } else {
    h = a.init ? a.init[(size_t)b * D + d] : 0.f;
    const float2 *ag = a.agg + (size_t)b * a.nrun * D + d;
    for (int k0 = 0; k0 < run; k0 += 8) {
      float2 v[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) v[e] = ag[(size_t)(k0 + e < run ? k0 + e : run - 1) * D];
#pragma unroll
      for (int e = 0; e < 8; ++e)
        if (k0 + e < run) h = fmaf(v[e].x, h, v[e].y);
    }
  }
#pragma unroll
  for (int r = 0; r < FT; ++r) {
    if (r < nt) {
      h = fmaf(av[r], h, bv[r]);   // eq. (4)
      const size_t o = yb + (size_t)r * D;
      if (!MERGE || p.y) ((float *)p.y)[o] = h;
      if (MERGE) ((float *)p.out)[o] = h * gelu<MERGE == 2, false>(br[r]);
    }
  }
  if (run == a.nrun - 1 && a.fin && !a.in) a.fin[(size_t)b * D + d] = h;
}

struct Plan {
  size_t off_A, off_B, off_agg, off_in, off_cell[2], total;
};
Plan plan(int B, int n, int D) {
  const size_t nrun = (size_t)(n + FT - 1) / FT;
  Plan q;
  size_t off = 256;
  for (int k = 0; k < 2; ++k) {
    q.off_cell[k] = off;
    off += align256((size_t)B * D * 4);
  }
  q.off_A = off; off += align256((size_t)B * n * D * 4);
  q.off_B = off; off += align256((size_t)B * n * D * 4);
  q.off_agg = off; off += align256((size_t)B * nrun * D * 8);
  q.off_in = off; off += nrun > MAX_DIRECT ? align256((size_t)B * nrun * D * 4) : 0;
  q.total = off;
  return q;
}
size_t lds_bytes(int bs, int rt) { return ((size_t)rt * FT * (bs + 4) + (size_t)2 * bs * WS) * sizeof(float); }
// (eight column tiles per wave, the weight tile in LDS)
bool block_ok(int bs) { return bs % 16 == 0 && bs <= 512 && lds_bytes(bs, 1) <= 160 * 1024; }
template <int MAXT, int RT>
hipError_t launch_coeff(const CoeffArgs &c, hipStream_t s) {
  const size_t lds = lds_bytes(c.p.bs, RT);
  hipError_t e;
  if (lds > 48 * 1024 && (e = pass::big_lds(f32_coeff_kernel<MAXT, RT>, (int)lds)) != hipSuccess) return e;
  hipLaunchKernelGGL((f32_coeff_kernel<MAXT, RT>), dim3(c.p.nb, (c.nrun + RT - 1) / RT, c.p.B), dim3(NTHREADS), lds, s, c);
  return hipGetLastError();
}
// steps of a chunk of the time axis that `bytes` hold (a multiple of FT unless the whole sequence fits)
int chunk_that_fits(int B, int T, int D, size_t bytes) {
  if (plan(B, T, D).total <= bytes) return T;
  int lo = 0, hi = T / FT;   // in runs
  while (lo < hi) {
    const int mid = (lo + hi + 1) / 2;
    if (plan(B, mid * FT, D).total <= bytes) lo = mid;
    else hi = mid - 1;
  }
  return lo * FT;
}

}  // namespace

size_t forward_f32_ws_bytes(int B, int T, int D) {
  // (the cap is the general kernels', whose scratch has one state: the second cell comes out of the pieces)
  const size_t most = 256 + align256((size_t)4 * B * D) + ((size_t)128 << 20), all = plan(B, T, D).total;
  return all < most ? all : most;
}
bool forward_f32_supported(const Problem &p, bool bf) {
  const uintptr_t all = (uintptr_t)p.W_a | (uintptr_t)p.W_x;
  return !bf && !p.reset && block_ok(p.bs) && p.T > GT && p.B <= 65535 && all % 16 == 0 && p.ws && (uintptr_t)p.ws % 256 == 0 &&
         chunk_that_fits(p.B, p.T, p.D, p.ws_bytes) >= FT && (p.T + FT - 1) / FT <= 65535;
}

hipError_t launch_forward_f32(const Problem &p, hipStream_t s) {
  const int n = chunk_that_fits(p.B, p.T, p.D, p.ws_bytes);
  const Plan q = plan(p.B, n, p.D);
  char *ws = (char *)p.ws;
  hipError_t e;
  // The state in front of a piece lies in one of two cells of the scratch, the one behind it in the other
  // or, after the last piece, in hT: what a launch reads is never what it writes. h0 may be the same
  // array as hT, so the first piece's coefficient pass copies it into a cell.
  float *cell[2] = {(float *)(ws + q.off_cell[0]), (float *)(ws + q.off_cell[1])};
  for (int t_lo = 0, k = 0; t_lo < p.T; t_lo += n, k ^= 1) {
    CoeffArgs c;
    c.p = p;
    c.t_lo = t_lo;
    c.n = p.T - t_lo < n ? p.T - t_lo : n;
    c.nrun = (c.n + FT - 1) / FT;
    c.A = (float *)(ws + q.off_A); c.Bv = (float *)(ws + q.off_B); c.agg = (float2 *)(ws + q.off_agg);
    c.h0 = t_lo == 0 ? p.h0 : nullptr;
    c.cell = cell[0];
    {
      KernelTimer kt("f32_coeff_kernel", s);
      // four runs per workgroup from two workgroups per CU on
      const bool four = (long long)p.nb * p.B * ((c.nrun + 3) / 4) >= 512;
      e = p.bs <= 64    ? (four ? launch_coeff<1, 4>(c, s) : launch_coeff<1, 1>(c, s))
          : p.bs <= 128 ? (four ? launch_coeff<2, 4>(c, s) : launch_coeff<2, 1>(c, s))
          : p.bs <= 256 ? (four ? launch_coeff<4, 4>(c, s) : launch_coeff<4, 1>(c, s))
                        : launch_coeff<8, 1>(c, s);
      if (e != hipSuccess) return e;
    }
    ApplyArgs y;
    y.p = p;
    y.t_lo = t_lo; y.n = c.n; y.nrun = c.nrun;
    y.last = t_lo + c.n == p.T;
    y.A = c.A; y.Bv = c.Bv; y.agg = c.agg;
    y.init = t_lo > 0 || p.h0 ? cell[k] : nullptr;
    y.fin = y.last ? p.hT : cell[k ^ 1];
    y.in = nullptr;
    if (c.nrun > MAX_DIRECT) {
      float *in = (float *)(ws + q.off_in);
      if ((e = pass::launch_chain_forward(c.agg, y.init, in, y.fin, p.B, p.D, c.nrun, s)) != hipSuccess) return e;
      y.in = in;
    }
    {
      KernelTimer kt("f32_apply_kernel", s);
      const dim3 grid((unsigned)(p.D + 63) / 64, (unsigned)((c.nrun + 3) / 4 + (y.last && p.state_out ? 1 : 0)), p.B);
      if (p.merge == 0) hipLaunchKernelGGL(f32_apply_kernel<0>, grid, dim3(NTHREADS), 0, s, y);
      else if (p.merge == 1) hipLaunchKernelGGL(f32_apply_kernel<1>, grid, dim3(NTHREADS), 0, s, y);
      else hipLaunchKernelGGL(f32_apply_kernel<2>, grid, dim3(NTHREADS), 0, s, y);
      if ((e = hipGetLastError()) != hipSuccess) return e;
    }
  }
  return hipSuccess;
}

}  // namespace rglru
