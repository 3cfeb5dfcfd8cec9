// What the two families of passes share (rglru_pass.hip: the real layer, rglru_cg_pass.hip: the
// complex-gated one): staging through LDS, transposing reads, the final sums.
#pragma once
#include "rglru_mfma.h"

namespace rglru {
namespace pass {
using namespace mfma;

constexpr int RUN = 64;                 // steps per run
constexpr int PR = 256;                 // rows per workgroup of the products
constexpr unsigned OOB = 0x80000000u;   // buffer offset past every range: loads give 0, stores are dropped

typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
// the same at any address a bf16 tensor may have (global memory takes such accesses; aligned ones cost the same)
typedef u32x4 u32x4_at2 __attribute__((aligned(2)));
typedef u32x2 u32x2_at2 __attribute__((aligned(2)));
typedef unsigned u32_at2 __attribute__((aligned(2)));

// 16 bytes per lane from global memory into 1 KB of LDS at the wave-uniform address dst
__device__ __forceinline__ void lds16(__amdgpu_buffer_rsrc_t rs, unsigned char *dst, unsigned vo, unsigned so) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (__attribute__((address_space(3))) void *)dst, 16, vo, so, 0, 0);
}
__device__ __forceinline__ u32x2 lds_tr(const unsigned char *at) {   // 4 rows x 16 channels -> 4 rows of a channel per lane
  const s16x4 v = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4 *)(at));
  return __builtin_bit_cast(u32x2, v);
}
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buf(const void *base, size_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(uniform_ptr(base), 0, (unsigned)bytes, 0x00020000);
}
// byte offset of a place in LDS
__device__ __forceinline__ unsigned lds_offset(const unsigned char *p) {
  return (unsigned)(uintptr_t)(__attribute__((address_space(3))) const unsigned char *)p;
}
// A buffer descriptor as the four words it is (buf() makes the opaque form of the same).
__device__ __forceinline__ u32x4 buf_words(const void *base, size_t bytes) {
  const u64 v = (u64)uniform_ptr(base);
  return u32x4{(unsigned)v, (unsigned)(v >> 32) & 0xffffu, (unsigned)__builtin_amdgcn_readfirstlane((unsigned)bytes), 0x00020000u};
}
// The same load written out, for kernels that keep it in flight across LDS reads: behind the builtin the compiler
// takes any LDS read for one of what it fetches and waits for all of it there. Whoever reads the data waits with an
// s_waitcnt of its own. (No register is written. The compiler does not count the load: its waits for older or
// younger loads then wait for more than they need, never for less.)
// NT: a stream that passes once through the L2s.
template <bool NT>
__device__ __forceinline__ void lds16(const u32x4 &rs, unsigned dst, unsigned vo, unsigned so) {   // dst: byte offset in LDS
  const unsigned at = __builtin_amdgcn_readfirstlane(dst), off = __builtin_amdgcn_readfirstlane(so);
  // (m0 is named as overwritten, so that nothing moves between a load of the compiler's own and the m0 it set for it. It is a
  // reserved register, of which the compiler notes that it does not keep it across: that is what is meant here. To save it
  // and put it back around each load instead costs up to 5 %, 160 channels with the merge, 40 units, T 512: 24.4 -> 25.7 us.)
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
  if (NT)
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen nt lds" :: "s"(at), "v"(vo), "s"(rs), "s"(off) : "memory", "m0");
  else
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds" :: "s"(at), "v"(vo), "s"(rs), "s"(off) : "memory", "m0");
#pragma clang diagnostic pop
}
// every wave's direct-to-LDS loads have landed (they count as vector-memory loads) and every wave is here
__device__ __forceinline__ void stage_barrier() {
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
}
// row of the A operand behind output row r of a 32-row block: accumulator register r of lane half
// hf is then row 16 hf + r, i.e. a lane owns 16 consecutive rows of one column
__device__ __forceinline__ int perm_row(int j) { return ((j >> 2) & 1) * 16 + (j >> 3) * 4 + (j & 3); }
__device__ __forceinline__ int key_a(int row) { return ((row >> 1) & 1) | (((row >> 4) & 1) << 1); }
__device__ __forceinline__ int key_b(int row) { return (row >> 1) & 3; }
__device__ __forceinline__ unsigned f16_bits(float v) {   // round to nearest
  return (unsigned)__builtin_bit_cast(unsigned short, (_Float16)v);
}
__device__ __forceinline__ unsigned pack_rn(float lo, float hi) { return f16_bits(lo) | (f16_bits(hi) << 16); }
// the same without overflow
__device__ __forceinline__ unsigned pack_sat(float lo, float hi) { return pack_rn(f16_range(lo), f16_range(hi)); }
__device__ __forceinline__ float neg_c_softplus(float lam, float c) {   // log of the fully open decay, eq. (3)
  const float z = -lam;
  return -c * (z > 0.f ? z + log1pf(expf(-z)) : log1pf(expf(z)));
}
// consecutive logical ids on one XCD (ids are dealt round-robin to 8): the workgroups that share
// rows or weights then share an L2
__device__ __forceinline__ unsigned xcd_id() {
  const unsigned per = (gridDim.x + 7) >> 3;
  return (blockIdx.x & 7) * per + (blockIdx.x >> 3);
}

// x = Conv1D(u) for steps [t_lo, t_lo + n) of every sequence as [B][n][D] in half precision, xl (may
// be null): the low part. Finite values past half precision's range stop at its end in xh.
hipError_t launch_conv_rows(const Problem &p, unsigned short *xh, unsigned short *xl, int t_lo, int n, hipStream_t s);

// n bf16 values (a multiple of 8) at any alignment, copied to a 16-byte aligned place
hipError_t launch_realign(const void *src, void *dst, size_t n, hipStream_t s);

// states entering the runs [B][nrun][D] and after the last one (fin, may be null) from the runs' aggregates
hipError_t launch_chain_forward(const float2 *agg, const float *init, float *in, float *fin, int B, int D, int nrun,
                                hipStream_t s);

// The adjoint of the Conv1D (conv_adjoint_kernel): du, and partial sums [B][ceil(T / 256)][5][D]
hipError_t launch_conv_adjoint(const Problem &p, const float *dx, float *part, hipStream_t s);

// Partial sums in a fixed order: dW from S slices of [g][gate][bb] (times sc[2] if sc), rowsA from nA
// rows of nrA vectors of DA channels, rowsC from nC rows of five vectors of D channels; with `edge` (S dx of the
// first and last three rows of every tile, [B][nrt][6][D]) the rows of du that two tiles share
struct FinishArgs {
  const float *partW, *partA, *partC, *sc;
  int S, nA, nrA, DA, nC, D, nb;
  size_t bb;             // elements of one gate matrix of a block (a multiple of 4)
  float *dW[2], *rowsA[4], *rowsC[5];
  const float *edge, *conv_w;
  unsigned short *du;
  int B, T, nrt;
  int rows = PR;               // rows per tile of `edge`
  const uint4 *rmask = nullptr;   // packed sequences: boundary masks per 32 steps (as launch_reset_masks leaves them)
  int nmask = 0;
};
hipError_t launch_finish(const FinishArgs &a, hipStream_t s);

inline size_t al256(size_t n) { return (n + 255) & ~(size_t)255; }
inline unsigned grid8(unsigned total) { return (total + 7) / 8 * 8; }
template <typename K>
inline hipError_t big_lds(K kernel, int bytes) {
  return hipFuncSetAttribute((const void *)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
}

}  // namespace pass
}  // namespace rglru
