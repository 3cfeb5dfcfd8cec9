// The forward in tiles (see rglru_fwd_tile.h): dispatch.
#include "rglru_fwd_tile.h"

#include <algorithm>

namespace rglru {
using namespace fused;

namespace {

Instance find_instance(int bs, int var) {
  const int nct = (bs + 31) / 32;
  return nct <= 6 ? find_fwd_instance_a(nct, var) : nct <= 8 ? find_fwd_instance_b(nct, var) : nct <= 12 ? find_fwd_instance_c(nct, var) : find_fwd_instance_d(nct, var);
}
int variant(const Problem &p) { return p.reset ? V_PACKED : p.merge == 2 ? V_MERGE_TANH : p.merge ? V_MERGE : V_PLAIN; }

struct Plan {
  int nct, ntile, G, R;
  size_t nrec, off_w, off_masks, off_rec, total;   // nrec: 16-byte words of records
};
// room: what the plan should keep to. It gives up slices for that, at most half of them; past that it is what it is.
Plan make_plan(int B, int T, int nb, int bs, bool packed, const Instance &in, int ncu, size_t room) {
  Plan q;
  q.nct = (bs + 31) / 32;
  q.ntile = (T + 32 * in.mt - 1) / (32 * in.mt);
  size_t off = 256;   // the status word
  q.off_w = off; off += (size_t)nb * q.nct * q.nct * 2 * 2 * 1024;
  q.off_masks = off; off += packed ? al256((size_t)B * ((T + 31) / 32) * sizeof(uint4)) : 0;
  q.off_rec = off;
  const int full = pick_slices(B * nb, q.ntile, in.per_cu * ncu, FWD_TILE_SLICES);
  const auto with = [&](int G) {
    q.G = G;
    q.R = 8;   // (five times the slices: see the carry records)
    while (q.R < 5 * G) q.R *= 2;
    q.nrec = G > 1 ? (size_t)B * nb * q.R * q.nct * 32 * sizeof(u64) / 16 : 0;
    q.total = q.off_rec + q.nrec * 16;
  };
  with(full);
  while (q.total > room && q.G > (full + 1) / 2) with(q.G - 1);
  if (q.total > room) with(full);
  return q;
}

}  // namespace

namespace {
// the shapes whose kernels wait for each other anyway: their workspace brings a status word
bool shape_ok(int B, int T, int D, int bs) {
  return bs % 16 == 0 && T >= 1 && (size_t)D * 2 * 64 < ((size_t)1 << 31) && (long long)B * ((T + 31) / 32) < ((long long)1 << 30) &&
         (forward_mfma_block(bs) || (D % 256 == 0 && (size_t)B * T * D * 2 < ((size_t)1 << 31)));
}
// Where tiles are the faster forward (us, tiles : before).
// Blocks the fused kernel does not take (through passes before): everywhere. 352 channels B 4 T 2048 165 : 274, B 1 T 16
// 25 : 40; 448 channels B 4 T 2048 227 : 338; 288 channels B 1 T 300 23 : 53. Up to 480 channels, though: at 512 the tiles
// would be faster too (275 : 402), but y as they round it (2-norm error 1.654e-3, 1.652e-3 being that of the exact y in
// bf16; the passes' 1.701e-3) puts dW_a at Lambda = -3 where the exact y does, 4.5e-2 off in one draw of six, and the
// bound held there is 4e-2, which the passes' y meets in the same draws (at most 3.96e-2).
// Blocks it takes, 128 channels: everywhere (B 1 T 16 10 : 15, B 8 T 2048 82 : 146). 144 and up:
// - not up to four tiles (160 channels, T 64: 15.7 : 14.3 and 18.4 : 14.6 with the merge; 256, T 200 with the merge
//   23 : 20), where the workgroups' own start is most of the time and they have no second tile to hide it behind;
// - 176 and 192 without the merge: up to 64 units. Six waves on four SIMDs leave two of these half idle; a chip full of
//   such workgroups loses to the fused kernel's eight (176, B 16 T 512: 77 : 67; B 4 T 512: 30 : 30; 160: 62 : 67);
// - 208 to 256: up to 32 units, where the fused kernel cuts a sequence into more than 8 slices and re-reads weights
//   that it otherwise keeps (256, T 32768 of 10 blocks: 202 : 280, T 777: 20 : 26; but 64 units, B 4 T 1024: 53 : 49);
//   with the merge up to 24 (32 units, B 2 T 4096: 111 : 103; 20 units: 88 : 90).
bool worth(int B, int T, int nb, int bs, int var, const Instance &in) {
  if (!forward_mfma_block(bs) || bs <= 128) return true;
  const bool merge = var == V_MERGE || var == V_MERGE_TANH;
  const long long units = (long long)B * nb;
  if (T <= 4 * 32 * in.mt) return false;
  return bs <= 160 || (bs <= 192 ? merge || units <= 64 : units <= (merge ? 24 : 32));
}
size_t bytes(int B, int T, int nb, int bs, int var, size_t room) {
  const Instance in = find_instance(bs, var);
  if (!in.kernel || !worth(B, T, nb, bs, var, in)) return 0;
  // (a size asked for where no card is visible must do on one: the whole chip's slices are the most there can be)
  return std::max(make_plan(B, T, nb, bs, var == V_PACKED, in, 256, room).total,
                  make_plan(B, T, nb, bs, var == V_PACKED, in, compute_units(), room).total);
}
}  // namespace

size_t forward_tile_ws_bytes(int B, int T, int D, int nb, bool packed, bool merge, size_t room) {
  const int bs = D / nb;
  if (!shape_ok(B, T, D, bs)) return 0;
  if (packed) return bytes(B, T, nb, bs, V_PACKED, room);
  return std::max(bytes(B, T, nb, bs, V_PLAIN, room), merge ? bytes(B, T, nb, bs, V_MERGE, room) : (size_t)0);
}

// By the size the call asks for: the same kernels for a shape, whoever lays the workspace out
bool forward_tile_supported(const Problem &p, bool bf, size_t asked) {
  if (!bf || !p.ws || (uintptr_t)p.ws % 16 != 0 || !shape_ok(p.B, p.T, p.D, p.bs)) return false;
  if (((uintptr_t)p.u | (uintptr_t)p.y | (p.merge ? (uintptr_t)p.out | (uintptr_t)p.branch : 0)) % 16 != 0) return false;
  const size_t need = bytes(p.B, p.T, p.nb, p.bs, variant(p), asked);
  return need && need <= asked && p.ws_bytes >= asked;
}

hipError_t launch_forward_tile(const Problem &p, size_t asked, hipStream_t s) {
  const Instance in = find_instance(p.bs, variant(p));
  const Plan q = make_plan(p.B, p.T, p.nb, p.bs, p.reset, in, compute_units(), asked);
  char *ws = (char *)p.ws;
  hipError_t e;
  if ((e = configure(in)) != hipSuccess) return e;
  uint4 *masks = (uint4 *)(ws + q.off_masks);
  if (p.reset && (e = launch_reset_masks(p.reset, masks, nullptr, p.B, p.T, s)) != hipSuccess) return e;
  u32x4 *wg = (u32x4 *)(ws + q.off_w);
  if ((e = launch_tile_prep(p, q.nct, wg, nullptr, ws, ws + q.off_rec, q.nrec, nullptr, s)) != hipSuccess) return e;
  FwdTileArgs a;
  a.p = p;
  a.G = q.G; a.ntile = q.ntile; a.R = q.R;
  a.total = (unsigned)(p.B * p.nb * q.G);
  a.rec = (u64 *)(ws + q.off_rec);
  a.err = (int *)ws;
  a.wg = wg;
  a.rmask = p.reset ? masks : nullptr;
  a.nmask = (p.T + 31) / 32;
  KernelTimer kt("fwd_tile_kernel", s);
  void *args[] = {&a};
  return hipLaunchKernel(in.kernel, dim3(grid8(a.total)), dim3(in.waves * 64), args, in.lds, s);
}

}  // namespace rglru
