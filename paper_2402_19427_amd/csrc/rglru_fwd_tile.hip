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
// The shapes whose products run in half precision whatever kernel takes them: the fused kernel's, and without document boundaries
// the passes'. What the general kernels serve (packed rows of the other blocks, sequences of 2^31 bytes and more, 2^32 at 256 channels) they
// serve in plain fp32 arithmetic: hT of packed rows of 352 channels is 2e-7 off, 7e-5 in tiles.
bool shape_ok(int B, int T, int D, int bs, bool packed) {
  if (bs % 16 != 0 || T < 1 || (size_t)D * 2 * 64 >= ((size_t)1 << 31) || (long long)B * ((T + 31) / 32) >= ((long long)1 << 30)) return false;
  if (forward_mfma_block(bs)) return (size_t)T * D * 2 < ((size_t)1 << (bs == 256 ? 32 : 31));
  return !packed && D % 256 == 0 && (size_t)B * T * D * 2 < ((size_t)1 << 31);
}
// Where tiles are the faster forward (us, tiles : before).
// Blocks the fused kernel does not take (through passes before): everywhere. 352 channels B 4 T 2048 165 : 274, B 1 T 16
// 25 : 40; 448 channels B 4 T 2048 227 : 338; 288 channels B 1 T 300 23 : 53. Up to 480 channels, though: whether 512
// may follow (275 : 402) is an open question of precision. The tiles' y is the more exact one (2-norm error 1.654e-3,
// 1.652e-3 being that of the exact y in bf16; the passes' 1.701e-3), but the bound held on dW_a at Lambda = -3, 4e-2, is below
// what the storage rounding of y supports: the exact y in bf16 is 4.5e-2 off in one draw of six, where the passes' y is not.
// Blocks it takes, 128 channels: everywhere (B 1 T 16 10 : 15, B 8 T 2048 82 : 146). 144 and up:
// - up to four tiles (of 32 steps, up to 192 channels): see worth_short. Tiles of 64 steps (from 208 channels on): see choose.
// What else decides is how often a workgroup of either kernel goes round (a round is a tile of each of its slices) and what the
// preparation costs: the tiles' converts both gates' weights of all blocks, the fused kernel's one gate's, 1 - 5 us more by the
// number of blocks. `half`: the tiles go round at most half as often.
// - 144 and 160: everywhere else (160, 8 - 512 units, T 129 - 2048: 0.63 - 1.02 of the fused kernel's time); with the merge
//   and more than 24 blocks where `half` (32 blocks, 64 units: T 257 - 300 30 : 28, T 400 32 : 35), or many units and more than 8 tiles
//   (32 blocks, 128 units: T 129 30 : 29, T 700 69 : 73).
// - 176 and 192, six waves on four SIMDs, two of which stay half idle: a chip full of such workgroups loses to the fused
//   kernel's eight. Without the merge up to 64 units, at 176 up to 48 (64 units: T 1024 48 : 46, T 129 18 : 20); with it up to 64
//   and 48 and beyond where `half` (176, 128 units: T 300 47 : 43, T 2048 198 : 212) or, at 192, from 129 units on (240 : 178 at
//   B 16 T 1024). Many blocks lose everywhere (24 blocks, 96 units: T 512 69 : 57; 32 blocks, 32 units, T 2048 58 : 48) but at 192 in
//   a single short sequence (32 blocks, T 257 22 : 25).
// - 208 to 256: up to 32 units, where the fused kernel cuts a sequence into more than 8 slices and re-reads weights that it otherwise
//   keeps (256, T 32768 of 10 blocks: 202 : 280; 16 blocks, B 1 T 1024 23 : 27, B 2 T 512 22 : 26; 64 units, B 4 T 1024: 53 : 49); with
//   the merge up to 24 (32 units, B 2 T 4096: 111 : 103). Not, with more than 12 blocks (16 at 256 channels without the merge), where the fused
//   kernel goes round no oftener (240, 16 blocks, T 300: 25 : 22 with the merge, 20 : 19 without), nor with more than 24 (240, 32 blocks,
//   T 2048 69 : 52). At 240 and 256 the gain is smaller: with the merge, many blocks or a long sequence take `half` (256, 24 blocks, T 2048
//   71 : 63; B 2 of 10 blocks, T 4096 93 : 89, T 6000 123 : 124), and 29 - 32 units of more than 8 blocks lose in between (256, 16 blocks: B 2 T 1400
//   43 : 45, T 2048 54 : 52, T 4096 90 : 85, T 8192 159 : 156, T 12000 226 : 228; 8 blocks, B 4 T 2048 50 : 52).
// Short sequences, up to 128 steps of 144 - 192 channels and 256 of 208 - 256 (160, 16 blocks: B 1 T 20 11.2 : 16.3, T 128 12.8 : 16.9, with the
// merge 14.8 : 16.8, B 16 T 128 25 : 30; 192, 10 blocks, B 16 T 128 25 : 32): up to 256 units. What the tiles give away there is the preparation
// of both gates' weights, in proportion to the blocks, so the line is the size of those weights (7200 calls, 1 - 128 blocks):
// - 192 and 256 channels, where the fused kernel itself takes longest: 20 and 16 MB (256: 64 blocks B 2 T 32 20.2 : 19.8, 96 blocks B 1 T 32
//   23.1 : 20.9).
// - one tile: 6.5 MB (176, 64 blocks T 9 15.8 : 15.1; 208, 40 blocks 15.5 : 15.1; 240, 32 blocks 16.0 : 15.5, 48 blocks 18.1 : 16.5); with the merge
//   or boundaries, which cost the fused kernel more, 10 (208, 64 blocks with the merge 19.3 : 18.6).
// - more tiles of one sequence: 6.5 MB (208, 48 blocks T 64 17.3 : 16.2), with boundaries 10, with the merge 5 (176, 40 blocks T 33 16.5 : 15.6; 240,
//   24 blocks T 64 17.6 : 16.1; 208, 32 blocks T 128 18.2 : 16.5); from five tiles on 10 and, with boundaries, 16 MB (208, 64 blocks T 256: with the
//   merge 28.6 : 26.0, with boundaries 27.7 : 28.6).
// - of several sequences: 16 MB (240, 64 blocks B 2 T 64 21.5 : 23.6), with the merge of more than 160 channels 10 (240, 96 blocks B 2 T 64 32.1 : 30.7).
// Past 128 units the second tile loses where a unit's workgroups share a compute unit and the fused kernel has one each: more than 16 blocks
// from 208 channels on (24 blocks, B 8 T 64, 208: 20.0 : 18.9), at 240 any (16 blocks, B 16 T 64 21.1 : 19.5), at 256 more than 24 (40 blocks, B 4
// T 64 23.9 : 22.7), at 176, past 160 units, more than 24 (48 blocks, B 4 T 128 27.7 : 26.2); five tiles from 113 units on (240, 16 blocks,
// B 8 T 160 29.9 : 28.6). Not with the merge, whose epilogue the fused kernel pays more for.
bool worth_short(int B, int T, int nb, int bs, int var) {
  const bool merge = var == V_MERGE || var == V_MERGE_TANH, plain = var == V_PLAIN;
  const int nct = (bs + 31) / 32, n = (T + 31) / 32;
  const long long units = (long long)B * nb, KB = (long long)nb * nct * nct * 4;
  if (units > 256) return false;
  const long long most = bs == 192 ? 20000 : bs == 256 ? 16384 : n == 1 ? (plain ? 6450 : 10000) : B > 1 ? (merge && bs > 160 ? 10000 : 16384)
                         : n <= 4 ? (plain ? 6450 : merge ? 5000 : 10000) : (plain || merge ? 10000 : 16384);
  if (KB > most) return false;
  if (merge || n == 1) return true;
  if (bs >= 208 && units > 112 && units <= 128 && n == 5) return false;
  if (bs >= 208 && units > 128) return nb <= (bs == 256 ? 24 : bs >= 240 ? 0 : 16);
  return bs != 176 || units <= 160 || nb <= 24;
}
bool worth(int B, int T, int nb, int bs, int var, const Instance &in) {
  if (!forward_mfma_block(bs) || bs <= 128) return true;
  const bool merge = var == V_MERGE || var == V_MERGE_TANH;
  const int steps = 32 * in.mt;
  const long long units = (long long)B * nb;
  if (T <= 4 * steps) return in.mt == 1 && worth_short(B, T, nb, bs, var);
  // (for 256 compute units on either side: the same rule where no card is visible)
  const auto rounds = [&](int step, int workgroups, int most) {
    const int n = (T + step - 1) / step, G = pick_slices(B * nb, n, workgroups, most);
    return (n + G - 1) / G;
  };
  const int own = rounds(steps, in.per_cu * 256, FWD_TILE_SLICES), fused = rounds(32, 256, FWD_MAX_SLICES);
  const bool half = 2 * own <= fused;
  if (bs <= 160) return !merge || nb <= 24 || half || (units > 64 && T > 256);
  if (bs <= 192) {
    if (nb > 24) return bs == 192 && units <= 32 && T <= 320;
    if (units <= 48) return true;
    if (nb > 16) return false;
    if (units <= 64) return bs == 192 || T <= 256;
    return merge && (half || (bs == 192 && units > 128));
  }
  // More units of 256 channels, up to 16 blocks (call times, tiles : fused): where the fused kernel goes in more than 4 slices, too (40 units T 300
  // 20 : 27, T 1024 38 : 43, T 4096 107 : 112; 50 units T 2048 72 : 77), with the merge only up to 640 steps (T 300 25 : 29, T 600 38 : 40, T 1024
  // 61 : 56); without it also in two slices that leave a fifth of the chip idle (100 units T 600 52 : 56, T 2048 139 : 142) and in short
  // sequences (80 units T 300 30 : 35, T 600 45 : 46, T 1024 63 : 61; 128 units T 300 37 : 39, T 2048 159 : 149). With the merge and one workgroup per
  // unit up to 216 of them, where the fused kernel's epilogue costs it most (130 units T 257 57 : 60, T 300 59 : 65, T 1024 163 : 184; 208 units T 300 61 : 66,
  // T 2048 333 : 354; 256 units 368 : 368). Boundaries cost the fused kernel more than the tiles: as without them (40 units T 257 20 : 28, T 2048
  // 67 : 71; 80 units T 640 48 : 51; 100 units T 2048 and 4096 0.95 - 0.97 of its time; 128 units T 300 40 : 43, T 640 62 : 64).
  if (bs == 256 && units > 32 && nb <= 16) {
    if (merge) return (units <= 51 && T <= 640) || (units > 128 && units <= 216);
    return units <= 51 || (units > 85 && units <= 100) || (units <= 128 && T <= 640);
  }
  if (units > (merge ? 24 : 32) || nb > 24) return false;
  if (nb > (bs == 256 && !merge ? 16 : 12) && own >= fused) return false;
  if (bs < 240) return true;
  if (merge) return half || units <= 16 || (nb <= 16 && T < 2048);
  return units <= 28 || nb <= 8 || units * T < 65536 || units * T >= 300000;
}
// The instance a call runs on; kernel null: not in tiles. Blocks of 208 - 256 channels have tiles of 64 steps, whose weights take half the way
// from L2 per step, and of 32, of which there are twice as many to fill the chip. What decides is how often a workgroup goes round. us, tiles of
// 32 : before (fused up to T 256, where the tiles' start is most of the time and those of 64 are no gain):
// - up to T 256, one round: B 1, 10 blocks of 256 T 20 13.3 : 19.7, T 128 14.7 : 20.7, T 256 15.1 : 21.8, with the merge 17.4 : 22.4; B 11 T 128
//   24 : 29; 16 blocks B 16 T 64 24.7 : 25.9; 10 of 208 B 1 T 256 15.6 : 18.9.
// - two rounds with the merge, or of three slices and more: B 5 T 256 16 blocks 30 : 33, with the merge 35 : 36, B 16 T 100 10 blocks 29 : 31;
//   two slices 33 : 31 (B 11 T 100, 16 blocks), 35 : 33 with B 16. Not from three rounds on (10 blocks, B 16 T 256 44 : 43).
// - past T 256, where tiles are the faster forward at all: in one round of a workgroup per compute unit (B 1, 10 blocks, T 777 with the merge
//   20.8 : 24.9 in tiles of 64; T 500 17.2 : 17.9), or in one round where those of 64 take two (B 2 T 777 25.5 : 29.7; but B 2 T 500, one round of
//   either, 23 : 20). Not where the plan gives up slices for its room, from 26 tiles on, and the round is none (8 blocks of 256, T 800
//   15.2 : 17.3 in tiles of 64, T 900 in 25 slices 19.9 : 17.4, T 1024 19.5 : 17.7, T 900 with the merge 21.8 : 20.7; one block of 208, which
//   leaves the room to two sequences, T 928 B 1 17.9 : 15.4, B 2 13.8 : 15.5).
Instance choose(int B, int T, int nb, int bs, int var, size_t room) {
  const Instance none = {nullptr, 0, 0, 0, 0}, in = find_instance(bs, var);
  if (!in.kernel) return none;
  if (in.mt == 1 || bs < 208 || bs > 256) return worth(B, T, nb, bs, var, in) ? in : none;
  const Instance one = find_fwd_short_instance(in.waves, var);
  const int n1 = (T + 31) / 32, n2 = (T + 63) / 64, G1 = pick_slices(B * nb, n1, one.per_cu * 256, FWD_TILE_SLICES),
            G2 = pick_slices(B * nb, n2, in.per_cu * 256, FWD_TILE_SLICES), r1 = (n1 + G1 - 1) / G1, r2 = (n2 + G2 - 1) / G2;
  if (T <= 256) return worth_short(B, T, nb, bs, var) && (r1 == 1 || (r1 == 2 && (var == V_MERGE || var == V_MERGE_TANH || G1 >= 3))) ? one : none;
  if (!worth(B, T, nb, bs, var, in)) return none;
  if (r1 > 1 || ((long long)B * nb * n1 > 256 && r2 == 1)) return in;
  return make_plan(B, T, nb, bs, var == V_PACKED, one, 256, room).G == G1 ? one : in;
}
// Of short calls the whole plan is asked for: the second gate's weights and up to some MB of records (10 blocks of 256, B 1 T 256 2.6 MB of weights
// and 1.3 of records; 16 blocks, B 16 T 64 8.4 and 4.2).
constexpr int SHORT = 256;
size_t bytes(int B, int T, int nb, int bs, int var, size_t room) {
  const Instance in = choose(B, T, nb, bs, var, room);
  if (!in.kernel) return 0;
  if (T <= SHORT) room = ~(size_t)0;
  // (a size asked for where no card is visible must do on one: the whole chip's slices are the most there can be)
  return std::max(make_plan(B, T, nb, bs, var == V_PACKED, in, 256, room).total,
                  make_plan(B, T, nb, bs, var == V_PACKED, in, compute_units(), room).total);
}
}  // namespace

size_t forward_tile_ws_bytes(int B, int T, int D, int nb, bool packed, bool merge, size_t room) {
  const int bs = D / nb;
  if (!shape_ok(B, T, D, bs, packed)) return 0;
  if (packed) return bytes(B, T, nb, bs, V_PACKED, room);
  return std::max(bytes(B, T, nb, bs, V_PLAIN, room), merge ? bytes(B, T, nb, bs, V_MERGE, room) : (size_t)0);
}

// By the size the call asks for: the same kernels for a shape, whoever lays the workspace out
bool forward_tile_supported(const Problem &p, bool bf, size_t asked) {
  if (!bf || !p.ws || (uintptr_t)p.ws % 16 != 0 || !shape_ok(p.B, p.T, p.D, p.bs, p.reset != nullptr)) return false;
  if (((uintptr_t)p.u | (uintptr_t)p.y | (p.merge ? (uintptr_t)p.out | (uintptr_t)p.branch : 0)) % 16 != 0) return false;
  const size_t need = bytes(p.B, p.T, p.nb, p.bs, variant(p), asked);
  return need && need <= asked && p.ws_bytes >= asked;
}

hipError_t launch_forward_tile(const Problem &p, size_t asked, hipStream_t s) {
  const Instance in = choose(p.B, p.T, p.nb, p.bs, variant(p), asked);
  const Plan q = make_plan(p.B, p.T, p.nb, p.bs, p.reset, in, compute_units(), p.T <= SHORT ? ~(size_t)0 : asked);
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
