// Weight gradients of the kernels in tiles (layouts: rglru_wgrad.h).
#include "rglru_wgrad_tile.h"

#include <algorithm>

namespace rglru {
using namespace wgrad;

namespace {

struct Shape {
  int njt, nkt, n;   // row and column tiles of a block; 32-column blocks of a tile
};
// all columns of a block up to 256 in one tile, or half of them
Shape shape(int ra, int cb, int parts, bool half) {
  const int blocks = (cb + 31) / 32, whole = (blocks + 7) / 8;
  Shape q;
  q.njt = (ra + 255) / 256;
  q.nkt = half ? 2 * whole : whole;
  q.n = std::max(parts == 1 ? 2 : 4, (blocks + q.nkt - 1) / q.nkt);
  return q;
}
// ns of S slices of `per` stages, nst in all. A compute unit runs one workgroup at a time: a round of them starts, ends and writes its sums in
// 0.9 us + 0.8 per 32 columns and takes 0.23 us + 0.025 per 32 columns for a stage, or all together as long as the operands need,
// 0.08 us for a MB of them and 0.02 for a MB that comes to a workgroup, more where workgroups are fewer than compute units; the final sums
// read 1 MB in 0.16 us (least squares over 7000 calls: 112 - 512 channels, 1 - 16 blocks, 1 - 2048 stages, 1 - 64 slices, tiles of all and of half the
// columns; what it takes is on average 0.6 %, at most 5 %, slower than the best of them). us of the backward, so : with as many slices as a
// fixed start of 12 us per workgroup pays for, and halves from 224 channels on only : with tiles of 256 x 128 and slices of 8 stages and more:
// one block of 208, B 18 T 273 51 : 62 : 50; one of 192, T 4096 97 : 119 : 103; two of 160, B 16 T 59 31 : 41 : 34; 16 of 128, T 512 33 : 38 :
// 35; 10 of 192, T 156 33 : 40 : 35.
// Against the second of these rules at 409 sizes: 3.9 % faster on average, more than 1 % faster at 250 and 1 - 3.4 % slower at 10, the worst of them 10
// and 16 blocks of 208 or 256 with 16 stages (16 of 256: 2 slices 56.4, 4 54.6; forward and backward of B 1 T 357 68.2, 67.4 before).
long long cost(const Shape &q, int nst, int nb, int ra, int cb, int S, int per) {
  const long long tiles = (long long)nb * q.njt * q.nkt, rounds = (tiles * S + 255) / 256, KB = ((long long)nb * ra * cb * S) >> 8;
  const long long all = ((long long)nb * (ra + cb) * nst) >> 4, moved = (tiles * (256 + 32 * q.n) * nst) >> 4;   // KB
  const long long memory = 51 * all + (31 * all + 20 * moved) * 256 * rounds / (tiles * S);
  return rounds * (880 + 760 * q.n) + std::max(rounds * per * (234 + 25 * q.n), memory >> 10) + (168 * KB >> 10);
}
template <int PARTS>
hipError_t launch_n(int n, const WgradArgs &a, hipStream_t s) {
  switch (n) {
    case 4: return launch<PARTS, 4>(a, s);
    case 5: return launch<PARTS, 5>(a, s);
    case 6: return launch<PARTS, 6>(a, s);
  }
  if constexpr (PARTS == 1) return n == 7 ? launch<1, 7>(a, s) : launch<1, 8>(a, s);
  return hipErrorInvalidValue;   // (never: halves, above)
}

}  // namespace

// As many slices as make the time least. Two parts: tiles of half the columns of 112 and 128 channels (a wave has no room for the sums of all), a
// stage takes 0.7 us, a workgroup's start, first loads and partial sums 12 us, 5 MB of partial sums 0.5 us more in the final sums.
int tile_wgrad_slices(int nst, int nb, int ra, int cb, int parts, long long fit) {
  const Shape one = shape(ra, cb, parts, false), two = shape(ra, cb, parts, true), &q = parts == 2 && one.n >= 7 ? two : one;
  const long long tiles = (long long)nb * q.njt * q.nkt, sums = ((long long)nb * ra * cb * 4) >> 10;
  long long best = 1, least = -1;
  for (long long S = 1; S <= 64 && S <= fit && S <= nst; ++S) {
    const int per = (int)((nst + S - 1) / S);
    const long long c = parts == 2 ? ((tiles * S + 255) / 256) * (per + 16) * 7000 + S * sums   // (a stage: 7 MB of sums)
                                   : std::min(cost(one, nst, nb, ra, cb, (int)S, per), cost(two, nst, nb, ra, cb, (int)S, per));
    if (least < 0 || c < least) best = S, least = c;
  }
  return (int)best;
}

hipError_t launch_tile_wgrad(const TileWgrad &w, int parts, hipStream_t s) {
  const Shape one = shape(w.ra, w.cb, parts, false), two = shape(w.ra, w.cb, parts, true);
  const bool half = parts == 2 ? one.n >= 7 : cost(two, w.nst, w.nb, w.ra, w.cb, w.S, w.per) < cost(one, w.nst, w.nb, w.ra, w.cb, w.S, w.per);
  const Shape &q = half ? two : one;
  WgradArgs a;
  a.w = w;
  a.njt = q.njt; a.nkt = q.nkt;
  a.total = (unsigned)w.S * w.nb * q.njt * q.nkt;
  KernelTimer kt("tile_wgrad_kernel", s);
  if (parts == 1 && q.n >= 4) return launch_n<1>(q.n, a, s);
  if (parts == 2) return launch_n<2>(q.n, a, s);
  return launch_small(q.n, a, s);
}

}  // namespace rglru
