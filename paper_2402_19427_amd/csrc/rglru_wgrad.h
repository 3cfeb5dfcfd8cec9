// Weight gradients from what the kernels in tiles leave (rglru_bwd_fused.h): dW = sum over the steps of
// (gate adjoint) x (input), both in stages of 32 steps, a kilobyte per 16 channels:
//   [stage][block][group of 16 channels][K-step of 16][half of it][channel][8 steps], 16 bits each,
// which a lane that owns 16 steps of a channel writes as two 16-byte pieces and a matrix fragment reads as it lies.
#pragma once
#include "rglru_pass.h"

namespace rglru {

struct TileWgrad {
  const unsigned short *A[2], *B[2];   // adjoints [..][ra channels], inputs [..][cb channels]; with two parts: bf16 high, low
  float *part;                         // [S][nb][ra][cb] sums of a slice of the stages
  int nst, S, per;                     // stages; slices of them, stages per slice
  int nb, ra, cb;                      // blocks; channels of a block on either side (multiples of 16)
};
// the number of slices the chip is filled best with, at most `fit`
int tile_wgrad_slices(int nst, int nb, int ra, int cb, int parts, long long fit);
// parts 1: half precision, one product; 2: bf16 high and low parts, three products
hipError_t launch_tile_wgrad(const TileWgrad &w, int parts, hipStream_t s);

}  // namespace rglru
