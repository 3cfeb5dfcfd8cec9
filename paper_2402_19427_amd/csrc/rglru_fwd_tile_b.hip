// Instances of the forward in tiles, by the number of 32-channel tiles of a block.
#include "rglru_fwd_tile.h"

namespace rglru {
namespace fused {

Instance find_fwd_instance_b(int nct, int var) {
  switch (nct) {   // (64 steps: half the weights' way from L2 per step; 256 channels, T 8192 of 10 blocks: 94 us with 32, 74)
    case 7: return fwd_pick<7, 2, 2, 4, 2, 2>(var);
    case 8: return fwd_pick<8, 2, 2, 4, 2, 2>(var);
    default: return {nullptr, 0, 0, 0, 0};
  }
}

}  // namespace fused
}  // namespace rglru
