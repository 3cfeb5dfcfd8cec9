// Instances of the backward in tiles, by the number of 32-channel tiles of a block.
#include "rglru_bwd_fused.h"

namespace rglru {
namespace fused {

// Sixteen waves to a compute unit leave 128 registers, and the compiler puts 19 - 34 of them into scratch: the least gain of all
// sizes (passes -> tiles, us, 16 blocks, B 4 T 2048: 416 channels 880 -> 714, 448 916 -> 756, 512 1009 -> 913; B 1 T 300: 136 -> 84,
// 142 -> 91, 150 -> 105), none with few long sequences (see `worth`).
Instance find_instance_d(int nct, int var) {
  switch (nct) {
    case 13: return pick<13, 1, 4, 2, 0>(var);
    case 14: return pick<14, 1, 4, 2, 0>(var);
    case 15: return pick<15, 1, 4, 2, 0>(var);
    case 16: return pick<16, 1, 4, 2, 0>(var);
    default: return {nullptr, 0, 0, 0, 0};
  }
}

}  // namespace fused
}  // namespace rglru
