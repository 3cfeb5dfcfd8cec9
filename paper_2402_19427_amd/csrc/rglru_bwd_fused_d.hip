// Instances of the backward in tiles, by the number of 32-channel tiles of a block.
#include "rglru_bwd_fused.h"

namespace rglru {
namespace fused {

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
