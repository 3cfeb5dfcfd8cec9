// Instances of the backward in tiles, by the number of 32-channel tiles of a block.
#include "rglru_bwd_fused.h"

namespace rglru {
namespace fused {

Instance find_instance_b(int nct, int var) {
  switch (nct) {
    case 7: return var == V_PLAIN || var == V_PACKED ? pick<7, 2, 2, 4, 2>(var) : pick_merge<7, 1, 2, 6, 2>(var);
    case 8: return var == V_PLAIN || var == V_PACKED ? pick<8, 2, 2, 4, 2>(var) : pick_merge<8, 1, 2, 6, 2>(var);
    default: return {nullptr, 0, 0, 0, 0};
  }
}

}  // namespace fused
}  // namespace rglru
