// Instances of the backward in tiles, by the number of 32-channel tiles of a block.
#include "rglru_bwd_fused.h"

namespace rglru {
namespace fused {

Instance find_instance_c(int nct, int var) {
  switch (nct) {
    case 9: return pick<9, 1, 3, 4, 1>(var);
    case 10: return pick<10, 1, 3, 4, 1>(var);
    case 11: return pick<11, 1, 3, 4, 1>(var);
    case 12: return pick<12, 1, 3, 4, 1>(var);
    default: return {nullptr, 0, 0, 0, 0};
  }
}

}  // namespace fused
}  // namespace rglru
