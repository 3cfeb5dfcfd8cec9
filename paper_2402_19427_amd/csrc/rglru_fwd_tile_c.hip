// Instances of the forward in tiles, by the number of 32-channel tiles of a block.
#include "rglru_fwd_tile.h"

namespace rglru {
namespace fused {

Instance find_fwd_instance_c(int nct, int var) {
  switch (nct) {
    case 9: return fwd_pick<9, 1, 3, 4, 1, 3>(var);
    case 10: return fwd_pick<10, 1, 3, 4, 1, 3>(var);
    case 11: return fwd_pick<11, 1, 3, 4, 1, 3>(var);
    case 12: return fwd_pick<12, 1, 3, 4, 1, 3>(var);
    default: return {nullptr, 0, 0, 0, 0};
  }
}

}  // namespace fused
}  // namespace rglru
