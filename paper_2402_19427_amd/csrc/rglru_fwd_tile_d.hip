// Instances of the forward in tiles, by the number of 32-channel tiles of a block.
#include "rglru_fwd_tile.h"

namespace rglru {
namespace fused {

Instance find_fwd_instance_d(int nct, int var) {
  switch (nct) {
    case 13: return fwd_pick<13, 1, 4, 3, 1, 4>(var);
    case 14: return fwd_pick<14, 1, 4, 3, 1, 4>(var);
    case 15: return fwd_pick<15, 1, 4, 3, 1, 4>(var);
    default: return {nullptr, 0, 0, 0, 0};
  }
}

}  // namespace fused
}  // namespace rglru
