// Instances of the forward in tiles, by the number of 32-channel tiles of a block.
#include "rglru_fwd_tile.h"

namespace rglru {
namespace fused {

Instance find_fwd_instance_a(int nct, int var) {
  switch (nct) {
    case 4: return fwd_pick<4, 1, 4, 4, 1, 4>(var);
    case 5: return fwd_pick<5, 1, 4, 4, 1, 4>(var);
    case 6: return fwd_pick<6, 1, 4, 4, 1, 4>(var);
    default: return {nullptr, 0, 0, 0, 0};
  }
}

}  // namespace fused
}  // namespace rglru
