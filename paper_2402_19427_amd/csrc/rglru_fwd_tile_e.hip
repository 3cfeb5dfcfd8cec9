// Instances of the forward in tiles of 32 steps for blocks of 7 and 8 waves: short sequences.
#include "rglru_fwd_tile.h"

namespace rglru {
namespace fused {

Instance find_fwd_short_instance(int nct, int var) {
  switch (nct) {
    case 7: return fwd_pick<7, 1, 4, 4, 1, 4>(var);
    case 8: return fwd_pick<8, 1, 4, 4, 1, 4>(var);
    default: return {nullptr, 0, 0, 0, 0};
  }
}

}  // namespace fused
}  // namespace rglru
