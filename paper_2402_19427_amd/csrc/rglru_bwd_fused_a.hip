// Instances of the backward in tiles, by the number of 32-channel tiles of a block.
#include "rglru_bwd_fused.h"

namespace rglru {
namespace fused {

Instance find_instance_a(int nct, int var) {
  switch (nct) {
    case 4: return pick<4, 1, 3, 4, 1>(var);
    case 5: return pick<5, 1, 3, 4, 1>(var);
    case 6: return pick<6, 1, 3, 4, 1>(var);
    default: return {nullptr, 0, 0, 0, 0};
  }
}

}  // namespace fused
}  // namespace rglru
