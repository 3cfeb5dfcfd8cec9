// Instances of the complex-gated forward walks (rglru_cg_tile_fwd.h), by the number of 32-channel tiles of a block.
#include "rglru_cg_tile_fwd.h"

namespace rglru {
namespace cgt {

CgInstance cg_instance_fwd(int nct, bool any) {
  return any ? cg_instance_fwd_any(nct) : nct == 3 ? fwd_instance<3, false>() : fwd_instance<4, false>();
}

}  // namespace cgt
}  // namespace rglru
