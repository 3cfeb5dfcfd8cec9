// Instances of the complex-gated forward walks (rglru_cg_tile_fwd.h), by the number of 32-channel tiles of a block.
#include "rglru_cg_tile_fwd.h"

namespace rglru {
namespace cgt {

template <int NCT, bool ANY>
static CgInstance instance() {
  return {(const void *)cg_tile_kernel<NCT, M_AGG, ANY>, (const void *)cg_tile_kernel<NCT, M_BAGG, ANY>, (const void *)cg_tile_kernel<NCT, M_Y, ANY>,
          nullptr, NCT};
}
CgInstance cg_instance_fwd(int nct, bool any) {
  return nct == 3 ? any ? instance<3, true>() : instance<3, false>() : any ? instance<4, true>() : instance<4, false>();
}

}  // namespace cgt
}  // namespace rglru
