// Instances of the complex-gated forward walks (rglru_cg_tile_fwd.h), by the number of 32-channel tiles of a block.
#include "rglru_cg_tile_fwd.h"

namespace rglru {
namespace cgt {

template <int NCT>
static CgInstance instance() {
  return {(const void *)cg_tile_kernel<NCT, M_AGG>, (const void *)cg_tile_kernel<NCT, M_BAGG>, (const void *)cg_tile_kernel<NCT, M_Y>, nullptr, NCT};
}
CgInstance cg_instance_fwd(int nct) { return nct == 3 ? instance<3>() : instance<4>(); }

}  // namespace cgt
}  // namespace rglru
