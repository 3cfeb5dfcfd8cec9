// Instances of the complex-gated backward walk (rglru_cg_tile_bwd.h), by the number of 32-channel tiles of a block.
#include "rglru_cg_tile_bwd.h"

namespace rglru {
namespace cgt {

template <int NCT>
static const void *kernel(bool any) {
  return any ? (const void *)cg_bwd_tile_kernel<NCT, 4, true> : (const void *)cg_bwd_tile_kernel<NCT, 4, false>;
}
CgInstance cg_instance_bwd(int nct, bool any) {
  CgInstance in = cg_instance_fwd(nct, any);
  in.bwd = nct == 3 ? kernel<3>(any) : kernel<4>(any);
  return in;
}

}  // namespace cgt
}  // namespace rglru
