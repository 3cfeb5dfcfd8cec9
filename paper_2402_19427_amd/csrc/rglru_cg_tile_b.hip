// Instances of the complex-gated backward walk (rglru_cg_tile_bwd.h), by the number of 32-channel tiles of a block.
#include "rglru_cg_tile_bwd.h"

namespace rglru {
namespace cgt {

CgInstance cg_instance_bwd(int nct, bool any) {
  CgInstance in = cg_instance_fwd(nct, any);
  in.bwd = any ? cg_instance_bwd_any(nct) : nct == 3 ? (const void *)cg_bwd_tile_kernel<3, 4> : (const void *)cg_bwd_tile_kernel<4, 4>;
  return in;
}

}  // namespace cgt
}  // namespace rglru
