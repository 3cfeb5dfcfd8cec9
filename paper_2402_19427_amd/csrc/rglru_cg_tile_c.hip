// Instances of the complex-gated walks for tensors off the 16-byte grid.
#include "rglru_cg_tile_bwd.h"
#include "rglru_cg_tile_fwd.h"

namespace rglru {
namespace cgt {

CgInstance cg_instance_fwd_any(int nct) { return nct == 3 ? fwd_instance<3, true>() : fwd_instance<4, true>(); }
const void *cg_instance_bwd_any(int nct) { return nct == 3 ? (const void *)cg_bwd_tile_kernel<3, 4 + AT_ANY> : (const void *)cg_bwd_tile_kernel<4, 4 + AT_ANY>; }

}  // namespace cgt
}  // namespace rglru
