// Instances of the weight gradients' kernel for tiles of 2 and 3 column blocks: few stages.
#include "rglru_wgrad_tile.h"

namespace rglru {

hipError_t wgrad::launch_small(int n, const WgradArgs &a, hipStream_t s) { return n == 2 ? launch<1, 2>(a, s) : launch<1, 3>(a, s); }

}  // namespace rglru
