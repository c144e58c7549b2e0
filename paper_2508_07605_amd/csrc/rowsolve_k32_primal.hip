// Ridge-solve kernels of size-class groups, each with its compiled configurations
// (lanes per system, waves per block, waves per SIMD); variant 0 is the default.
#include "rowsolve.h"

namespace openk {

OPEN_GROUP(g_k32_primal) {
  return launch_variant<32, 32, false, cfg(4, 8, 2), cfg(4, 4, 1)>(choice, "ridge_k32_primal", kPrimalLo, kPrimalHi, OPEN_TIER_PASS, X,
                       status, m);
}

}  // namespace openk
