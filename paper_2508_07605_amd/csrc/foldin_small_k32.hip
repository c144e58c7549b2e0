// The one-launch fold-in of small batches at rank 32.
#include "foldin_small.h"

namespace openk {

open_status foldin_small_k32(OPEN_SMALL_ARGS) {
  return launch_small<32, 8, 2, SmallSection<4, false, 32>, SmallSection<4, true, 32, 28, 24, 20, 16, 12, 8, 4>>(
      ctx, "foldin_small_k32", OPEN_SMALL_PASS);
}

}  // namespace openk
