// The one-launch fold-in of small batches at ranks 8 and 16, with the lanes per system of
// their classes' default kernels.
#include "foldin_small.h"

namespace openk {

open_status foldin_small_k8(OPEN_SMALL_ARGS) {
  return launch_small<8, 8, 2, SmallSection<4, false, 8>, SmallSection<1, true, 8, 4>>(ctx, "foldin_small_k8",
                                                                                       OPEN_SMALL_PASS);
}
open_status foldin_small_k16(OPEN_SMALL_ARGS) {
  return launch_small<16, 8, 2, SmallSection<4, false, 16>, SmallSection<4, true, 16>,
                      SmallSection<1, true, 12, 8, 4>>(ctx, "foldin_small_k16", OPEN_SMALL_PASS);
}

}  // namespace openk
