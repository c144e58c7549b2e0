// Training pieces shared by the surrogate network and the NCF model: the step state on the
// device and the seeded on-device shuffle (kernels in mlp.hip).
#pragma once
#include "common.h"

namespace openk {

// Optimizer state on the device, so that a recorded training step can be replayed as is:
// t = Adam steps taken, cursor = batch index within the epoch.  The step's first launch reads
// these and sets, for its second one, the bias corrections c1, c2 and tag = t + 1; the second
// launch advances t and cursor, which nothing else in it reads.
struct TrainState {
  int64_t t, cursor;
  float c1, c2;
  int64_t tag;
};
__device__ __forceinline__ void train_state_begin(TrainState *st) {
  st->c1 = (float)(1.0 - pow(0.9, (double)(st->t + 1)));
  st->c2 = (float)(1.0 - pow(0.999, (double)(st->t + 1)));
  st->tag = st->t + 1;
}

open_status dense_train_state_reset(open_ctx *ctx, TrainState *st);
// perm = the seeded order of [0, m) for `epoch` (a Feistel bijection walked along its cycles);
// rewinds the batch cursor
open_status dense_shuffle(open_ctx *ctx, int64_t m, uint64_t seed, int64_t epoch, int64_t *perm, TrainState *st);

}  // namespace openk
