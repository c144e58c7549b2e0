// Forward and backward pass of the surrogate network over a batch (kernel in mlp_train.hip).
#pragma once
#include "wgrad.h"

namespace openk {

struct MlpBatch {
  int64_t B;               // batch rows
  const int64_t *rows;     // CSR row of batch row b at rows[b] (nullable: row b), or, with
  int use_cursor;          //   use_cursor, at rows[st->cursor * B + b]
  const int64_t *ptr;
  const int32_t *col;
  const float *val;
  int n, k;
  const uint32_t *W1P;     // first-layer weight pairs
  const float *b1, *b2, *b3;
  const uint4 *W2P, *W3P, *W2T, *W3T;  // operands of the layers and of their transposes
  float *out;              // forward only: B x k
  const float *target;     // m x k
  uint16_t *X, *h1, *h2;   // packed operands over pad_rows(B) rows: pad_units(2n), 256, 256 wide
  uint16_t *d1p, *d2p, *d3p;  //   256, 256 and pad_units(k) wide
  float *d1, *d2, *d3;     // output gradients, float32
  double *lpart;           // mlp_batch_loss_parts(B, k) partial sums of the squared errors
  TrainState *st;
};

open_status mlp_batch_launch(open_ctx *ctx, const MlpBatch &p, bool forward_only);
int mlp_batch_loss_parts(const open_ctx *ctx, int64_t B, int k);

}  // namespace openk
