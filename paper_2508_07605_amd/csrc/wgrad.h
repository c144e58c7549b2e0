// Weight gradients of a training step's dense layers and the optimizer, one launch per step
// (kernels in wgrad.hip).  The forward-and-backward kernel of a network leaves, per layer, the
// output gradients and the inputs as bfloat16 MFMA operands along the batch:
// [batch / 8][units][8], the eight values of one unit contiguous (16 bytes), rows past the batch
// and units past the layer's width zero.
#pragma once
#include "dense.h"

namespace openk {

// batch rows of the packed operands are padded to this many
constexpr int kBatchPad = 32;
__host__ __device__ constexpr int64_t pad_rows(int64_t B) { return (B + kBatchPad - 1) / kBatchPad * kBatchPad; }
__host__ __device__ constexpr int pad_units(int u) { return (u + 31) / 32 * 32; }

struct WgradLayer {
  const uint16_t *A, *X;     // packed output gradients (pad_units(M) wide) and inputs (pad_units(N))
  const float *Af;           // output gradients in float32 (batch x M): the bias gradient
  int M, N;                  // outputs, inputs
  int64_t w;                 // the layer's weights (M x N) in the parameter vector, its M biases after them
  // bfloat16 copies refreshed with the weights (each nullable): P in the operand order of W
  // (M x N), PT of its transpose, pairs as first-layer weight pairs (N = 2n inputs)
  uint16_t *P, *PT, *pairs;
  // filled by wgrad_step: batch slices of kc rows, output tiles per block, blocks of the launch
  int S, kc, nt, blocks;
};

// Embedding gradients of the NCF model, whose batch rows pair each of G applications with each of
// n settings: dX (batch x 64) holds the gradients of [e ; s], summed per application over the
// settings and per setting over the applications, each in order.
struct WgradEmb {
  int G = 0, n = 0;          // G = 0: no embeddings
  int64_t m = 0;             // applications of the model
  const float *dX = nullptr;
  const int64_t *apps = nullptr;  // the batch's applications
  const int64_t *mark = nullptr;  // step tag of each application's last batch
  int64_t e = 0, s = 0;      // offsets of E (m x 32) and S (n x 32) in the parameter vector
};

// floats of the partial bias sums for every 32 outputs of a layer: slices, four sums each
constexpr int kWgBiasPart = 256 * 4 * 32;

struct WgradStep {
  WgradLayer l[3];
  WgradEmb emb;
  int64_t B;                 // batch rows
  float *w, *g, *m, *v;      // parameters, gradient, Adam moments
  float lr;
  TrainState *st;
  const double *lpart;       // partial sums of the squared errors, their number, the mean's divisor
  int nlpart;
  int64_t ltotal;
  float *bias;               // nullable: the bias gradients' slices are summed into this by a launch of
                             // their own (kWgBiasPart floats for every 32 outputs)
  double *loss_d;            // the batch loss (each nullable; loss_steps indexed by the Adam step)
  float *loss_f, *loss_steps;
};

// adam: update the parameters (and their copies) and the step state; otherwise write the
// gradient to g.
open_status wgrad_step(open_ctx *ctx, const char *name, WgradStep p, bool adam);

}  // namespace openk
