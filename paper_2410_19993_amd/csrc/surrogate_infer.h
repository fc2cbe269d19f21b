// One-pass surrogate inference, called by the package's Python front end (surrogate.py); not
// part of the public header, which declares the steps it replaces.
#pragma once

#include <stdint.h>

#include "xbar.h"

#ifdef __cplusplus
extern "C" {
#endif

/* Currents and error estimates as xbar_sg_features, `depth` bfloat16 convolutions (C
 * hidden channels, ReLU after all but the last, 2 output channels; params: each layer's
 * weights [O][C][3][3], then its biases [O], in turn) and xbar_sg_predict give them, in
 * one pass that writes no activation maps.  The last map has the same bits; sums over its
 * rows may differ in rounding.  2 <= depth <= 5, 1 <= C <= XBAR_SG_MAX_CHANNELS, m, n <=
 * XBAR_SG_MAX_LINE.  work: 16-byte aligned device memory of at least
 * xbar_sg_infer_workspace_bytes bytes (-1: a size this call does not take), overlapping
 * nothing else.  I must not overlap G or V; est (NULL: none) must not overlap I. */
int64_t xbar_sg_infer_workspace_bytes(int32_t B, int32_t m, int32_t n, int32_t C, int32_t depth);
xbar_status xbar_sg_infer_bf16(int32_t B, int32_t m, int32_t n, int32_t C, int32_t depth, const double* G,
                               const double* V, const double* r, const float* params, void* work,
                               int64_t work_bytes, double* I, double* est, void* stream);

#ifdef __cplusplus
}
#endif
