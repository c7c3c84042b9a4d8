// First kernel of a single call (best shifts, jump values): the caller's point
// into internal order, its byte copy, and, when the call needs no objective
// sum (no cutoff row), the walk state.
#pragma once

#include <hip/hip_runtime.h>

#include <climits>

#include "chap_internal.h"

namespace chap {

// The state fields that do not depend on the point.
__device__ __forceinline__ void reset_state(WalkState* st, int64_t iters, int32_t tenure, float wc) {
  st->k = 0;
  st->iters = iters;
  st->tenure = tenure;
  st->sel_k = -1;
  st->mv_j = -1;
  st->dV = 0ull;
  st->choice = 0ull;
  // single passes: the compact copy holds the cutoff weight as a count of
  // half weights only when it is an integer below 2^16 (the rows are
  // checked where the copy is written)
  st->compact_rows = (wc == floorf(wc) && wc >= 0.0f && wc < 65535.0f) ? 1 : 0;
  st->aff_ok = 0;
  st->pass_skip = 0;
  st->aff_iters = 0;
}

// State of a single pass without a cutoff row (one thread).
__device__ __forceinline__ void single_state(WalkState* st, const SingleInit& I) {
  const float wc = *I.cutoff_w;
  reset_state(st, 1, 0, wc);
  st->inf_V = LLONG_MAX;
  st->inf_k = -2;
  st->f = 0.0;
  st->fbest = HUGE_VAL;
  st->bc = 0.0;
  st->rc = 0.0;
  st->V = 0;
  st->wc = wc;
  st->has_best = 0;
  st->copy_best = 0;
  st->cut_active = 0;
  st->obj_integral = I.obj_integral;
}

// Byte copy of value v of column q; a value that does not fit flags the call.
__device__ __forceinline__ void stage_byte(double v, int q, int8_t* xc, WalkState* st, uint32_t epoch) {
  const bool fits = v == floor(v) && v >= -128.0 && v <= 127.0;
  xc[q] = fits ? (int8_t)v : (int8_t)0;
  if (!fits) st->x_misfit = epoch;  // every writer stores the same value
}

}  // namespace chap
