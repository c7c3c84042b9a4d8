// Best-shift pass kernels for gfx950 (wave64).
//
// One pass computes, for every variable j, the best shift (Eq. 1 of section
// 3.1 "Best Shift Moves") at the current point: the flip for a binary
// variable, and for every other variable the result of Algorithm 1 ("Best
// Shift via Sort-Scan-Argmax"). Columns are routed by class and length:
//
//   k_group        columns with at most 64 stored entries: 4, 8, 16, 32 or 64
//                  lanes per column, one stored entry each. Binaries: the flip
//                  score, summed across the group. Others: every candidate
//                  position (bounds and breakpoints, incumbent excluded) is
//                  scored directly from the penalty definition written in
//                  breakpoint form, each lane scoring its own entry's
//                  candidates against all entries. Longer binaries: one
//                  wavefront per column.
//   k_narrow_pack  longer integer columns with <= 64 values, packed whole into
//                  workgroups: the sort of Algorithm 1 becomes a counting sort
//                  into 64 LDS bins per column, the scan a wavefront prefix
//                  sum, the argmax a wavefront reduction over candidate bins.
//   k_narrow_chunk the same for long columns split over many workgroups by
//                  row range; k_narrow_combine adds the partial bins.
//   k_sort_block   one workgroup per longer general column: LDS bitonic sort of the
//                  breakpoints, block scan, block argmax.
//   k_sort_long    general columns beyond the LDS capacity: the same steps in
//                  global scratch memory.
//
// On all-integer instances with 0 < eps <= 1/2 the narrow columns are
// row-block staged instead:
//   k_stage_rows   one workgroup per slice of an 8192-row block held in LDS:
//                  each staged entry becomes an 8-byte breakpoint record, and
//                  single-entry columns are scored on the spot.
//   k_stage_score  one launch for the rest: packs of columns (counting sort
//                  of their records into LDS bins), groups of short columns
//                  of one degree (one lane per column) and the chunks of long
//                  columns, as interleaved units of the grid.
//
// Phase 1 of Algorithm 1 emits, per row, the accumulators beta/alpha and up to
// two triplets. Here the two triplets of an a_ij > 0 row, (t,-1,0) and
// (t,+1,d), are merged into one entry "d applies strictly after t, and t is a
// candidate"; an a_ij < 0 row gives "d applies from t on". The score at a
// candidate position p is beta + (sum of entries applying at p) +
// alpha [p > xbar], the value Algorithm 1's scan produces at that position.
// Only finite positions inside [l, u] other than xbar are candidates, ties go
// to the smallest position, and (xbar, 0) is returned when no candidate scores
// above zero.

#include <algorithm>
#include <cfloat>
#include <cmath>
#include <type_traits>

#include "chap_internal.h"
#include "move_best.h"
#include "narrow_finish.h"

namespace chap {
namespace {


// Row accessors: the walk's RowState array, or its compact GatherRow copy.
struct FullRows {
  gptr<const RowState> p;
  __device__ __forceinline__ RowState operator[](int i) const { return gload(p, i); }
};

struct CompactRows {
  gptr<const GatherRow> p;
  __device__ __forceinline__ RowState operator[](int i) const {
    const GatherRow g = gload(p, i);
    RowState o;
    o.r = (double)g.r;
    o.w0 = (float)g.w0;
    o.w1 = (g.w1 == kNoTwin) ? -1.0f : (float)g.w1;
    return o;
  }
};

// Either of the two, as the walk state says (single passes with caller weights).
struct DualRows {
  gptr<const RowState> p;
  gptr<const GatherRow> g;
  int32_t use_g;
  __device__ __forceinline__ RowState operator[](int i) const {
    if (use_g) return CompactRows{g}[i];
    return gload(p, i);
  }
};

template <typename Rows>
__device__ __forceinline__ Rows rows_of(const WalkCtx& C);
template <>
__device__ __forceinline__ DualRows rows_of<DualRows>(const WalkCtx& C) {
  return DualRows{gmem((const RowState*)C.rs), gmem((const GatherRow*)C.grow), C.st->compact_rows};
}
template <>
__device__ __forceinline__ FullRows rows_of<FullRows>(const WalkCtx& C) {
  return FullRows{gmem((const RowState*)C.rs)};
}
template <>
__device__ __forceinline__ CompactRows rows_of<CompactRows>(const WalkCtx& C) {
  return CompactRows{gmem((const GatherRow*)C.grow)};
}

// Whether staged records carry the weights (exact in 16 bits): always with
// the compact row copy, as the walk state says for single passes, never with
// full rows (the scoring kernel then reads them from the row states).
template <typename Rows>
__device__ __forceinline__ bool stage_weights(const WalkCtx& C);
template <>
__device__ __forceinline__ bool stage_weights<CompactRows>(const WalkCtx&) {
  return true;
}
template <>
__device__ __forceinline__ bool stage_weights<DualRows>(const WalkCtx& C) {
  return C.st->compact_rows != 0;
}
template <>
__device__ __forceinline__ bool stage_weights<FullRows>(const WalkCtx&) {
  return false;
}

// Whether the rows are read from the walk's compact copy (whose words then
// have the staged LDS row format, weights included).
__device__ __forceinline__ bool compact_source(const CompactRows&) { return true; }
__device__ __forceinline__ bool compact_source(const DualRows& r) { return r.use_g != 0; }
__device__ __forceinline__ bool compact_source(const FullRows&) { return false; }

__device__ __forceinline__ double breakpoint(double xb, double r, double a, double eps, bool is_int) {
  double t = xb + (eps - r) / a;
  if (is_int) t = (a > 0.0) ? floor(t) : ceil(t);
  return t;
}

// Penalty p_ij of section 3.1 "Scoring Functions" for a residual r -> r2.
__device__ __forceinline__ double penalty(double r, double r2, double w, double eps) {
  const bool v = r > eps, v2 = r2 > eps;
  if (!v && v2) return -w;
  if (v && !v2) return w;
  if (v && v2) {
    if (r2 < r) return 0.5 * w;
    if (r2 > r) return -0.5 * w;
  }
  return 0.0;
}

// Phase 1 of Algorithm 1 for one normalised row entry (a, r, w) of a
// non-binary column at xbar. Updates beta/alpha, returns the merged entry.
struct BkEntry {
  double t;
  double delta;
  int marker;  // -1: applies from t on, +1: applies after t
  bool has;
};

__device__ __forceinline__ BkEntry phase1(double xb, double r, double a, double w, double eps, bool is_int,
                                          double& beta, double& alpha) {
  BkEntry e;
  e.t = breakpoint(xb, r, a, eps, is_int);
  e.has = true;
  if (a < 0.0) {
    e.marker = -1;
    if (xb < e.t) {
      beta -= 0.5 * w;
      alpha += w;
      e.delta = 0.5 * w;
    } else if (xb > e.t) {
      beta -= w;
      e.delta = w;
    } else {
      beta -= w;
      alpha += w;
      e.delta = 0.0;
      e.has = false;
    }
  } else {
    e.marker = 1;
    if (xb > e.t) {
      beta += w;
      alpha -= w;
      e.delta = -0.5 * w;
    } else if (xb < e.t) {
      e.delta = -w;
    } else {
      alpha -= w;
      e.delta = 0.0;
      e.has = false;
    }
  }
  return e;
}

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, kWave);
  return v;
}

__device__ __forceinline__ unsigned long long wave_or(unsigned long long v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v |= __shfl_xor(v, o, kWave);
  return v;
}


// ---------------------------------------------------------------------------
// k_group: a group of lanes per column (at most kGroupMax stored entries).
//
// Bound: latency. The columns are short, so the kernel is one chain of loads
// (row index and coefficient of the lane's entry, its row state) followed by a
// few hundred instructions; a lane per entry makes every load of a column one
// request, starts all chains at once and needs one division per lane where a
// lane per column needs one per entry. On the general instance of 100k
// columns it replaces three kernels on forked streams (one lane per column of
// at most 8 normalised entries 25-30 us, one wavefront per longer binary
// 5-15 us, a bitonic sort across a wavefront per longer general column 30 us,
// and the events between them).
// ---------------------------------------------------------------------------

// One normalised entry in breakpoint form: satisfied at p when p <= t (a > 0)
// or p >= t (a < 0), kept as p' <= t' with the sign of both flipped for a < 0;
// what it adds to the score where it is satisfied, and where it is not on
// either side of xbar.
struct GroupTerm {
  double t;
  float sat;      // satisfied
  float left;     // not satisfied, p < xbar
  float right;    // not satisfied, p > xbar
  uint32_t flip;  // sign bit to flip
};

// A wavefront's columns: the terms of a column side by side in entry order
// (a row, then its twin; the cutoff row last), its candidate positions
// likewise with the bounds after them. Both lists are dense, so that columns
// with few equality rows cost neither terms nor candidates for the twins that
// they do not have.
constexpr int kGroupTerms = 144;  // most of any width: 64 / G columns of 2 G + 1
constexpr int kGroupCands = 176;  // 64 / G columns of 2 G + 3
struct GroupSmem {
  GroupTerm term[4][kGroupTerms];
  double cand[4][kGroupCands];
};

__device__ __forceinline__ double flip_sign(double v, uint32_t flip) {
  const unsigned long long u = __double_as_longlong(v);
  return __longlong_as_double(u ^ ((unsigned long long)flip << 32));
}

__device__ __forceinline__ GroupTerm group_term(double t, bool ap, float w, double xb) {
  GroupTerm g;
  const bool s0 = ap ? (xb <= t) : (xb >= t);
  g.flip = ap ? 0u : 0x80000000u;
  g.t = flip_sign(t, g.flip);
  g.sat = s0 ? 0.0f : w;
  g.left = s0 ? -w : (ap ? 0.5f * w : -0.5f * w);
  g.right = s0 ? -w : (ap ? -0.5f * w : 0.5f * w);
  return g;
}

// Half of a weight below 2^-125 may be no float: a wavefront that meets one
// (kTiny) forms the halves of all its terms in FP64, from the whole weights that
// they hold. Only calls with the caller's weights (kCaller) look for one: the
// weights of a walk are counts. FP64 terms for every wavefront cost 4 % of a walk
// on 100k columns, looking 0.5 %.
constexpr float kTinyWeight = 0x1p-125f;
__device__ __forceinline__ bool tiny_weight(float w) { return w > 0.0f && w < kTinyWeight; }

template <bool kTiny>
__device__ __forceinline__ double term_at(const GroupTerm& g, double p, bool right) {
  const float sat = g.sat, left = g.left, rgt = g.right;  // values, not addresses, to select from
  const bool in = flip_sign(p, g.flip) <= g.t;
  if constexpr (kTiny) {
    if (in || sat == 0.0f) return (double)(in ? sat : left);
    return (double)sat * ((g.flip != 0) == right ? 0.5 : -0.5);
  }
  const float off = right ? rgt : left;
  return (double)(in ? sat : off);
}

// Orders the LDS writes and reads of one wavefront.
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Column q by the G lanes of its group; row, a: this lane's stored entry (row
// < 0: none; a column's entries fill its first lanes). Groups without a column
// (in = false) take part in the exchanges and write nothing. Returns the
// column's kept score on the group's first lane, 0 on the others. kCaller: the
// weights are the caller's (see kTinyWeight).
template <int G, bool kFlip, bool kCaller, typename Rows>
__device__ __forceinline__ double score_group(const WalkCtx& C, const Rows& rs, const WalkState* st, int q, bool in,
                                            int row, double a, GroupSmem& S) {
  const DevProblem& P = C.P;
  const int tid = threadIdx.x, g = tid & (G - 1);
  const double eps = P.eps;
  const bool has = row >= 0;
  const double xb = gmem((const double*)C.x)[q];
  const double c = st->cut_active ? gmem(P.obj)[q] : 0.0;
  RowState r{0.0, 0.0f, -1.0f};
  if (has) r = rs[row];
  if constexpr (kFlip) {
    const double xn = 1.0 - xb, d = xn - xb;
    double s = 0.0;
    if (has) {
      const double r2 = r.r + a * d;
      s = penalty(r.r, r2, (double)r.w0, eps);
      if (r.w1 >= 0.0f) s += penalty(-r.r, -r2, (double)r.w1, eps);
    }
    if (g == 0 && c != 0.0) s += penalty(st->rc, st->rc + c * d, (double)st->wc, eps);
#pragma unroll
    for (int o = 1; o < G; o <<= 1) s += __shfl_xor(s, o, kWave);
    if (g != 0 || !in) return 0.0;
    write_result(gmem(C.xhat), gmem(C.s), q, true, s, xn, xb);
    return fmax(s, 0.0);
  }
  const bool isint = gmem(P.is_int)[q] != 0;
  const double l = gmem(P.lb)[q], u = gmem(P.ub)[q];
  const bool twin = has && r.w1 >= 0.0f;
  // the column's terms and candidates: slots by the entries and twins before
  const int lane = tid & (kWave - 1), col = lane / G;
  const unsigned long long mine = (G < kWave ? (1ull << (G & 63)) - 1ull : ~0ull) << (lane & ~(G - 1) & 63);
  const unsigned long long bt = __ballot(twin) & mine;
  const int deg = __popcll(__ballot(has) & mine), tw = __popcll(bt);
  const int slot = g + __popcll(bt & ((1ull << lane) - 1ull));
  const int nt = deg + tw + (c != 0.0 ? 1 : 0), nc = nt + 2;
  GroupTerm* term = S.term[tid >> 6] + col * (2 * G + 1);
  double* cand = S.cand[tid >> 6] + col * (2 * G + 3);
  if (has) {
    const double t = breakpoint(xb, r.r, a, eps, isint);
    term[slot] = group_term(t, a > 0.0, r.w0, xb);
    cand[slot] = t;
  }
  if (twin) {
    const double t = breakpoint(xb, -r.r, -a, eps, isint);
    term[slot + 1] = group_term(t, !(a > 0.0), r.w1, xb);
    cand[slot + 1] = t;
  }
  if (g == 0) {
    if (c != 0.0) {
      const double t = breakpoint(xb, st->rc, c, eps, isint);
      term[nt - 1] = group_term(t, c > 0.0, st->wc, xb);
      cand[nt - 1] = t;
    }
    cand[nc - 2] = l;
    cand[nc - 1] = u;
  }
  wave_sync();
  // candidates g, g + G (and g + 2 G where a column of the wavefront has that
  // many) against every term of the column
  constexpr int kC = 3;
  const bool third = __any(nc > 2 * G);
  double p[kC], v[kC];
  bool right[kC];
#pragma unroll
  for (int k = 0; k < kC; ++k) {
    p[k] = (g + k * G < nc) ? cand[g + k * G] : HUGE_VAL;
    right[k] = p[k] > xb;
    v[k] = 0.0;
  }
  bool tiny = false;
  if constexpr (kCaller)
    tiny = __any((has && (tiny_weight(r.w0) || tiny_weight(r.w1))) || (c != 0.0 && tiny_weight(st->wc)));
  if (kCaller && tiny) {
    for (int e = 0; e < nt; ++e) {
      const GroupTerm t = term[e];
#pragma unroll
      for (int k = 0; k < kC; ++k) v[k] += term_at<true>(t, p[k], right[k]);
    }
  } else if (third) {
    for (int e = 0; e < nt; ++e) {
      const GroupTerm t = term[e];
#pragma unroll
      for (int k = 0; k < kC; ++k) v[k] += term_at<false>(t, p[k], right[k]);
    }
  } else {
    for (int e = 0; e < nt; ++e) {
      const GroupTerm t = term[e];
      v[0] += term_at<false>(t, p[0], right[0]);
      v[1] += term_at<false>(t, p[1], right[1]);
    }
  }
  double best = -HUGE_VAL, at = HUGE_VAL;
#pragma unroll
  for (int k = 0; k < kC; ++k) {
    if (!(p[k] >= l && p[k] <= u) || p[k] == xb || !isfinite(p[k])) continue;
    if (v[k] > best || (v[k] == best && p[k] < at)) {
      best = v[k];
      at = p[k];
    }
  }
#pragma unroll
  for (int o = 1; o < G; o <<= 1) {
    const double ov = __shfl_xor(best, o, kWave), op = __shfl_xor(at, o, kWave);
    if (ov > best || (ov == best && op < at)) {
      best = ov;
      at = op;
    }
  }
  if (g != 0 || !in) return 0.0;
  write_result(gmem(C.xhat), gmem(C.s), q, best > -HUGE_VAL, best, at, xb);
  return fmax(best, 0.0);
}

// What a workgroup of the group kernel hands to the move selection: the
// column of this lane and its kept score (0: none).
struct GroupScore {
  double s = 0.0;
  int q = -1;
  int j = 0;           // its original index
  bool tabu = false;
};

// The move selection's data of column q, loaded ahead of the scoring.
__device__ __forceinline__ void group_ids(const WalkCtx& C, const WalkState* st, bool first, int q, GroupScore& o) {
  if (C.group_rec == 0 || !first) return;
  o.j = gmem(C.P.perm)[q];
  o.tabu = st->k <= (int64_t)gmem((const int32_t*)C.tabu)[q];
}

template <int G, bool kFlip, bool kCaller, typename Rows>
__device__ __forceinline__ GroupScore group_block(const WalkCtx& C, const Rows& rs, const WalkState* st, int cls,
                                                  int b, GroupSmem& S) {
  const PassPlan& L = C.plan;
  const int64_t t = L.grp_off[cls] + (int64_t)b * 256 + (int)threadIdx.x;
  const int row = gmem(L.grp_row)[t];
  const double a = gmem(L.grp_val)[t];
  const int end = L.grp_col[cls + 1];
  const int qt = L.grp_col[cls] + b * (256 / G) + (int)threadIdx.x / G;
  const int q = min(qt, end - 1);
  GroupScore o;
  group_ids(C, st, ((int)threadIdx.x & (G - 1)) == 0, q, o);
  o.s = score_group<G, kFlip, kCaller, Rows>(C, rs, st, q, qt < end, row, a, S);
  o.q = qt < end ? q : -1;
  return o;
}

// A binary column of any length by one wavefront.
template <typename Rows>
__device__ __forceinline__ double flip_wave(const WalkCtx& C, const Rows& rs, const WalkState* st, int q) {
  const DevProblem& P = C.P;
  const int lane = threadIdx.x & (kWave - 1);
  const double eps = P.eps;
  const double xb = gmem((const double*)C.x)[q];
  const double xn = 1.0 - xb;
  const double d = xn - xb;
  double s = 0.0;
  const int beg = gmem(P.col_ptr)[q], end = gmem(P.col_ptr)[q + 1];
  for (int e = beg + lane; e < end; e += kWave) {
    const RowState r = rs[gmem(P.col_row)[e]];
    const double r2 = r.r + gmem(P.col_val)[e] * d;
    s += penalty(r.r, r2, (double)r.w0, eps);
    if (r.w1 >= 0.0f) s += penalty(-r.r, -r2, (double)r.w1, eps);
  }
  if (lane == 0 && st->cut_active) {
    const double c = gmem(P.obj)[q];
    if (c != 0.0) s += penalty(st->rc, st->rc + c * d, (double)st->wc, eps);
  }
  s = wave_sum(s);
  if (lane != 0) return 0.0;
  write_result(gmem(C.xhat), gmem(C.s), q, true, s, xn, xb);
  return fmax(s, 0.0);
}

// Workgroup b of the lane-group columns.
template <bool kCaller, typename Rows>
__device__ __forceinline__ GroupScore group_task(const WalkCtx& C, const Rows& rs, const WalkState* st, int b,
                                                 GroupSmem& S) {
  const int32_t* blk = C.plan.grp_blk;
  int c = 0;
#pragma unroll
  for (int k = 1; k <= kGroupClasses; ++k)
    if (b >= blk[k]) c = k;
  b -= blk[c];
  switch (c) {
    case 0: return group_block<4, true, kCaller, Rows>(C, rs, st, 0, b, S);
    case 1: return group_block<8, true, kCaller, Rows>(C, rs, st, 1, b, S);
    case 2: return group_block<16, true, kCaller, Rows>(C, rs, st, 2, b, S);
    case 3: return group_block<32, true, kCaller, Rows>(C, rs, st, 3, b, S);
    case 4: return group_block<64, true, kCaller, Rows>(C, rs, st, 4, b, S);
    case 5: return group_block<4, false, kCaller, Rows>(C, rs, st, 5, b, S);
    case 6: return group_block<8, false, kCaller, Rows>(C, rs, st, 6, b, S);
    case 7: return group_block<16, false, kCaller, Rows>(C, rs, st, 7, b, S);
    case 8: return group_block<32, false, kCaller, Rows>(C, rs, st, 8, b, S);
    case 9: return group_block<64, false, kCaller, Rows>(C, rs, st, 9, b, S);
    default: {
      GroupScore o;
      const int q = C.plan.grp_col[kGroupClasses] + b * 4 + (int)(threadIdx.x >> 6);
      if (q < C.plan.grp_col[kGroupClasses + 1]) {
        group_ids(C, st, (threadIdx.x & 63) == 0, q, o);
        o.s = flip_wave(C, rs, st, q);
        o.q = q;
      }
      return o;
    }
  }
}

// Eight wavefronts a SIMD (60 registers): 107.6 us for 64 walks of 28k columns,
// 113.3 with seven; alone on a walk of 100k columns 10.5 either way.
template <bool kCaller, typename Rows>
__global__ __launch_bounds__(256, 8) void k_group(const WalkCtx* __restrict__ walks, const int32_t* __restrict__ off,
                                               int32_t nw) {
  int lb;
  const int w_ = block_walk(off, nw, lb);
  if (w_ < 0) return;
  const WalkCtx& C = walks[w_];
  const WalkState* st = C.st;
  const bool rec = C.group_rec > 0;
  const bool active = st->k < st->iters && !st->pass_skip;
  if (rec && lb == 0 && threadIdx.x == 0) snapshot(C.st, active);
  if (!active) return;
  __shared__ GroupSmem S;
  const Rows rs = rows_of<Rows>(C);
  const GroupScore o = group_task<kCaller, Rows>(C, rs, st, lb, S);
  if (!rec) return;
  // the walk's move selection: this workgroup's best moves, and the pending
  // copy of a new incumbent (flagged by the previous iteration, before this
  // iteration's move changes x)
  if (st->copy_best && o.q >= 0) gmem(C.best_x)[o.q] = gmem((const double*)C.x)[o.q];
  block_record_one<4>(o.s, o.j, o.q, o.tabu, C.best + lb);
}

// The lane-group columns of an affected-rescoring iteration (b of nb
// workgroups): the listed ones, a wavefront each, or all of them. With `rec`
// their best moves go there.
template <typename Rows>
__device__ __forceinline__ void aff_group_body(const WalkCtx& C, const AffRun* run, int b, int nb, GroupSmem& S,
                                               MoveRecord* rec) {
  const WalkState* st = C.st;
  if (st->k >= st->iters) return;
  const Rows rs = rows_of<Rows>(C);
  const int count = run->n_s;
  BestPair best;
  if (count < 0) {
    for (int t = b; t < C.plan.grp_blk[kGroupClasses]; t += nb) {
      const GroupScore o = group_task<false, Rows>(C, rs, st, t, S);
      if (rec && o.s > 0.0) best.offer(o.s, o.j, o.q, o.tabu);
    }
  } else {
    const int lane = threadIdx.x & (kWave - 1);
    const int n_flip = C.plan.grp_col[kGroupWidths];
    for (int i = b * 4 + (int)(threadIdx.x >> 6); i < count; i += nb * 4) {
      const int q = __builtin_amdgcn_readfirstlane(run->slist[i]);
      const int beg = C.P.col_ptr[q], deg = C.P.col_ptr[q + 1] - beg;
      GroupScore o;
      if (rec) group_ids(C, st, lane == 0, q, o);
      int row = -1;
      double a = 1.0;
      if (lane < deg) {
        row = gmem(C.P.col_row)[beg + lane];
        a = gmem(C.P.col_val)[beg + lane];
      }
      if (q < n_flip)
        o.s = score_group<kWave, true, false, Rows>(C, rs, st, q, true, row, a, S);
      else
        o.s = score_group<kWave, false, false, Rows>(C, rs, st, q, true, row, a, S);
      if (rec && o.s > 0.0) best.offer(o.s, o.j, q, o.tabu);
    }
  }
  if (rec) block_record<4>(best, rec);
}

// ---------------------------------------------------------------------------
// Narrow integer columns: counting sort into LDS bins.
// ---------------------------------------------------------------------------

// Adds one normalised entry of column (l, u, W) at xbar into the bins.
__device__ __forceinline__ void narrow_entry(double xb, double r, double a, double w, double eps, double l,
                                             double u, int W, double* bins, double& beta, double& alpha,
                                             unsigned long long& cand) {
  const BkEntry e = phase1(xb, r, a, w, eps, true, beta, alpha);
  if (!e.has) return;
  if (e.t < l) {
    beta += e.delta;
    return;
  }
  if (e.t > u) return;
  const int k = (int)(e.t - l);
  cand |= 1ull << k;
  if (e.marker < 0)
    atomicAdd(&bins[k], e.delta);
  else if (k + 1 < W)
    atomicAdd(&bins[k + 1], e.delta);
}


// One workgroup per pack of whole narrow columns (consecutive internal
// columns, at most kPackCols of them, about kPackEntries entries). The 256
// threads stream the pack's concatenated CSC entries as one flat range; each
// entry finds its column by binary search over the column starts and adds
// into that column's 64 LDS bins, beta, alpha and candidate mask. Each
// wavefront then scans and reduces a quarter of the pack's columns.
template <typename Rows>
__global__ __launch_bounds__(256) void k_narrow_pack(const WalkCtx* __restrict__ walks,
                                                     const int32_t* __restrict__ off, int32_t nw) {
  int lb;
  const int w_ = block_walk(off, nw, lb);
  if (w_ < 0) return;
  const WalkCtx& C = walks[w_];
  const DevProblem& P = C.P;
  const double* x = C.x;
  const Rows rs = rows_of<Rows>(C);
  const WalkState* st = C.st;
  double* xhat = C.xhat;
  double* sc = C.s;
  if (st->k >= st->iters || st->pass_skip) return;
  __shared__ double bins[kPackCols][kNarrowBins];
  __shared__ double sbeta[kPackCols], salpha[kPackCols], sxb[kPackCols], sl[kPackCols], su[kPackCols];
  __shared__ unsigned long long scand[kPackCols];
  __shared__ int sstart[kPackCols + 1];
  const int tid = threadIdx.x;
  const PackTask T = C.plan.packs[lb];
  const int nc = T.q_end - T.q_begin;
  if (tid < nc) {
    const int q = T.q_begin + tid;
    sxb[tid] = x[q];
    sl[tid] = P.lb[q];
    su[tid] = P.ub[q];
    sstart[tid] = P.col_ptr[q];
    sbeta[tid] = 0.0;
    salpha[tid] = 0.0;
    scand[tid] = 0ull;
  }
  if (tid == 0) sstart[nc] = P.col_ptr[T.q_end];
  for (int i = tid; i < nc * kNarrowBins; i += blockDim.x) bins[i / kNarrowBins][i % kNarrowBins] = 0.0;
  __syncthreads();
  const double eps = P.eps;
  const int e0 = sstart[0], e1 = sstart[nc];
  // Each thread takes kPackRun consecutive entries per step (the loads of a
  // run are issued together); runs mostly stay inside one column, so beta,
  // alpha and the candidate mask are summed in registers and added to LDS
  // once per column change instead of once per entry.
  constexpr int kPackRun = 4;
  const int step = blockDim.x * kPackRun;
  for (int base = e0 + tid * kPackRun; base < e1; base += step) {
    const int cnt = min(kPackRun, e1 - base);
    int row[kPackRun];
    double a[kPackRun];
    RowState r[kPackRun];
#pragma unroll
    for (int u = 0; u < kPackRun; ++u)
      if (u < cnt) {
        row[u] = P.col_row[base + u];
        a[u] = P.col_val[base + u];
      }
#pragma unroll
    for (int u = 0; u < kPackRun; ++u)
      if (u < cnt) r[u] = rs[row[u]];
    int lo = 0, hi = nc - 1;  // largest slot with sstart[slot] <= base
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if (sstart[mid] <= base)
        lo = mid;
      else
        hi = mid - 1;
    }
    int slot = lo;
    double db = 0.0, da = 0.0;
    unsigned long long dc = 0ull;
#pragma unroll
    for (int u = 0; u < kPackRun; ++u) {
      if (u >= cnt) break;
      while (base + u >= sstart[slot + 1]) {
        if (db != 0.0) atomicAdd(&sbeta[slot], db);
        if (da != 0.0) atomicAdd(&salpha[slot], da);
        if (dc) atomicOr(&scand[slot], dc);
        db = 0.0;
        da = 0.0;
        dc = 0ull;
        ++slot;
      }
      const double xb = sxb[slot], l = sl[slot], u2 = su[slot];
      const int W = (int)(u2 - l) + 1;
      narrow_entry(xb, r[u].r, a[u], (double)r[u].w0, eps, l, u2, W, bins[slot], db, da, dc);
      if (r[u].w1 >= 0.0f) narrow_entry(xb, -r[u].r, -a[u], (double)r[u].w1, eps, l, u2, W, bins[slot], db, da, dc);
    }
    if (db != 0.0) atomicAdd(&sbeta[slot], db);
    if (da != 0.0) atomicAdd(&salpha[slot], da);
    if (dc) atomicOr(&scand[slot], dc);
  }
  if (tid < nc && st->cut_active) {
    const double c = P.obj[T.q_begin + tid];
    if (c != 0.0) {
      const double xb = sxb[tid], l = sl[tid], u = su[tid];
      double db = 0.0, da = 0.0;
      unsigned long long dc = 0ull;
      narrow_entry(xb, st->rc, c, (double)st->wc, eps, l, u, (int)(u - l) + 1, bins[tid], db, da, dc);
      if (db != 0.0) atomicAdd(&sbeta[tid], db);
      if (da != 0.0) atomicAdd(&salpha[tid], da);
      if (dc) atomicOr(&scand[tid], dc);
    }
  }
  __syncthreads();
  const int lane = tid & (kWave - 1);
  for (int slot = tid >> 6; slot < nc; slot += (int)(blockDim.x >> 6)) {
    const double l = sl[slot], xb = sxb[slot];
    const int W = (int)(su[slot] - l) + 1;
    bool found;
    double best, bestp;
    narrow_finish(bins[slot][lane], sbeta[slot], salpha[slot], scand[slot], xb, l, W, lane, found, best, bestp);
    if (lane == 0) write_result(xhat, sc, T.q_begin + slot, found, best, bestp, xb);
  }
}

// Offset of the cutoff row's breakpoint from xbar, clamped like the records.
__device__ __forceinline__ int cutoff_offset(double xb, const WalkState* st, double c, double eps) {
  const double t = breakpoint(xb, st->rc, c, eps, true);
  return (int)fmin(fmax(t - xb, -(double)kStageClamp), (double)kStageClamp);
}

// The cases of phase1() in offset form (coefficient sign ap, breakpoint t =
// xbar + d): 3 [a > 0] + sign(d) + 1, and two for a breakpoint above every
// narrow column (d > 63), whose delta never applies and which is no
// candidate: 6 for a > 0, 7 for a < 0. Tables of 4-bit fields: the
// coefficients, in half weights, of what the row adds to beta, alpha and (from
// its breakpoint on, or after it where kCaseAfter is 1) delta.
constexpr uint32_t pack8(int c0, int c1, int c2, int c3, int c4, int c5, int c6, int c7) {
  return (uint32_t)(c0 & 15) | (uint32_t)(c1 & 15) << 4 | (uint32_t)(c2 & 15) << 8 | (uint32_t)(c3 & 15) << 12 |
         (uint32_t)(c4 & 15) << 16 | (uint32_t)(c5 & 15) << 20 | (uint32_t)(c6 & 15) << 24 |
         (uint32_t)(c7 & 15) << 28;
}
constexpr uint32_t kCoefBeta = pack8(-2, -2, -1, 2, 0, 0, 0, -1);
constexpr uint32_t kCoefAlpha = pack8(0, 2, 2, -2, -2, 0, 0, 2);
constexpr uint32_t kCoefDelta = pack8(2, 0, 1, -1, 0, -2, 0, 0);
constexpr uint32_t kCaseAfter = pack8(0, 0, 0, 1, 1, 1, 1, 0);
constexpr int kCaseNone = 24;  // four times case 6
// Field `at` (four times the case) of a table: one bit-field extract.
__device__ __forceinline__ int row_coef(uint32_t table, int at) { return __builtin_amdgcn_sbfe((int)table, at, 4); }
// Four times the case of a row with offset d in [-64, 64] (64: above).
__device__ __forceinline__ int row_case(bool ap, int d) {
  const int at = (ap ? 16 : 4) + 4 * min(max(d, -1), 1);
  return d >= kStageClamp ? (ap ? 24 : 28) : at;
}

// Offsets of a row with integer residual r and coefficient a != 0, clamped to
// [-64, 64]: *d0 of the row, *d1 of its negated twin. With A = |a|, f =
// floor(-r / A) and c = ceil(-r / A), they are f and c for a > 0 and -f and -c
// for a < 0. kSmall (A <= 127): the quotient is a float product with the
// reciprocal, within 1.2e-5 of -r / A where |r / A| <= 65 (one ulp of the
// reciprocal, half of one of the sum); 1/512 moves an integer quotient past its
// own floor, and any other lies at least 1/127 from an integer, so floor and
// ceil are exact; larger quotients are clamped whatever their rounding. 12
// instructions against about 40 of the FP64 division with its clamps.
template <bool kSmall>
__device__ __forceinline__ void row_offsets(int r, int a, int* d0, int* d1) {
  int f, c;
  if constexpr (kSmall) {
    constexpr float kBias = 1.0f / 512.0f, kLim = (float)kStageClamp;
    const float n = -(float)r;
    const float rc = __builtin_amdgcn_rcpf(fabsf((float)a));
    f = (int)__builtin_amdgcn_fmed3f(floorf(__builtin_fmaf(n, rc, kBias)), -kLim, kLim);
    c = (int)__builtin_amdgcn_fmed3f(ceilf(__builtin_fmaf(n, rc, -kBias)), -kLim, kLim);
  } else {
    const double q = -(double)r / fabs((double)a);
    f = (int)fmin(fmax(floor(q), -(double)kStageClamp), (double)kStageClamp);
    c = (int)fmin(fmax(ceil(q), -(double)kStageClamp), (double)kStageClamp);
  }
  *d0 = a > 0 ? f : -f;
  *d1 = a > 0 ? c : -c;
}

// One row of a long column (one column per workgroup) in half weights:
// beta, alpha and the candidate mask summed by the caller, delta into the
// bins. half = w/2 in value units (a weight below 2^16).
__device__ __forceinline__ void add_row_reg(bool ap, int d, int32_t half, int k0, int W, int32_t* bins,
                                            int32_t& beta, int32_t& alpha, unsigned long long& cand) {
  const int at = (ap ? 16 : 4) + 4 * min(max(d, -1), 1);
  beta += __mul24(row_coef(kCoefBeta, at), half);
  alpha += __mul24(row_coef(kCoefAlpha, at), half);
  if (d == 0) return;
  const int32_t dl = __mul24(row_coef(kCoefDelta, at), half);
  const int k = k0 + d;
  if (k < 0) {
    beta += dl;
    return;
  }
  if (k >= W) return;
  cand |= 1ull << k;
  const int kb = k + (ap ? 1 : 0);
  if (kb < W) atomicAdd(&bins[kb], dl);
}

// Bounds of a narrow column, from the packed copy where there is one (4 bytes
// for 16).
__device__ __forceinline__ void narrow_bounds(const WalkCtx& C, int q, double& l, double& u) {
  if (C.plan.stage_lu) {
    const uint32_t v = gmem(C.plan.stage_lu)[q];
    l = (double)(int16_t)(v & 0xFFFFu);
    u = (double)(int16_t)(v >> 16);
  } else {
    l = gmem(C.P.lb)[q];
    u = gmem(C.P.ub)[q];
  }
}

// One workgroup per chunk of a long narrow column: bins, beta, alpha and the
// candidate mask of the chunk go to the chunk's partial record. Chunks are
// cut along row ranges and ordered so that consecutive workgroups (placed on
// consecutive XCDs) gather rows from one range each.
struct ChunkSmem {
  double bins[kNarrowBins];
  int32_t ibins[kNarrowBins];
  double red_b[4], red_a[4];
  unsigned long long red_c[4];
};

template <typename Rows>
__device__ __forceinline__ void chunk_task(const WalkCtx& C, int lb, ChunkSmem& S) {
  const DevProblem& P = C.P;
  const double* x = C.x;
  const Rows rs = rows_of<Rows>(C);
  const WalkState* st = C.st;
  ChunkPartial* partials = C.partials;
  if (st->k >= st->iters || st->pass_skip) return;
  double* bins = S.bins;
  int32_t* ibins = S.ibins;
  double* red_b = S.red_b;
  double* red_a = S.red_a;
  unsigned long long* red_c = S.red_c;
  const int tid = threadIdx.x;
  const int lane = tid & (kWave - 1);
  const int wv = tid >> 6;
  const ChunkTask T = C.plan.chunks[lb];
  // integer data with integral weights: breakpoint offsets from one quotient
  // and half-weight integer bins (the identity of row-block staging)
  const bool exact = C.plan.stage_exact != 0 && stage_weights<Rows>(C);
  if (tid < kNarrowBins) {
    bins[tid] = 0.0;
    ibins[tid] = 0;
  }
  __syncthreads();
  double beta = 0.0, alpha = 0.0;
  unsigned long long cand = 0;
  if (T.col >= 0 && exact) {
    const int q = T.col;
    const double xb = gmem(x)[q];
    const double l = gmem(P.lb)[q];
    const int W = (int)(gmem(P.ub)[q] - l) + 1, k0 = (int)(xb - l);
    int32_t ib = 0, ia = 0;
    auto add = [&](const GatherRow& g, int a, int d0, int d1) {
      add_row_reg(a > 0, d0, (int32_t)g.w0, k0, W, ibins, ib, ia, cand);
      if (g.w1 != kNoTwin) add_row_reg(a < 0, d1, (int32_t)g.w1, k0, W, ibins, ib, ia, cand);
    };
    const gptr<const GatherRow> rows = gmem((const GatherRow*)C.grow);
    // software pipeline: the next step's entries are in flight while this
    // step's rows are gathered and binned, two entries per thread and step
    int e = T.e_beg + tid;
    if (C.plan.chunk_ent) {
      const gptr<const uint32_t> ent = gmem(C.plan.chunk_ent);
      const int o = C.plan.chunk_e0;
      uint32_t n0 = 0, n1 = 0;
      if (e < T.e_end) n0 = __builtin_nontemporal_load(&ent[e - o]);
      if (e + 256 < T.e_end) n1 = __builtin_nontemporal_load(&ent[e - o + 256]);
      for (; e < T.e_end; e += 512) {
        const bool two = e + 256 < T.e_end;
        const uint32_t e0 = n0, e1 = two ? n1 : n0;
        const GatherRow g0 = gload(rows, (int64_t)(e0 >> 8));
        const GatherRow g1 = gload(rows, (int64_t)(e1 >> 8));
        if (e + 512 < T.e_end) n0 = __builtin_nontemporal_load(&ent[e - o + 512]);
        if (e + 768 < T.e_end) n1 = __builtin_nontemporal_load(&ent[e - o + 768]);
        const int a0 = (int)(int8_t)(e0 & 0xFFu), a1 = (int)(int8_t)(e1 & 0xFFu);
        int p0, p1, q0, q1;
        row_offsets<true>(g0.r, a0, &p0, &p1);
        row_offsets<true>(g1.r, a1, &q0, &q1);
        add(g0, a0, p0, p1);
        if (two) add(g1, a1, q0, q1);
      }
    } else {
      const gptr<const int32_t> crow = gmem(P.col_row);
      const gptr<const double> cval = gmem(P.col_val);
      for (; e < T.e_end; e += 256) {
        const GatherRow g = gload(rows, (int64_t)crow[e]);
        const int a = (int)cval[e];
        int d0, d1;
        row_offsets<false>(g.r, a, &d0, &d1);
        add(g, a, d0, d1);
      }
    }
    if (tid == 0 && T.first && st->cut_active) {
      const double c = P.obj[q];
      if (c != 0.0)
        add_row_reg(c > 0.0, cutoff_offset(xb, st, c, P.eps), (int32_t)st->wc, k0, W, ibins, ib, ia, cand);
    }
    beta = 0.5 * (double)ib;
    alpha = 0.5 * (double)ia;
  } else if (T.col >= 0) {
    const int q = T.col;
    const double eps = P.eps;
    const double xb = gmem(x)[q];
    const double l = gmem(P.lb)[q], u2 = gmem(P.ub)[q];
    const gptr<const int32_t> crow = gmem(P.col_row);
    const gptr<const double> cval = gmem(P.col_val);
    const int W = (int)(u2 - l) + 1;
    int e = T.e_beg + tid;
    // two entries per step: both gathers are issued before either is used
    for (; e + 256 < T.e_end; e += 512) {
      const int i0 = __builtin_nontemporal_load(&crow[e]);
      const int i1 = __builtin_nontemporal_load(&crow[e + 256]);
      const double a0 = __builtin_nontemporal_load(&cval[e]);
      const double a1 = __builtin_nontemporal_load(&cval[e + 256]);
      const RowState r0 = rs[i0];
      const RowState r1 = rs[i1];
      narrow_entry(xb, r0.r, a0, (double)r0.w0, eps, l, u2, W, bins, beta, alpha, cand);
      if (r0.w1 >= 0.0f) narrow_entry(xb, -r0.r, -a0, (double)r0.w1, eps, l, u2, W, bins, beta, alpha, cand);
      narrow_entry(xb, r1.r, a1, (double)r1.w0, eps, l, u2, W, bins, beta, alpha, cand);
      if (r1.w1 >= 0.0f) narrow_entry(xb, -r1.r, -a1, (double)r1.w1, eps, l, u2, W, bins, beta, alpha, cand);
    }
    if (e < T.e_end) {
      const int i0 = __builtin_nontemporal_load(&crow[e]);
      const double a0 = __builtin_nontemporal_load(&cval[e]);
      const RowState r0 = rs[i0];
      narrow_entry(xb, r0.r, a0, (double)r0.w0, eps, l, u2, W, bins, beta, alpha, cand);
      if (r0.w1 >= 0.0f) narrow_entry(xb, -r0.r, -a0, (double)r0.w1, eps, l, u2, W, bins, beta, alpha, cand);
    }
    if (tid == 0 && T.first && st->cut_active) {
      const double c = P.obj[q];
      if (c != 0.0) narrow_entry(xb, st->rc, c, (double)st->wc, eps, l, u2, W, bins, beta, alpha, cand);
    }
  }
  beta = wave_sum(beta);
  alpha = wave_sum(alpha);
  cand = wave_or(cand);
  if (lane == 0) {
    red_b[wv] = beta;
    red_a[wv] = alpha;
    red_c[wv] = cand;
  }
  __syncthreads();
  if (T.col < 0) return;
  const gptr<ChunkPartial> mine = gmem(partials) + T.slot;
  if (tid < kNarrowBins) mine->bins[tid] = exact ? 0.5 * (double)ibins[tid] : bins[tid];
  if (tid == 0) {
    mine->beta = red_b[0] + red_b[1] + red_b[2] + red_b[3];
    mine->alpha = red_a[0] + red_a[1] + red_a[2] + red_a[3];
    mine->cand = red_c[0] | red_c[1] | red_c[2] | red_c[3];
  }
}

template <typename Rows>
__global__ __launch_bounds__(256) void k_narrow_chunk(const WalkCtx* __restrict__ walks,
                                                      const int32_t* __restrict__ off, int32_t nw) {
  int lb;
  const int w_ = block_walk(off, nw, lb);
  if (w_ < 0) return;
  const WalkCtx& C = walks[w_];
  __shared__ ChunkSmem S;
  chunk_task<Rows>(C, lb, S);
}

// One wavefront per long narrow column.
__global__ __launch_bounds__(256) void k_narrow_combine(const WalkCtx* __restrict__ walks,
                                                        const int32_t* __restrict__ off, int32_t nw) {
  int lb;
  const int w_ = block_walk(off, nw, lb);
  if (w_ < 0) return;
  const WalkCtx& W0 = walks[w_];
  if (W0.st->k >= W0.st->iters || W0.st->pass_skip) return;
  const int idx = lb * 4 + (threadIdx.x >> 6);
  if (idx >= W0.plan.n_chunk_cols) return;
  int q;
  (void)combine_col(W0, idx, threadIdx.x & (kWave - 1), &q);
}

// ---------------------------------------------------------------------------
// Row-range staging (all-integer instances).
// ---------------------------------------------------------------------------

// Staged scoring keeps values as int32 counts of half weights when the
// weights are integers (every term is a multiple of w/2: exact), else FP64.
__device__ __forceinline__ int32_t stage_one(double w, int32_t) { return 2 * (int32_t)w; }
__device__ __forceinline__ int32_t stage_half(double w, int32_t) { return (int32_t)w; }
__device__ __forceinline__ double stage_one(double w, double) { return w; }
__device__ __forceinline__ double stage_half(double w, double) { return 0.5 * w; }
__device__ __forceinline__ double stage_score_of(int32_t v) { return 0.5 * (double)v; }
__device__ __forceinline__ double stage_score_of(double v) { return v; }

// One normalised row of a narrow column in offset form (coefficient sign ap,
// breakpoint t = xbar + d, one = w and half = w/2 in value units): the cases
// of Algorithm 1 phase 1, as phase1() takes them, decided by the sign of d.
// The row adds beta at every position, alpha above xbar and delta from
// offset thr on (thr = d, or d + 1 when the row holds after t).
template <typename V>
__device__ __forceinline__ void row_terms(bool ap, int d, V one, V half, V& beta, V& alpha, V& delta, int& thr) {
  if (ap) {
    thr = d + 1;
    if (d < 0) {
      beta += one;
      alpha -= one;
      delta = -half;
    } else if (d > 0) {
      delta = -one;
    } else {
      alpha -= one;
      delta = 0;
    }
  } else {
    thr = d;
    if (d > 0) {
      beta -= half;
      alpha += one;
      delta = half;
    } else if (d < 0) {
      beta -= one;
      delta = one;
    } else {
      beta -= one;
      alpha += one;
      delta = 0;
    }
  }
}

// The same row added to a column's bins (k0 = xbar - l, W values; half =
// w/2 in value units): beta goes to bin 0, alpha to bin k0 + 1 (the first
// position above xbar), delta to the bin where it starts to apply (bin 0 when
// that is below l, the sink bin kNarrowBins when above u). The breakpoint is
// a candidate when inside [l, u].
template <typename V>
__device__ __forceinline__ void add_row(bool ap, int d, V half, int k0, int W, V* bins, unsigned long long* cand) {
  const int at = row_case(ap, d);
  const V b = (V)row_coef(kCoefBeta, at) * half;
  const V al = (V)row_coef(kCoefAlpha, at) * half;
  const V dl = (V)row_coef(kCoefDelta, at) * half;
  const int k = k0 + d;
  const int kb = k + (ap ? 1 : 0);
  const int idx = k < 0 ? 0 : ((k >= W || kb >= W) ? kNarrowBins : kb);
  const int ia = k0 + 1 < W ? k0 + 1 : kNarrowBins;
  const V zero = 0;
  if (b != zero) atomicAdd(&bins[0], b);
  if (al != zero) atomicAdd(&bins[ia], al);
  if (dl != zero) atomicAdd(&bins[idx], dl);
  if (d != 0 && k >= 0 && k < W) atomicOr(cand, 1ull << k);
}

__device__ __forceinline__ int32_t coef_mul(int c, int32_t half) { return __mul24(c, half); }
__device__ __forceinline__ double coef_mul(int c, double half) { return (double)c * half; }

// add_row for a run of records of one column, from a record's case and offset:
// beta, alpha and the candidate mask go to the caller's registers (flushed
// once per run), the delta to its bin; deltas for bin 0 join beta, those
// beyond u (the sink bin, never read) are dropped.
template <typename V>
__device__ __forceinline__ void add_row_run(int at, int d, V half, int k0, int W, V* bins, V& beta, V& alpha,
                                            unsigned long long& cand) {
  beta += coef_mul(row_coef(kCoefBeta, at), half);
  alpha += coef_mul(row_coef(kCoefAlpha, at), half);
  const V dl = coef_mul(row_coef(kCoefDelta, at), half);
  const int k = k0 + d;
  const int kb = k + row_coef(kCaseAfter, at);
  if (dl != (V)0) {
    if (k < 0)
      beta += dl;
    else if (kb < W)
      atomicAdd(&bins[kb], dl);
  }
  if (d != 0 && (unsigned)k < (unsigned)W) cand |= 1ull << k;
}

// A record's fields.
__device__ __forceinline__ uint32_t rec_half(bool ap, int d) {
  return (uint32_t)row_case(ap, d) | (uint32_t)((d >= kStageClamp ? 0 : d) & 0x7F) << 5;
}
__device__ __forceinline__ uint64_t make_rec(int lc, bool ap, int d0, bool twin, int d1, uint32_t top) {
  const uint32_t lo = (uint32_t)lc | rec_half(ap, d0) << 8 | (twin ? rec_half(!ap, d1) : (uint32_t)kCaseNone) << 20;
  return (uint64_t)lo | (uint64_t)top << 32;
}
__device__ __forceinline__ int rec_case0(uint32_t lo) { return (int)__builtin_amdgcn_ubfe(lo, 8, 5); }
__device__ __forceinline__ int rec_d0(uint32_t lo) { return __builtin_amdgcn_sbfe((int)lo, 13, 7); }
__device__ __forceinline__ int rec_case1(uint32_t lo) { return (int)__builtin_amdgcn_ubfe(lo, 20, 5); }
__device__ __forceinline__ int rec_d1(uint32_t lo) { return (int)lo >> 25; }

// A record's row or twin in the form row_terms takes.
__device__ __forceinline__ bool case_after(int at) { return row_coef(kCaseAfter, at) != 0; }
__device__ __forceinline__ int case_offset(int at, int d) { return at >= 24 ? kStageClamp : d; }

// One single-entry column's row and twin.
struct StageRec {
  bool ap, twin;
  int d0, d1;
  double w0, w1;
};

template <typename V>
struct StagePackSmem {
  // columns binned at once: a whole pack with int32 values, half of one with
  // FP64 values (which then takes two passes over the records)
  static constexpr int kCols = sizeof(V) == 4 ? kStagePackCols : kStagePackCols / 2;
  V bins[kCols][kNarrowBins + 1];  // padded: lane c reads row c without bank conflicts
  unsigned long long cand[kCols];
  double xb[kCols];
  int32_t W[kCols], k0[kCols];
};

struct StageShortSmem {
  uint64_t rec[kShortMax][kStageShort];  // slot-major: thread c reads rec[*][c]
  int32_t cnt[kStageShort];
};

// Segment table of scoring task t in LDS: beg[rb] = first record of the
// task in row block rb, pre[rb] = the task's records in blocks before rb
// (pre[nrb] = all of them). Ends with a barrier.
struct StageSegs {
  int32_t beg[kStageMaxRb];
  int32_t pre[kStageMaxRb + 1];
};

__device__ __forceinline__ int stage_segments(const WalkCtx& C, int t, StageSegs& G) {
  const int nrb = C.plan.n_stage_rb;
  const int per = 2 * nrb + 1;
  const gptr<const int32_t> tab = gmem(C.plan.stage_seg + (size_t)t * per);
  for (int k = threadIdx.x; k < per; k += blockDim.x) {
    const int32_t v = tab[k];
    if (k < nrb)
      G.beg[k] = v;
    else
      G.pre[k - nrb] = v;
  }
  __syncthreads();
  return G.pre[nrb];
}

// Half weights of a record's row and twin in value units.
template <typename Rows>
__device__ __forceinline__ void rec_weights(uint64_t r, bool, const Rows&, int32_t& w0, int32_t& w1) {
  w0 = (int32_t)((r >> 32) & 0xFFFFu);
  w1 = (int32_t)(r >> 48);
}
template <typename Rows>
__device__ __forceinline__ void rec_weights(uint64_t r, bool wts, const Rows& rs, double& w0, double& w1) {
  if (wts) {
    w0 = 0.5 * (double)((r >> 32) & 0xFFFFu);
    w1 = 0.5 * (double)(r >> 48);
  } else {
    const RowState g = rs[(int)(r >> 32)];
    w0 = 0.5 * (double)g.w0;
    w1 = g.w1 >= 0.0f ? 0.5 * (double)g.w1 : 0.0;
  }
}

// A pack of narrow columns from its records: counting sort into LDS bins
// that also hold beta (bin 0) and alpha (bin xbar - l + 1), so the score of
// position l + k is the prefix sum of bins 0..k; one lane per column then
// scans its bins and keeps the best candidate (smallest position on ties).
// kPairs: the records of every segment are whole pairs at even positions (see
// PassPlan::stage_pairs).
template <bool kPairs, typename Rows, typename V>
__device__ __forceinline__ void stage_pack(const WalkCtx& C, const Rows& rs, bool wts, int tix, StagePackSmem<V>& S,
                                           StageSegs& G) {
  constexpr int kCols = StagePackSmem<V>::kCols;
  const StageTask T = C.plan.stage_tasks[tix];
  const DevProblem& P = C.P;
  const WalkState* st = C.st;
  const int tid = threadIdx.x;
  const int nc = T.q_end - T.q_begin;
  const V zero = 0;
  const int nrb = C.plan.n_stage_rb;
  stage_segments(C, tix, G);
  constexpr int kPer = kPairs ? 2 : 1;  // records per load
  typedef unsigned long long Unit __attribute__((ext_vector_type(kPer)));
  const gptr<const Unit> recs = (gptr<const Unit>)gmem((const uint64_t*)C.stage_rec);
  for (int c0 = 0; c0 < nc; c0 += kCols) {
    const int ncw = min(kCols, nc - c0);
    if (tid < ncw) {
      const int q = T.q_begin + c0 + tid;
      const double xb = gmem((const double*)C.x)[q];
      double l, u;
      narrow_bounds(C, q, l, u);
      S.xb[tid] = xb;
      S.W[tid] = (int)(u - l) + 1;
      S.k0[tid] = (int)(xb - l);
      S.cand[tid] = 0ull;
    }
    for (int i = tid; i < ncw * (kNarrowBins + 1); i += blockDim.x)
      S.bins[i / (kNarrowBins + 1)][i % (kNarrowBins + 1)] = 0;
    __syncthreads();
    // every thread takes an equal contiguous share of the task's records (in
    // segment order, crossing row-block segments), kRun loads of kPer of them
    // per step; records of columns outside this window (and padding) are
    // skipped
    constexpr int kRun = 4 / kPer;
    {
      const int total = G.pre[nrb] / kPer;
      const int per = (total + (int)blockDim.x - 1) / (int)blockDim.x;
      const int f0 = min(total, tid * per), f1 = min(total, f0 + per);
      // segment of f0: the last one starting at or before it
      int lo = 0, hi = nrb - 1;
      while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (G.pre[mid] <= kPer * f0)
          lo = mid;
        else
          hi = mid - 1;
      }
      int sg = lo;
      int base = (G.beg[sg] - G.pre[sg]) / kPer;  // load index of the f-th load: base + f
      int send = G.pre[sg + 1] / kPer;
      // a thread's run is sorted by column within a segment: beta, alpha and
      // the candidate mask of the current column stay in registers until the
      // column changes
      int cur = -1, k0 = 0, W = 0;
      V rb_ = 0, ra_ = 0;
      unsigned long long rc_ = 0ull;
      auto flush = [&]() {
        if (cur < 0) return;
        if (rb_ != zero) atomicAdd(&S.bins[cur][0], rb_);
        if (ra_ != zero && k0 + 1 < W) atomicAdd(&S.bins[cur][k0 + 1], ra_);
        if (rc_) atomicOr(&S.cand[cur], rc_);
        rb_ = zero;
        ra_ = zero;
        rc_ = 0ull;
      };
      for (int f = f0; f < f1; f += kRun) {
        Unit r[kRun];
#pragma unroll
        for (int u = 0; u < kRun; ++u) {
          const int fu = f + u;
          if (fu < f1) {
            while (fu >= send) {
              ++sg;
              base = (G.beg[sg] - G.pre[sg]) / kPer;
              send = G.pre[sg + 1] / kPer;
            }
            r[u] = recs[base + fu];
          }
        }
#pragma unroll
        for (int u = 0; u < kRun; ++u) {
          if (f + u >= f1) break;
#pragma unroll
          for (int h = 0; h < kPer; ++h) {
            const uint64_t rec = r[u][h];
            const uint32_t lo = (uint32_t)rec;
            const int lc = (int)(lo & 0xFFu) - c0;
            if (lc < 0 || lc >= ncw) continue;
            if (lc != cur) {
              flush();
              cur = lc;
              k0 = S.k0[lc];
              W = S.W[lc];
            }
            V w0, w1;
            rec_weights(rec, wts, rs, w0, w1);
            add_row_run(rec_case0(lo), rec_d0(lo), w0, k0, W, S.bins[lc], rb_, ra_, rc_);
            if (rec_case1(lo) != kCaseNone)
              add_row_run(rec_case1(lo), rec_d1(lo), w1, k0, W, S.bins[lc], rb_, ra_, rc_);
          }
        }
      }
      flush();
    }
    if (tid < ncw && st->cut_active) {
      const double c = gmem(P.obj)[T.q_begin + c0 + tid];
      if (c != 0.0) {
        const double wc = (double)st->wc;
        add_row(c > 0.0, cutoff_offset(S.xb[tid], st, c, P.eps), stage_half(wc, zero), S.k0[tid], S.W[tid],
                S.bins[tid], &S.cand[tid]);
      }
    }
    __syncthreads();
    if (tid < ncw) {
      const int W = S.W[tid], k0 = S.k0[tid];
      const unsigned long long cand = S.cand[tid];
      const uint32_t clo = (uint32_t)cand, chi = (uint32_t)(cand >> 32);
      V acc = 0, best = 0;
      int bk = -1;
#pragma unroll
      for (int k = 0; k < kNarrowBins; ++k) {
        if (k < W) {
          acc += S.bins[tid][k];
          const bool bit = k < 32 ? ((clo >> k) & 1u) != 0 : ((chi >> (k - 32)) & 1u) != 0;
          const bool ok = (bit || k == 0 || k == W - 1) && k != k0;
          if (ok && (bk < 0 || acc > best)) {
            best = acc;
            bk = k;
          }
        }
      }
      const double xb = S.xb[tid];
      write_result(gmem(C.xhat), gmem(C.s), T.q_begin + c0 + tid, bk >= 0, stage_score_of(best),
                   xb + (double)(bk - k0), xb);
    }
    __syncthreads();  // the next window reuses the LDS
  }
}

// One short narrow column with D stored entries (decoded records e[0..D-1])
// scored directly: value(c) = beta + alpha [c >= 1] + sum of delta [c >= thr]
// at the candidate offsets c (both bounds, breakpoints inside [l, u]; c = 0
// is xbar and excluded), the largest value, the smallest position on ties.
template <int D, typename V>
__device__ __forceinline__ void stage_short_col(const StageRec* e, double xb, int k0, int W, bool cut, bool cpos,
                                                int dcut, double wc, bool& found, double& best, double& bestp) {
  constexpr int NR = 2 * D + 1;
  const V zero = 0;
  V beta = 0, alpha = 0;
  V dl[NR];
  int th[NR], cd[NR];
  bool cv[NR];
#pragma unroll
  for (int k = 0; k < D; ++k) {
    row_terms(e[k].ap, e[k].d0, stage_one(e[k].w0, zero), stage_half(e[k].w0, zero), beta, alpha, dl[2 * k],
              th[2 * k]);
    cd[2 * k] = e[k].d0;
    cv[2 * k] = true;
    if (e[k].twin) {
      row_terms(!e[k].ap, e[k].d1, stage_one(e[k].w1, zero), stage_half(e[k].w1, zero), beta, alpha,
                dl[2 * k + 1], th[2 * k + 1]);
      cd[2 * k + 1] = e[k].d1;
      cv[2 * k + 1] = true;
    } else {
      dl[2 * k + 1] = 0;
      th[2 * k + 1] = 0;
      cd[2 * k + 1] = 0;
      cv[2 * k + 1] = false;
    }
  }
  if (cut) {
    row_terms(cpos, dcut, stage_one(wc, zero), stage_half(wc, zero), beta, alpha, dl[NR - 1], th[NR - 1]);
    cd[NR - 1] = dcut;
    cv[NR - 1] = true;
  } else {
    dl[NR - 1] = 0;
    th[NR - 1] = 0;
    cd[NR - 1] = 0;
    cv[NR - 1] = false;
  }
  const int lo = -k0, hi = W - 1 - k0;
  V bv = 0;
  int bc = 0;
  found = false;
  auto consider = [&](int c) {
    if (c < lo || c > hi || c == 0) return;
    V val = beta + (c >= 1 ? alpha : zero);
#pragma unroll
    for (int j = 0; j < NR; ++j) val += (c >= th[j]) ? dl[j] : zero;
    if (!found || val > bv || (val == bv && c < bc)) {
      found = true;
      bv = val;
      bc = c;
    }
  };
  consider(lo);
  consider(hi);
#pragma unroll
  for (int j = 0; j < NR; ++j)
    if (cv[j]) consider(cd[j]);
  best = stage_score_of(bv);
  bestp = xb + (double)bc;
}

// The integer case of stage_short_col for a column whose records sit in LDS
// slots rec[k][lane]: the records are decoded one at a time into thresholds
// and half-weight deltas, and the breakpoint of each term is its threshold,
// or one less where bit j of `below` is set (a row that holds after its
// breakpoint). Two registers per term, so a short group's workgroup keeps
// the occupancy of the other scoring kernels.
template <int D>
__device__ __forceinline__ void stage_short_int(const StageShortSmem& S, int lane, double xb, int k0, int W, bool cut,
                                                bool cpos, int dcut, int32_t wc, bool& found, double& best,
                                                double& bestp) {
  constexpr int NR = 2 * D + 1;
  constexpr int kNone = 127;  // threshold of an absent term: above every offset
  int32_t beta = 0, alpha = 0;
  int32_t dl[NR];
  int th[NR];
  uint32_t below = 0;
#pragma unroll
  for (int k = 0; k < D; ++k) {
    const uint64_t r = S.rec[k][lane];
    const uint32_t lo = (uint32_t)r;
    const int at0 = rec_case0(lo), at1 = rec_case1(lo);
    const bool ap0 = case_after(at0), ap1 = case_after(at1);
    const int32_t w0 = (int32_t)((r >> 32) & 0xFFFFu), w1 = (int32_t)(r >> 48);
    row_terms(ap0, case_offset(at0, rec_d0(lo)), 2 * w0, w0, beta, alpha, dl[2 * k], th[2 * k]);
    below |= (uint32_t)ap0 << (2 * k);
    // without a twin: weight 0 and an offset above every column
    row_terms(ap1, case_offset(at1, rec_d1(lo)), 2 * w1, w1, beta, alpha, dl[2 * k + 1], th[2 * k + 1]);
    below |= (uint32_t)ap1 << (2 * k + 1);
  }
  if (cut) {
    row_terms(cpos, dcut, 2 * wc, wc, beta, alpha, dl[NR - 1], th[NR - 1]);
    below |= (uint32_t)cpos << (NR - 1);
  } else {
    dl[NR - 1] = 0;
    th[NR - 1] = kNone;
  }
  const int lo = -k0, hi = W - 1 - k0;
  int32_t bv = 0;
  int bc = 0;
  found = false;
  auto consider = [&](int c) {
    if (c < lo || c > hi || c == 0) return;
    int32_t val = beta + (c >= 1 ? alpha : 0);
#pragma unroll
    for (int j = 0; j < NR; ++j) val += (c >= th[j]) ? dl[j] : 0;
    if (!found || val > bv || (val == bv && c < bc)) {
      found = true;
      bv = val;
      bc = c;
    }
  };
  consider(lo);
  consider(hi);
#pragma unroll
  for (int j = 0; j < NR; ++j) consider(th[j] - (int)((below >> j) & 1u));
  best = stage_score_of(bv);
  bestp = xb + (double)bc;
}

// The FP64 case (weights gathered from the row states) in the same form:
// the records are decoded one at a time from the LDS slots, which the
// caller has sorted, so a lane holds three registers per term.
template <int D, typename Rows>
__device__ __forceinline__ void stage_short_dbl(const StageShortSmem& S, int lane, const Rows& rs, double xb, int k0,
                                                int W, bool cut, bool cpos, int dcut, double wc, bool& found,
                                                double& best, double& bestp) {
  constexpr int NR = 2 * D + 1;
  constexpr int kNone = 127;
  const double zero = 0.0;
  double beta = 0.0, alpha = 0.0;
  double dl[NR];
  int th[NR];
  uint32_t below = 0;
#pragma unroll
  for (int k = 0; k < D; ++k) {
    const uint64_t r = S.rec[k][lane];
    const uint32_t lo = (uint32_t)r;
    const int at0 = rec_case0(lo), at1 = rec_case1(lo);
    const bool ap0 = case_after(at0), ap1 = case_after(at1);
    double h0, h1;
    rec_weights(r, false, rs, h0, h1);
    row_terms(ap0, case_offset(at0, rec_d0(lo)), 2.0 * h0, h0, beta, alpha, dl[2 * k], th[2 * k]);
    below |= (uint32_t)ap0 << (2 * k);
    row_terms(ap1, case_offset(at1, rec_d1(lo)), 2.0 * h1, h1, beta, alpha, dl[2 * k + 1], th[2 * k + 1]);
    below |= (uint32_t)ap1 << (2 * k + 1);
  }
  if (cut) {
    row_terms(cpos, dcut, stage_one(wc, zero), stage_half(wc, zero), beta, alpha, dl[NR - 1], th[NR - 1]);
    below |= (uint32_t)cpos << (NR - 1);
  } else {
    dl[NR - 1] = 0.0;
    th[NR - 1] = kNone;
  }
  const int lo = -k0, hi = W - 1 - k0;
  double bv = 0.0;
  int bc = 0;
  found = false;
  auto consider = [&](int c) {
    if (c < lo || c > hi || c == 0) return;
    double val = beta + (c >= 1 ? alpha : zero);
#pragma unroll
    for (int j = 0; j < NR; ++j) val += (c >= th[j]) ? dl[j] : zero;
    if (!found || val > bv || (val == bv && c < bc)) {
      found = true;
      bv = val;
      bc = c;
    }
  };
  consider(lo);
  consider(hi);
#pragma unroll
  for (int j = 0; j < NR; ++j) consider(th[j] - (int)((below >> j) & 1u));
  best = bv;
  bestp = xb + (double)bc;
}

template <typename Rows>
__device__ __forceinline__ void stage_short(const WalkCtx& C, const Rows& rs, bool wts, int tix, StageShortSmem& S,
                                            StageSegs& G) {
  const StageTask T = C.plan.stage_tasks[tix];
  const DevProblem& P = C.P;
  const WalkState* st = C.st;
  const int tid = threadIdx.x;
  const int nc = T.q_end - T.q_begin;
  const int D = T.deg;
  // the column's own data is loaded while the records arrive
  const int q = T.q_begin + min(tid, max(nc - 1, 0));
  const double xb = gmem((const double*)C.x)[q];
  const double c = st->cut_active ? gmem(P.obj)[q] : 0.0;
  double l, ub;
  narrow_bounds(C, q, l, ub);
  S.cnt[tid] = 0;  // stage_segments ends with a barrier
  const int nrb = C.plan.n_stage_rb;
  stage_segments(C, tix, G);
  const gptr<const uint64_t> recs = gmem((const uint64_t*)C.stage_rec);
  constexpr int kRun = 4;
  const int tps = max(1, (int)blockDim.x / nrb);
  for (int sg = tid / tps; sg < nrb; sg += (int)blockDim.x / tps) {
    const int len = G.pre[sg + 1] - G.pre[sg];
    const int per = (len + tps - 1) / tps;
    const int i1 = G.beg[sg] + min(len, (tid % tps + 1) * per);
    for (int i0 = G.beg[sg] + min(len, (tid % tps) * per); i0 < i1; i0 += kRun) {
      uint64_t r[kRun];
#pragma unroll
      for (int u = 0; u < kRun; ++u)
        if (i0 + u < i1) r[u] = recs[i0 + u];
#pragma unroll
      for (int u = 0; u < kRun; ++u)
        if (i0 + u < i1) {
          const int lc = (int)(r[u] & 0xFFu);
          const int k = atomicAdd(&S.cnt[lc], 1);
          S.rec[k][lc] = r[u];
        }
    }
  }
  __syncthreads();
  if (tid >= nc) return;
  const int W = (int)(ub - l) + 1, k0 = (int)(xb - l);
  const bool cut = st->cut_active && c != 0.0;
  const int dcut = cut ? cutoff_offset(xb, st, c, P.eps) : 0;
  bool found = false;
  double best = 0.0, bestp = xb;
  if (wts) {
    const int32_t wc = (int32_t)st->wc;
#define CHAP_SHORT_CASE(DD)                                                                   \
  case DD:                                                                                    \
    stage_short_int<DD>(S, tid, xb, k0, W, cut, c > 0.0, dcut, wc, found, best, bestp);      \
    break;
    switch (D) {
      CHAP_SHORT_CASE(0)
      CHAP_SHORT_CASE(1)
      CHAP_SHORT_CASE(2)
      CHAP_SHORT_CASE(3)
      CHAP_SHORT_CASE(4)
      CHAP_SHORT_CASE(5)
      CHAP_SHORT_CASE(6)
      CHAP_SHORT_CASE(7)
      default:
        CHAP_SHORT_CASE(8)
    }
#undef CHAP_SHORT_CASE
  } else {
    // records arrive in varying order; sort each lane's slots (in LDS) so
    // that sums of non-integral weights are formed in one order
    for (int i = 0; i + 1 < D; ++i)
      for (int k = 0; k + 1 < D - i; ++k) {
        const uint64_t a = S.rec[k][tid], b = S.rec[k + 1][tid];
        if (b < a) {
          S.rec[k][tid] = b;
          S.rec[k + 1][tid] = a;
        }
      }
    const double wc = (double)st->wc;
#define CHAP_SHORT_CASE(DD)                                                                                \
  case DD:                                                                                                 \
    stage_short_dbl<DD, Rows>(S, tid, rs, xb, k0, W, cut, c > 0.0, dcut, wc, found, best, bestp);          \
    break;
    switch (D) {
      CHAP_SHORT_CASE(0)
      CHAP_SHORT_CASE(1)
      CHAP_SHORT_CASE(2)
      CHAP_SHORT_CASE(3)
      CHAP_SHORT_CASE(4)
      CHAP_SHORT_CASE(5)
      CHAP_SHORT_CASE(6)
      CHAP_SHORT_CASE(7)
      default:
        CHAP_SHORT_CASE(8)
    }
#undef CHAP_SHORT_CASE
  }
  write_result(gmem(C.xhat), gmem(C.s), q, found, best, bestp, xb);
}

// One workgroup per slice of a row block's staged entries: the block's rows
// go to LDS (as GatherRow; weights only when the records carry them), then
// every entry of the slice becomes the record of the same index, and the
// slice's single-entry columns (their entry lies in this block) are scored.
template <typename Rows, bool kPacked>
__device__ __forceinline__ void stage_rows_body(const WalkCtx& C, const StageRowTask& T, GatherRow* rows) {
  const Rows rs = rows_of<Rows>(C);
  const bool wts = stage_weights<Rows>(C);
  const int r0 = T.rb * kStageRowBlock;
  const int nr = min(kStageRowBlock, C.P.ms - r0);
  const gptr<const uint64_t> ent = gmem(C.plan.stage_ent);
  const gptr<uint64_t> rec = gmem(C.stage_rec);
  constexpr int kThreads = 512;
  constexpr int kU = 8;  // entries per thread and step, loaded before any is used
  const int tid = threadIdx.x;
  const gptr<const uint32_t> ent32 = gmem(C.plan.stage_ent32);
  using Word = typename std::conditional<kPacked, uint32_t, uint64_t>::type;
  Word wd[kU];
  auto load_step = [&](int base) {
#pragma unroll
    for (int u = 0; u < kU; ++u) {
      const int i = base + u * kThreads;
      if (i < T.e_end) {
        if constexpr (kPacked)
          wd[u] = __builtin_nontemporal_load(&ent32[i]);
        else
          wd[u] = __builtin_nontemporal_load(&ent[i]);
      }
    }
  };
  // the first step's entries are in flight while the row block is loaded
  load_step(T.e_beg + tid);
  {
    constexpr int kPer = kStageRowBlock / kThreads;
    if (compact_source(rs)) {
      // the compact copy already has the LDS format (weights included)
      const gptr<const GatherRow> src = gmem((const GatherRow*)C.grow);
      GatherRow g[kPer];
#pragma unroll
      for (int k = 0; k < kPer; ++k)
        if (tid + k * kThreads < nr) g[k] = gload(src, r0 + tid + k * kThreads);
#pragma unroll
      for (int k = 0; k < kPer; ++k)
        if (tid + k * kThreads < nr) rows[tid + k * kThreads] = g[k];
    } else {
      RowState g[kPer];
#pragma unroll
      for (int k = 0; k < kPer; ++k)
        if (tid + k * kThreads < nr) g[k] = rs[r0 + tid + k * kThreads];
#pragma unroll
      for (int k = 0; k < kPer; ++k)
        if (tid + k * kThreads < nr) {
          GatherRow o;
          o.r = (int32_t)g[k].r;
          o.w0 = wts ? (uint16_t)g[k].w0 : (uint16_t)0;
          o.w1 = g[k].w1 >= 0.0f ? (wts ? (uint16_t)g[k].w1 : (uint16_t)0) : kNoTwin;
          rows[tid + k * kThreads] = o;
        }
    }
  }
  __syncthreads();
  for (int base = T.e_beg + tid; base < T.e_end; base += kU * kThreads) {
    if (base != T.e_beg + tid) load_step(base);
#pragma unroll
    for (int u = 0; u < kU; ++u) {
      const int i = base + u * kThreads;
      if (i < T.e_end) {
        int local, lc, a;
        if constexpr (kPacked) {
          const uint32_t w = wd[u];
          local = (int)(w & 0x1FFFu);
          lc = (int)__builtin_amdgcn_ubfe(w, 13, 8);
          a = __builtin_amdgcn_sbfe((int)w, 21, 8);
        } else {
          local = (int)(wd[u] & 0xFFFFu);
          lc = (int)((wd[u] >> 16) & 0xFFu);
          a = ((int32_t)((uint32_t)(wd[u] >> 24) << 8)) >> 8;
        }
        const GatherRow g = rows[local];
        int d0, d1;
        row_offsets<kPacked>(g.r, a, &d0, &d1);
        const bool twin = g.w1 != kNoTwin;
        const uint32_t top = wts ? ((uint32_t)g.w0 | (twin ? (uint32_t)g.w1 << 16 : 0u)) : (uint32_t)(r0 + local);
        rec[i] = make_rec(lc, a > 0, d0, twin, d1, top);
      }
    }
  }
  // single-entry columns of this block: scored here from the LDS rows
  const DevProblem& P = C.P;
  const WalkState* st = C.st;
  const bool cut_on = st->cut_active != 0;
  const double wc = (double)st->wc;
  const gptr<const double> xg = gmem((const double*)C.x), objg = gmem(P.obj);
  const gptr<double> xhat = gmem(C.xhat), sco = gmem(C.s);
  auto one = [&](int q, int local, int a, double xb, double l, double u, double c) {
    const GatherRow g = rows[local];
    StageRec re;
    re.ap = a > 0;
    row_offsets<kPacked>(g.r, a, &re.d0, &re.d1);
    re.twin = g.w1 != kNoTwin;
    if (wts) {
      re.w0 = (double)g.w0;
      re.w1 = (double)g.w1;
    } else {
      const RowState full = rs[r0 + local];
      re.w0 = (double)full.w0;
      re.w1 = (double)full.w1;
    }
    const int W = (int)(u - l) + 1, k0 = (int)(xb - l);
    const bool cut = c != 0.0;
    const int dcut = cut ? cutoff_offset(xb, st, c, P.eps) : 0;
    bool found;
    double best, bestp;
    if (wts)
      stage_short_col<1, int32_t>(&re, xb, k0, W, cut, c > 0.0, dcut, wc, found, best, bestp);
    else
      stage_short_col<1, double>(&re, xb, k0, W, cut, c > 0.0, dcut, wc, found, best, bestp);
    write_result(xhat, sco, q, found, best, bestp, xb);
  };
  if constexpr (kPacked) {
    // kOne columns per thread and step; a column's loads do not depend on one
    // another, and all of a step's are issued before any is used
    constexpr int kOne = 4;
    const gptr<const uint32_t> oneg = gmem(C.plan.stage_one);
    const int o = C.plan.stage_one_begin;
    for (int q0 = T.c_beg + tid; q0 < T.c_end; q0 += kOne * kThreads) {
      uint32_t w[kOne];
      double xb[kOne], l[kOne], u[kOne], c[kOne];
#pragma unroll
      for (int k = 0; k < kOne; ++k) {
        const int q = q0 + k * kThreads;
        if (q < T.c_end) {
          w[k] = oneg[q - o];
          xb[k] = xg[q];
          narrow_bounds(C, q, l[k], u[k]);
          c[k] = cut_on ? objg[q] : 0.0;
        }
      }
#pragma unroll
      for (int k = 0; k < kOne; ++k) {
        const int q = q0 + k * kThreads;
        if (q < T.c_end) one(q, (int)(w[k] & 0x1FFFu), __builtin_amdgcn_sbfe((int)w[k], 16, 8), xb[k], l[k], u[k], c[k]);
      }
    }
  } else {
    const gptr<const int32_t> cptr = gmem(P.col_ptr), crow = gmem(P.col_row);
    const gptr<const double> cval = gmem(P.col_val);
    for (int q = T.c_beg + tid; q < T.c_end; q += kThreads) {
      const int e = cptr[q];
      double l, u;
      narrow_bounds(C, q, l, u);
      one(q, crow[e] - r0, (int)cval[e], xg[q], l, u, cut_on ? objg[q] : 0.0);
    }
  }
}

// Single passes with caller weights (DualRows) choose the row source once
// per workgroup from the walk state and run the specialised body, so the
// kernel holds the registers of one row accessor, not of both.
template <typename Rows>
__global__ __launch_bounds__(512) void k_stage_rows(const WalkCtx* __restrict__ walks,
                                                    const int32_t* __restrict__ off, int32_t nw) {
  int lb;
  const int w_ = block_walk(off, nw, lb);
  if (w_ < 0) return;
  const WalkCtx& C = walks[w_];
  if (C.st->k >= C.st->iters || C.st->pass_skip) return;
  const StageRowTask T = C.plan.stage_rtasks[lb];
  if (T.rb < 0) return;
  __shared__ GatherRow rows[kStageRowBlock];
  auto body = [&](auto packed) {
    constexpr bool kPacked = decltype(packed)::value;
    if constexpr (std::is_same<Rows, DualRows>::value) {
      if (C.st->compact_rows)
        stage_rows_body<CompactRows, kPacked>(C, T, rows);
      else
        stage_rows_body<FullRows, kPacked>(C, T, rows);
    } else {
      stage_rows_body<Rows, kPacked>(C, T, rows);
    }
  };
  if (C.plan.stage_packed)
    body(std::true_type());
  else
    body(std::false_type());
}

// Workgroups of a walk over ntask scoring tasks: kXcds * ceil(ntask / kXcds)
// of them, workgroup lb taking task (lb mod kXcds) * ceil(ntask / kXcds) +
// lb / kXcds, so that each XCD scores a contiguous run of tasks (whose
// segments share cache lines); -1 for the padding.
__device__ __forceinline__ int stage_task_of(int lb, int ntask) {
  const int per = (ntask + kXcds - 1) / kXcds;
  const int t = (lb % kXcds) * per + lb / kXcds;
  return t < ntask ? t : -1;
}


// The scoring of a staged pass in one launch: the long-column chunks, the packs and the short groups are units of kXcds
// workgroups of one grid, interleaved so that every CU runs latency-bound
// gathers beside VALU-bound scoring; a role's workgroups keep their
// XCD-aware task order. One launch on one stream, instead of three on three,
// keeps the iteration a chain of kernels without event hops between them.
union StageScoreSmem {
  ChunkSmem chunk;
  StagePackSmem<int32_t> pack_i;
  StagePackSmem<double> pack_d;
  StageShortSmem sh;
};

template <bool kPairs, typename Rows>
__device__ __forceinline__ void stage_score_body(const WalkCtx& C, int lb, StageScoreSmem& sm, StageSegs& G) {
  const int32_t unit = gmem(C.plan.stage_units)[lb / kXcds];
  const int role = unit >> 28;
  const int rb = (unit & kStageUnitMask) * kXcds + lb % kXcds;
  if (role == 0) {
    chunk_task<Rows>(C, rb, sm.chunk);
    return;
  }
  const int npk = C.plan.n_stage_packs;
  const Rows rs = rows_of<Rows>(C);
  const bool wts = stage_weights<Rows>(C);
  if (role == 1) {
    const int t = stage_task_of(rb, npk);
    if (t < 0) return;
    if (wts)
      stage_pack<kPairs, Rows, int32_t>(C, rs, true, t, sm.pack_i, G);
    else
      stage_pack<kPairs, Rows, double>(C, rs, false, t, sm.pack_d, G);
    return;
  }
  const int t = stage_task_of(rb, C.plan.n_stage_tasks - npk);
  if (t >= 0) stage_short<Rows>(C, rs, wts, npk + t, sm.sh, G);
}

template <bool kPairs, typename Rows>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(8))) void k_stage_score(
    const WalkCtx* __restrict__ walks, const int32_t* __restrict__ off, int32_t nw) {
  int lb;
  const int w_ = block_walk(off, nw, lb);
  if (w_ < 0) return;
  const WalkCtx& C = walks[w_];
  if (C.st->k >= C.st->iters || C.st->pass_skip) return;
  __shared__ StageScoreSmem sm;
  __shared__ StageSegs G;
  if constexpr (std::is_same<Rows, DualRows>::value) {
    if (C.st->compact_rows)
      stage_score_body<kPairs, CompactRows>(C, lb, sm, G);
    else
      stage_score_body<kPairs, FullRows>(C, lb, sm, G);
  } else {
    stage_score_body<kPairs, Rows>(C, lb, sm, G);
  }
}

// ---------------------------------------------------------------------------
// General columns: Algorithm 1 with a bitonic sort.
// ---------------------------------------------------------------------------

// Sort key: position (canonical +0.0), then marker (-1 < +1 < pad).
__device__ __forceinline__ bool key_greater(double pa, int ma, double pb, int mb) {
  return pa > pb || (pa == pb && ma > mb);
}

constexpr int kPadMarker = 3;

// Emits the entries of column j into (pos, marker, delta) arrays through an
// atomic slot counter; beta/alpha are accumulated per thread.
template <typename Rows, typename Emit>
__device__ __forceinline__ void general_phase1(const DevProblem& P, const Rows& rs, const WalkState* st,
                                               int j, double xb, int tid, int nthreads, double& beta,
                                               double& alpha, Emit emit) {
  const double eps = P.eps;
  const bool isint = P.is_int[j] != 0;
  const int beg = P.col_ptr[j], end = P.col_ptr[j + 1];
  for (int e = beg + tid; e < end; e += nthreads) {
    const RowState q = rs[P.col_row[e]];
    const double a = P.col_val[e];
    BkEntry b0 = phase1(xb, q.r, a, (double)q.w0, eps, isint, beta, alpha);
    if (b0.has) emit(b0.t + 0.0, b0.marker, b0.delta);
    if (q.w1 >= 0.0f) {
      BkEntry b1 = phase1(xb, -q.r, -a, (double)q.w1, eps, isint, beta, alpha);
      if (b1.has) emit(b1.t + 0.0, b1.marker, b1.delta);
    }
  }
  if (tid == 0) {
    const double l = P.lb[j], u = P.ub[j];
    if (isfinite(l)) emit(l + 0.0, -1, 0.0);
    if (isfinite(u)) emit(u + 0.0, -1, 0.0);
    if (st->cut_active) {
      const double c = P.obj[j];
      if (c != 0.0) {
        BkEntry b2 = phase1(xb, st->rc, c, (double)st->wc, eps, isint, beta, alpha);
        if (b2.has) emit(b2.t + 0.0, b2.marker, b2.delta);
      }
    }
  }
}

__device__ __forceinline__ double block_sum256(double v, double* red) {
  v = wave_sum(v);
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  __syncthreads();
  if (lane == 0) red[wv] = v;
  __syncthreads();
  double t = 0.0;
  for (int q = 0; q < (int)(blockDim.x >> 6); ++q) t += red[q];
  return t;
}

// In-place ascending bitonic sort of cap (power of two) keyed entries.
template <typename PosT, typename MarkT, typename DelT>
__device__ __forceinline__ void bitonic_sort(PosT pos, MarkT mk, DelT dl, int cap) {
  for (int size = 2; size <= cap; size <<= 1) {
    for (int stride = size >> 1; stride > 0; stride >>= 1) {
      for (int p = threadIdx.x; p < (cap >> 1); p += blockDim.x) {
        const int i = 2 * p - (p & (stride - 1));
        const int k = i + stride;
        const bool up = (i & size) == 0;
        const double pi = pos[i], pk = pos[k];
        const int mi = mk[i], mk2 = mk[k];
        if (key_greater(pi, mi, pk, mk2) == up) {
          const double di = dl[i];
          pos[i] = pk;
          pos[k] = pi;
          mk[i] = mk2;
          mk[k] = mi;
          dl[i] = dl[k];
          dl[k] = di;
        }
      }
      __syncthreads();
    }
  }
}

// Scan (phase 3) and argmax (phase 4) over sorted entries; one workgroup.
// Elements [0, cap) are split into contiguous per-thread runs.
template <typename PosT, typename MarkT, typename DelT>
__device__ __forceinline__ void scan_argmax(PosT pos, MarkT mk, DelT dl, int cap, double beta, double alpha,
                                            double xb, double l, double u, double* red, int* redk, bool& found,
                                            double& best, double& bestp) {
  const int tid = threadIdx.x, nt = blockDim.x;
  const int per = (cap + nt - 1) / nt;
  const int lo = min(cap, tid * per), hi = min(cap, lo + per);
  double run = 0.0;
  for (int i = lo; i < hi; ++i) run += dl[i];
  // exclusive scan of run totals across the workgroup
  const int lane = tid & 63, wv = tid >> 6;
  double inc = run;
#pragma unroll
  for (int o = 1; o < kWave; o <<= 1) {
    const double y = __shfl_up(inc, o, kWave);
    if (lane >= o) inc += y;
  }
  __syncthreads();
  if (lane == 63) red[wv] = inc;
  __syncthreads();
  double off = inc - run;
  for (int q = 0; q < wv; ++q) off += red[q];
  // per-entry score, best per thread (value desc, index asc)
  double bv = -DBL_MAX;
  int bk = INT_MAX;
  double prefix = off;
  for (int i = lo; i < hi; ++i) {
    const double d = dl[i];
    const double incl = prefix + d;
    const double p = pos[i];
    const int m = mk[i];
    if (m != kPadMarker && isfinite(p) && p >= l && p <= u && p != xb) {
      const double sigma = beta + ((m < 0) ? incl : prefix) + ((p > xb) ? alpha : 0.0);
      if (sigma > bv) {
        bv = sigma;
        bk = i;
      }
    }
    prefix = incl;
  }
  wave_argmax(bv, bk);
  __syncthreads();
  if (lane == 0) {
    red[wv] = bv;
    redk[wv] = bk;
  }
  __syncthreads();
  bv = red[0];
  bk = redk[0];
  for (int q = 1; q < (nt >> 6); ++q) {
    if (red[q] > bv || (red[q] == bv && redk[q] < bk)) {
      bv = red[q];
      bk = redk[q];
    }
  }
  found = bk != INT_MAX;
  best = bv;
  bestp = found ? pos[bk] : xb;
}

template <int CAP, typename Rows>
__global__ __launch_bounds__(256) void k_sort_block(const WalkCtx* __restrict__ walks, const int32_t* __restrict__ off,
                                                    int32_t nw) {
  int lb;
  const int w_ = block_walk(off, nw, lb);
  if (w_ < 0) return;
  const WalkCtx& C = walks[w_];
  const DevProblem& P = C.P;
  const double* x = C.x;
  const Rows rs = rows_of<Rows>(C);
  const WalkState* st = C.st;
  double* xhat = C.xhat;
  double* sc = C.s;
  int c = 0;
  while (c < kSortCaps - 1 && kSortCap[c] != CAP) ++c;
  const int32_t q0 = C.plan.sort_begin[c];
  if (st->k >= st->iters || st->pass_skip) return;
  __shared__ double spos[CAP];
  __shared__ double sdel[CAP];
  __shared__ int smk[CAP];
  __shared__ int scount;
  __shared__ double red[8];
  __shared__ int redk[8];
  const int j = q0 + lb;
  const double xb = x[j];
  if (threadIdx.x == 0) scount = 0;
  __syncthreads();
  double beta = 0.0, alpha = 0.0;
  general_phase1(P, rs, st, j, xb, threadIdx.x, blockDim.x, beta, alpha, [&](double p, int m, double d) {
    const int s = atomicAdd(&scount, 1);
    spos[s] = p;
    smk[s] = m;
    sdel[s] = d;
  });
  beta = block_sum256(beta, red);
  alpha = block_sum256(alpha, red);
  __syncthreads();
  const int cnt = scount;
  for (int i = cnt + threadIdx.x; i < CAP; i += blockDim.x) {
    spos[i] = HUGE_VAL;
    smk[i] = kPadMarker;
    sdel[i] = 0.0;
  }
  __syncthreads();
  int cap = 64;
  while (cap < cnt) cap <<= 1;
  bitonic_sort(spos, smk, sdel, cap);
  bool found;
  double best, bestp;
  scan_argmax(spos, smk, sdel, cap, beta, alpha, xb, P.lb[j], P.ub[j], red, redk, found, best, bestp);
  if (threadIdx.x == 0) write_result(xhat, sc, j, found, best, bestp, xb);
}

template <typename Rows>
__global__ __launch_bounds__(1024) void k_sort_long(const WalkCtx* __restrict__ walks,
                                                    const int32_t* __restrict__ off, int32_t nw) {
  int lb;
  const int w_ = block_walk(off, nw, lb);
  if (w_ < 0) return;
  const WalkCtx& C = walks[w_];
  const DevProblem& P = C.P;
  const double* x = C.x;
  const Rows rs = rows_of<Rows>(C);
  const WalkState* st = C.st;
  double* xhat = C.xhat;
  double* sc = C.s;
  double* gpos = C.long_pos;
  int32_t* gmk = C.long_marker;
  double* gdel = C.long_delta;
  if (st->k >= st->iters || st->pass_skip) return;
  __shared__ int scount;
  __shared__ double red[16];
  __shared__ int redk[16];
  const LongTask T = C.plan.long_tasks[lb];
  const int j = T.col;
  double* pos = gpos + T.offset;
  int32_t* mk = gmk + T.offset;
  double* dl = gdel + T.offset;
  const double xb = x[j];
  if (threadIdx.x == 0) scount = 0;
  __syncthreads();
  double beta = 0.0, alpha = 0.0;
  general_phase1(P, rs, st, j, xb, threadIdx.x, blockDim.x, beta, alpha, [&](double p, int m, double d) {
    const int s = atomicAdd(&scount, 1);
    pos[s] = p;
    mk[s] = m;
    dl[s] = d;
  });
  {
    double b = wave_sum(beta), a = wave_sum(alpha);
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    __syncthreads();
    if (lane == 0) {
      red[wv] = b;
      redk[wv] = 0;
    }
    __syncthreads();
    b = 0.0;
    for (int q = 0; q < 16; ++q) b += red[q];
    __syncthreads();
    if (lane == 0) red[wv] = a;
    __syncthreads();
    a = 0.0;
    for (int q = 0; q < 16; ++q) a += red[q];
    beta = b;
    alpha = a;
  }
  __syncthreads();
  const int cnt = scount;
  for (int i = cnt + threadIdx.x; i < T.cap; i += blockDim.x) {
    pos[i] = HUGE_VAL;
    mk[i] = kPadMarker;
    dl[i] = 0.0;
  }
  __threadfence_block();
  __syncthreads();
  bitonic_sort(pos, mk, dl, T.cap);
  bool found;
  double best, bestp;
  scan_argmax(pos, mk, dl, T.cap, beta, alpha, xb, P.lb[j], P.ub[j], red, redk, found, best, bestp);
  if (threadIdx.x == 0) write_result(xhat, sc, j, found, best, bestp, xb);
}

// ---------------------------------------------------------------------------
// Subset pass: exact best shift of the columns of a proposal set, with the
// same per-entry arithmetic as the full pass. Binary and narrow columns of
// any length are cut into chunks of kSubsetChunk stored entries
// (k_subset_chunks, partial flip sum or bins per chunk) and combined in chunk
// order (k_subset_combine); general columns use one workgroup's LDS sort
// (k_subset_general).
// ---------------------------------------------------------------------------

struct SubsetChunkSmem {
  double bins[kNarrowBins];
  double red[4];
  unsigned long long scand;
};

template <typename Rows>
__device__ __forceinline__ void subset_chunks_body(const WalkCtx& C, const LearnCtx& L, int b, int nb,
                                                   SubsetChunkSmem& SM) {
  const Rows rs = rows_of<Rows>(C);
  const DevProblem& P = C.P;
  const WalkState* st = C.st;
  if (st->k >= st->iters || L.ls->idle) return;
  double* bins = SM.bins;
  double* red = SM.red;
  unsigned long long& scand = SM.scand;
  const int cnt = L.ls->tk[0].count;
  const int chunks = L.ls->tk[0].chunks;
  const int tid = threadIdx.x;
  const double eps = P.eps;
  for (int c = b; c < chunks; c += nb) {
    // selected column of chunk c: the largest i with sub_off[i] <= c
    int lo = 0, hi = cnt - 1;
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if (L.sub_off[mid] <= c)
        lo = mid;
      else
        hi = mid - 1;
    }
    const int q = L.sel[0][lo];
    const int first = (c == L.sub_off[lo]);
    const int e_beg = P.col_ptr[q] + (c - L.sub_off[lo]) * kSubsetChunk;
    const int e_end = min(P.col_ptr[q + 1], e_beg + kSubsetChunk);
    const double xb = C.x[q];
    ChunkPartial* out = L.sub_parts + c;
    if (L.cls[q] == SUB_FLIP) {
      const double d = (1.0 - xb) - xb;
      double v = 0.0;
      for (int e = e_beg + tid; e < e_end; e += blockDim.x) {
        const RowState r = rs[P.col_row[e]];
        const double r2 = r.r + P.col_val[e] * d;
        v += penalty(r.r, r2, (double)r.w0, eps);
        if (r.w1 >= 0.0f) v += penalty(-r.r, -r2, (double)r.w1, eps);
      }
      if (tid == 0 && first && st->cut_active && P.obj[q] != 0.0)
        v += penalty(st->rc, st->rc + P.obj[q] * d, (double)st->wc, eps);
      v = block_sum256(v, red);
      if (tid == 0) out->beta = v;
      __syncthreads();
      continue;
    }
    const double l = P.lb[q], u = P.ub[q];
    const int W = (int)(u - l) + 1;
    if (tid < kNarrowBins) bins[tid] = 0.0;
    if (tid == 0) scand = 0ull;
    __syncthreads();
    double beta = 0.0, alpha = 0.0;
    unsigned long long cand = 0ull;
    for (int e = e_beg + tid; e < e_end; e += blockDim.x) {
      const RowState r = rs[P.col_row[e]];
      const double a = P.col_val[e];
      narrow_entry(xb, r.r, a, (double)r.w0, eps, l, u, W, bins, beta, alpha, cand);
      if (r.w1 >= 0.0f) narrow_entry(xb, -r.r, -a, (double)r.w1, eps, l, u, W, bins, beta, alpha, cand);
    }
    if (tid == 0 && first && st->cut_active && P.obj[q] != 0.0)
      narrow_entry(xb, st->rc, P.obj[q], (double)st->wc, eps, l, u, W, bins, beta, alpha, cand);
    cand = wave_or(cand);
    if ((tid & 63) == 0 && cand) atomicOr(&scand, cand);
    beta = block_sum256(beta, red);
    alpha = block_sum256(alpha, red);
    __syncthreads();
    if (tid < kNarrowBins) out->bins[tid] = bins[tid];
    if (tid == 0) {
      out->beta = beta;
      out->alpha = alpha;
      out->cand = scand;
    }
    __syncthreads();
  }
}

template <typename Rows>
__global__ __launch_bounds__(256) void k_subset_chunks(const WalkCtx* __restrict__ walks,
                                                       const LearnCtx* __restrict__ lc) {
  __shared__ SubsetChunkSmem SM;
  subset_chunks_body<Rows>(walks[0], *lc, (int)blockIdx.x, (int)gridDim.x, SM);
}


// One wavefront per selected binary or narrow column (grid-stride): its
// chunks in order, then the flip score or the bins' scan and argmax.
// With rec (proposal iterations), also the iteration's snapshot and the best
// moves of every workgroup.
__global__ __launch_bounds__(256) void k_subset_combine(const WalkCtx* __restrict__ walks,
                                                        const LearnCtx* __restrict__ lc, int32_t rec) {
  const WalkCtx& C = walks[0];
  const LearnCtx& L = *lc;
  const DevProblem& P = C.P;
  const WalkState* st = C.st;
  const bool active = st->k < st->iters && !L.ls->idle;
  if (rec && blockIdx.x == 0 && threadIdx.x == 0) snapshot(C.st, active);
  if (!active) return;
  BestPair best_pair;
  auto offer = [&](int q, bool found, double v) {
    if (rec && found && v > 0.0) best_pair.offer(v, C.P.perm[q], q, st->k <= (int64_t)C.tabu[q]);
  };
  const int count = L.ls->tk[0].count;
  const int lane = threadIdx.x & 63;
  for (int i = blockIdx.x * 4 + (threadIdx.x >> 6); i < count; i += gridDim.x * 4) {
    const int q = L.sel[0][i];
    const uint8_t cl = L.cls[q];
    if (cl == SUB_GENERAL) continue;
    if (L.group_role && q >= C.plan.grp_col[0] && q < C.plan.grp_col[kGroupClasses]) continue;
    const int c0 = L.sub_off[i], c1 = L.sub_off[i + 1];
    const double xb = C.x[q];
    if (cl == SUB_FLIP) {
      double v = 0.0;
      for (int c = c0; c < c1; ++c) v += L.sub_parts[c].beta;
      if (lane == 0) {
        write_result(C.xhat, C.s, q, true, v, 1.0 - xb, xb);
        offer(q, true, v);
      }
      continue;
    }
    double bv = 0.0, b = 0.0, a = 0.0;
    unsigned long long cand = 0ull;
    for (int c = c0; c < c1; ++c) {
      const ChunkPartial* pp = L.sub_parts + c;
      bv += pp->bins[lane];
      b += pp->beta;
      a += pp->alpha;
      cand |= pp->cand;
    }
    const double l = P.lb[q];
    const int W = (int)(P.ub[q] - l) + 1;
    bool found;
    double best, bestp;
    narrow_finish(bv, b, a, cand, xb, l, W, lane, found, best, bestp);
    if (lane == 0) {
      write_result(C.xhat, C.s, q, found, best, bestp, xb);
      offer(q, found, best);
    }
  }
  if (rec) block_record<4>(best_pair, C.best + blockIdx.x);
}

// One workgroup per selected general column (grid-stride; Algorithm 1 with
// the LDS sort).
struct SubsetGeneralSmem {
  double spos[kSubsetCap];
  double sdel[kSubsetCap];
  int smk[kSubsetCap];
  int scount;
  double red[8];
  int redk[8];
};

// out: this workgroup's best moves, or null.
__device__ __forceinline__ void subset_general_body(const WalkCtx& C, const LearnCtx& L, int b, int nb,
                                                    SubsetGeneralSmem& SM, MoveRecord* out) {
  const DevProblem& P = C.P;
  const WalkState* st = C.st;
  if (st->k >= st->iters || L.ls->idle) return;
  double* spos = SM.spos;
  double* sdel = SM.sdel;
  int* smk = SM.smk;
  int& scount = SM.scount;
  double* red = SM.red;
  int* redk = SM.redk;
  const int tid = threadIdx.x;
  const int count = L.ls->tk[0].count;
  BestPair best_pair;
  for (int i = b; i < count; i += nb) {
    const int q = L.sel[0][i];
    if (L.cls[q] != SUB_GENERAL) continue;
    if (L.group_role && q >= C.plan.grp_col[0] && q < C.plan.grp_col[kGroupClasses]) continue;
    const double xb = C.x[q];
    if (tid == 0) scount = 0;
    __syncthreads();
    double beta = 0.0, alpha = 0.0;
    general_phase1(P, FullRows{gmem((const RowState*)C.rs)}, st, q, xb, tid, blockDim.x, beta, alpha,
                   [&](double p, int m, double d) {
                     const int k = atomicAdd(&scount, 1);
                     spos[k] = p;
                     smk[k] = m;
                     sdel[k] = d;
                   });
    beta = block_sum256(beta, red);
    alpha = block_sum256(alpha, red);
    __syncthreads();
    const int cnt = scount;
    int cap = 64;
    while (cap < cnt) cap <<= 1;
    for (int t = cnt + tid; t < cap; t += blockDim.x) {
      spos[t] = HUGE_VAL;
      smk[t] = kPadMarker;
      sdel[t] = 0.0;
    }
    __syncthreads();
    bitonic_sort(spos, smk, sdel, cap);
    bool found;
    double best, bestp;
    scan_argmax(spos, smk, sdel, cap, beta, alpha, xb, P.lb[q], P.ub[q], red, redk, found, best, bestp);
    if (tid == 0) {
      write_result(C.xhat, C.s, q, found, best, bestp, xb);
      if (out && found && best > 0.0) best_pair.offer(best, P.perm[q], q, st->k <= (int64_t)C.tabu[q]);
    }
    // every reader of this column's LDS arrays is done before the next one
    __syncthreads();
  }
  if (out && tid == 0) *out = best_pair.record();
}

__global__ __launch_bounds__(256) void k_subset_general(const WalkCtx* __restrict__ walks,
                                                        const LearnCtx* __restrict__ lc, int32_t rec_from) {
  __shared__ SubsetGeneralSmem SM;
  subset_general_body(walks[0], *lc, (int)blockIdx.x, (int)gridDim.x, SM,
                      rec_from >= 0 ? walks[0].best + rec_from + blockIdx.x : nullptr);
}

// The scoring of an affected-rescoring iteration in one launch: workgroups
// [0, g0) score the lane-group columns, the next g1 the subset chunks, the other
// g2 scan the kept scores of the columns that the iteration does not score
// (stamp: AffLists::stamp), each role striding over its own work. With the scan
// (every column a lane-group one) the kernel records the iteration's best moves
// and nothing is left for a scanning launch: 21.5 us per iteration on 100k
// columns, 23.0 with one.
template <typename Rows>
__global__ __launch_bounds__(256) void k_aff_score(const WalkCtx* __restrict__ walks,
                                                   const LearnCtx* __restrict__ lc, const AffRun* __restrict__ run,
                                                   const int32_t* __restrict__ stamp, int g0, int g1, int g2) {
  __shared__ union {
    GroupSmem s;
    SubsetChunkSmem c;
  } U;
  const WalkCtx& C = walks[0];
  const int b = (int)blockIdx.x;
  if (b < g0) {
    if (g2 > 0 && b == 0 && threadIdx.x == 0) snapshot(C.st, C.st->k < C.st->iters);
    aff_group_body<Rows>(C, run, b, g0, U.s, g2 > 0 ? C.best + b : nullptr);
  } else if (b < g0 + g1) {
    subset_chunks_body<Rows>(C, *lc, b - g0, g1, U.c);
  } else {
    const WalkState* st = C.st;
    if (st->k >= st->iters) return;
    const bool all = run->n_s < 0;
    const int32_t tag = (int32_t)st->k + 1;
    BestPair best;
    scan_scores(C, st->k, st->copy_best != 0, (b - g0 - g1) * 256 + (int)threadIdx.x, g2 * 256, best,
                [&](int q) { return all || gmem(stamp)[q] == tag; });
    block_record<4>(best, C.best + b - g1);
  }
}

}  // namespace

hipError_t launch_aff_score(const WalkCtx* C, const LearnCtx* L, const AffLists& A, const int g[4], int combine_grid,
                            int compact, hipStream_t s) {
  const unsigned total = (unsigned)(g[0] + g[1] + g[3]);
  if (compact)
    hipLaunchKernelGGL(k_aff_score<CompactRows>, dim3(total), dim3(256), 0, s, C, L, A.run, A.stamp, g[0], g[1], g[3]);
  else
    hipLaunchKernelGGL(k_aff_score<FullRows>, dim3(total), dim3(256), 0, s, C, L, A.run, A.stamp, g[0], g[1], g[3]);
  if (g[2] > 0) hipLaunchKernelGGL(k_subset_general, dim3((unsigned)g[2]), dim3(256), 0, s, C, L, -1);
  // without columns outside the lane-group range there is nothing to combine
  if (g[1] > 0)
    hipLaunchKernelGGL(k_subset_combine, dim3((unsigned)std::max(combine_grid, 1)), dim3(256), 0, s, C, L, 0);
  return hipGetLastError();
}

static int subset_general_grid(const LearnCtx& Lh) { return std::min(Lh.K[0], kSubsetGeneralGrid); }

int32_t subset_records(const LearnCtx& Lh, int has_general) {
  return (Lh.K[0] + 3) / 4 + (has_general ? subset_general_grid(Lh) : 0);
}

hipError_t launch_subset_pass(const WalkCtx* C, const LearnCtx* L, const LearnCtx& Lh, int has_general, int compact,
                              hipStream_t s) {
  const dim3 chunks((unsigned)std::min(kSubsetGrid, std::max(Lh.sub_cap, 1)));
  const int combine = (Lh.K[0] + 3) / 4;
  if (compact)
    hipLaunchKernelGGL(k_subset_chunks<CompactRows>, chunks, dim3(256), 0, s, C, L);
  else
    hipLaunchKernelGGL(k_subset_chunks<FullRows>, chunks, dim3(256), 0, s, C, L);
  hipLaunchKernelGGL(k_subset_combine, dim3((unsigned)combine), dim3(256), 0, s, C, L, 1);
  if (has_general)
    hipLaunchKernelGGL(k_subset_general, dim3((unsigned)subset_general_grid(Lh)), dim3(256), 0, s, C, L, combine);
  return hipGetLastError();
}

int32_t kernel_blocks(const WalkCtx& c, int slot) {
  const PassPlan& p = c.plan;
  switch (slot) {
    case KS_GROUP: return p.grp_blk[kGroupClasses + 1];
    case KS_PACK: return p.n_packs;
    case KS_CHUNK: return p.stage ? 0 : p.n_chunks;  // a staged pass scores its chunks in k_stage_score
    case KS_COMBINE: return (p.n_chunk_cols + 3) / 4;
    case KS_LONG: return p.n_long;
    case KS_STAGE: return p.n_stage_rtasks;
    case KS_STAGE_SCORE: return p.n_stage_units * kXcds;
    case KS_ARGMAX: return c.argmax_blocks + c.argmax_comb;
    case KS_STEP: return c.apply_blocks;
    case KS_COPY: return blocks_for_host(c.P.n, 256);
    default:
      if (slot >= KS_SORT0 && slot < KS_SORT0 + kSortCaps)
        return p.sort_begin[slot - KS_SORT0 + 1] - p.sort_begin[slot - KS_SORT0];
      return 0;
  }
}

hipError_t PassStreams::create() {
  hipError_t e = hipStreamCreateWithFlags(&side, hipStreamNonBlocking);
  if (e == hipSuccess) e = hipEventCreateWithFlags(&join, hipEventDisableTiming);
  if (e == hipSuccess) e = hipEventCreateWithFlags(&fork, hipEventDisableTiming);
  return e;
}

void PassStreams::destroy() {
  if (side) (void)hipStreamDestroy(side);
  if (join) (void)hipEventDestroy(join);
  if (fork) (void)hipEventDestroy(fork);
  side = nullptr;
  join = nullptr;
  fork = nullptr;
}

template <typename Rows>
#define CHAP_LAUNCH(...)      \
  do {                        \
    hipLaunchKernelGGL(__VA_ARGS__); \
    check();                  \
  } while (0)

hipError_t launch_pass_rows(const BatchLaunch& L, hipStream_t stream, const PassStreams* ps, bool defer_combine) {
  const int nw = L.nw;
  auto grid = [&](int slot) { return dim3((unsigned)L.grid[slot]); };
  // a launch error (say, an LDS size the device refuses) is kept by the first
  // check after it; later successful calls would otherwise clear it
  hipError_t first = hipSuccess;
  auto check = [&]() {
    const hipError_t le = hipGetLastError();
    if (first == hipSuccess) first = le;
  };
  // the side stream carries the chunks and the long sorts of unstaged columns
  const bool fork = ps && pass_forks(L);
  hipStream_t s_long = stream;
  hipError_t e = hipSuccess;
  if (fork) {
    e = hipEventRecord(ps->fork, stream);
    if (e == hipSuccess) e = hipStreamWaitEvent(ps->side, ps->fork, 0);
    if (e != hipSuccess) return e;
    s_long = ps->side;
  }
  if (L.total[KS_GROUP] > 0 && L.caller_weights)
    CHAP_LAUNCH((k_group<true, Rows>), grid(KS_GROUP), dim3(256), 0, stream, L.walks, L.off[KS_GROUP], nw);
  else if (L.total[KS_GROUP] > 0)
    CHAP_LAUNCH((k_group<false, Rows>), grid(KS_GROUP), dim3(256), 0, stream, L.walks, L.off[KS_GROUP], nw);
  // staged columns: the records (alone: they are bound by HBM), then the
  // scoring of every staged task and long-column chunk
  if (L.total[KS_STAGE] > 0)
    CHAP_LAUNCH(k_stage_rows<Rows>, grid(KS_STAGE), dim3(512), 0, stream, L.walks, L.off[KS_STAGE], nw);
  // long narrow columns: the chunks of staged walks are roles of
  // k_stage_score, those of unstaged walks k_narrow_chunk workgroups; a batch
  // may hold both, and k_narrow_combine then waits for both (after the join)
  bool combine_after_join = false;
  const bool combine = L.total[KS_COMBINE] > 0 && !(defer_combine && pass_defers_combine(L));
  if (L.total[KS_STAGE_SCORE] > 0 && L.stage_pairs)
    CHAP_LAUNCH((k_stage_score<true, Rows>), grid(KS_STAGE_SCORE), dim3(256), 0, stream, L.walks,
                L.off[KS_STAGE_SCORE], nw);
  else if (L.total[KS_STAGE_SCORE] > 0)
    CHAP_LAUNCH((k_stage_score<false, Rows>), grid(KS_STAGE_SCORE), dim3(256), 0, stream, L.walks,
                L.off[KS_STAGE_SCORE], nw);
  if (L.total[KS_CHUNK] > 0)
    CHAP_LAUNCH(k_narrow_chunk<Rows>, grid(KS_CHUNK), dim3(256), 0, s_long, L.walks, L.off[KS_CHUNK], nw);
  if (combine) {
    if (L.total[KS_CHUNK] == 0)
      CHAP_LAUNCH(k_narrow_combine, grid(KS_COMBINE), dim3(256), 0, stream, L.walks, L.off[KS_COMBINE], nw);
    else if (L.total[KS_STAGE_SCORE] == 0)
      CHAP_LAUNCH(k_narrow_combine, grid(KS_COMBINE), dim3(256), 0, s_long, L.walks, L.off[KS_COMBINE], nw);
    else
      combine_after_join = true;
  }
  if (L.total[KS_LONG] > 0)
    CHAP_LAUNCH(k_sort_long<Rows>, grid(KS_LONG), dim3(1024), 0, s_long, L.walks, L.off[KS_LONG], nw);
  if (L.total[KS_PACK] > 0)
    CHAP_LAUNCH(k_narrow_pack<Rows>, grid(KS_PACK), dim3(256), 0, stream, L.walks, L.off[KS_PACK], nw);
  if (L.total[KS_SORT0] > 0)
    CHAP_LAUNCH((k_sort_block<256, Rows>), grid(KS_SORT0), dim3(256), 0, stream, L.walks, L.off[KS_SORT0], nw);
  if (L.total[KS_SORT0 + 1] > 0)
    CHAP_LAUNCH((k_sort_block<1024, Rows>), grid(KS_SORT0 + 1), dim3(256), 0, stream, L.walks,
                L.off[KS_SORT0 + 1], nw);
  if (L.total[KS_SORT0 + 2] > 0)
    CHAP_LAUNCH((k_sort_block<4096, Rows>), grid(KS_SORT0 + 2), dim3(256), 0, stream, L.walks,
                L.off[KS_SORT0 + 2], nw);
  check();
  e = first;
  if (fork && e == hipSuccess) {
    e = hipEventRecord(ps->join, ps->side);
    if (e == hipSuccess) e = hipStreamWaitEvent(stream, ps->join, 0);
  }
  if (e == hipSuccess && combine_after_join) {
    hipLaunchKernelGGL(k_narrow_combine, grid(KS_COMBINE), dim3(256), 0, stream, L.walks, L.off[KS_COMBINE], nw);
    e = hipGetLastError();
  }
  return e;
}

#undef CHAP_LAUNCH

hipError_t launch_pass(const BatchLaunch& L, hipStream_t stream, const PassStreams* ps, bool defer_combine) {
  if (L.compact == 1) return launch_pass_rows<CompactRows>(L, stream, ps, defer_combine);
  if (L.compact == 2) return launch_pass_rows<DualRows>(L, stream, ps, false);
  return launch_pass_rows<FullRows>(L, stream, ps, false);
}

}  // namespace chap
