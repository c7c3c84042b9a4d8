// Jump values: for every variable the value that minimises the weighted
// violation of its constraints with the other variables held (the jump
// value of Feasibility Jump, which section 3.1 "Best Shift Moves" recalls
// as the move the paper's line sweep generalises).
//
// For column q at the point xbar,
//   V_q(t) = sum over q's stored rows i, in ascending order, of
//            w0_i max(0, y) and, for an equality row, then w1_i max(0, -y),
//            with y = r_i + a_iq (t - xbar_q);
//            then, with the cutoff row active and c_q != 0,
//            w_c max(0, r_c + c_q (t - xbar_q)).
// The jump value minimises V_q over the domain without xbar_q (ties: the
// value closest to xbar_q, then the smaller); the score is V_q(xbar_q) -
// V_q(t*); no value to try gives (xbar_q, 0). An integer variable with at
// most 64 values tries every value; any other variable the kinks of V_q
// (xbar - r_i / a_iq; an integer variable: the integers on either side),
// its finite bounds and, for an integer variable, xbar +- 1 (V_q is convex
// and piecewise linear, so its minimum over the domain is among them).
//
// Every V_q(t) is one sum in the order above, evaluated directly at t, by the
// roles of one launch, k_jump (independent of one another):
//   single  columns with at most one stored entry, one lane each;
//   group   columns with 2 .. kJumpLane stored entries, eight lanes each: the
//           lanes load an entry each into LDS and share the candidates (on
//           exact integer data narrow columns too try only the kinks'
//           neighbours, bounds and xbar +- 1);
//   bins    longer narrow columns on exact integer data: slope and offset
//           bins, one wavefront per chunk of entries;
//   tasks   other longer columns: one wavefront per (column, tile of 64
//           candidates, chunk of kJumpChunk entries), a lane per candidate; the
//           wavefront loads 64 entries at a time into its LDS slice and every
//           lane adds each entry's terms in order (one broadcast read per
//           entry);
// and of a second one, k_jump_combine:
//   columns one wavefront per column scored by tasks: the chunks' partial sums
//           in chunk order, the cutoff term, the argmin over tiles;
//   bins    one workgroup per chunked bins column: the chunks' bins, the scan
//           and the argmin.
// A column of one chunk is summed exactly in the stored order; longer
// columns add per-chunk partial sums, exact on integer data.

#include <algorithm>

#include "chap_internal.h"
#include "move_best.h"

namespace chap {
namespace {

__device__ __forceinline__ double relu(double y) { return y > 0.0 ? y : 0.0; }

__device__ __forceinline__ bool jump_narrow(bool isint, double l, double u) {
  return isint && isfinite(l) && isfinite(u) && u - l + 1.0 <= (double)kJumpNarrow;
}

// (v, |t - xb|, t) lexicographically smaller than (bv, |bt - xb|, bt).
__device__ __forceinline__ bool jump_better(double v, double t, double bv, double bt, double xb) {
  if (v != bv) return v < bv;
  const double dt = fabs(t - xb), db = fabs(bt - xb);
  if (dt != db) return dt < db;
  return t < bt;
}

// Exact data for this call: the instance's data are integers with every
// residual within the bounds in int32 (exact_data), the weights are integers
// below 2^16 (st->compact_rows), and the cutoff row, when active, has small
// integer terms.
__device__ __forceinline__ bool jump_exact(const WalkState* st, int32_t exact_data, int32_t obj_small) {
  return exact_data && st->compact_rows &&
         (!st->cut_active || (obj_small && st->rc == floor(st->rc) && fabs(st->rc) < 2147483648.0));
}

// One entry of a column as the wavefront tasks read it from LDS.
struct JumpEntry {
  double r;
  double a;
  float w0;
  float w1;
};

// Candidate c of a longer column (its tile-major numbering): for a narrow
// column the value l + c; otherwise entry c / 2's kink (integer: floor for
// even c, ceil for odd; continuous: even c only), then the cutoff row's
// kink(s), l, u, xb - 1, xb + 1 (integers) and last xb itself, the point
// whose V the score needs. `valid`: a value to try; `current`: t = xb.
struct JumpCand {
  double t;
  bool valid;
  bool current;
};

__device__ __forceinline__ JumpCand jump_candidate(const DevProblem& P, const RowState* rs, const WalkState* st,
                                                   int q, int beg, int deg, double xb, double l, double u, bool isint,
                                                   bool narrow, int c) {
  JumpCand o{xb, false, false};
  if (narrow) {
    const int W = (int)(u - l) + 1;
    if (c < W) {
      o.t = l + (double)c;
      o.current = o.t == xb;
      o.valid = !o.current;
    }
    return o;
  }
  double t = xb;
  bool ok = false;
  if (c < 2 * deg) {
    const int e = beg + (c >> 1);
    const double kink = xb - rs[P.col_row[e]].r / P.col_val[e];
    if (isint) {
      t = (c & 1) ? ceil(kink) : floor(kink);
      ok = true;
    } else {
      t = kink;
      ok = (c & 1) == 0;
    }
  } else {
    const int s = c - 2 * deg;
    const double cq = P.obj[q];
    const bool cact = st->cut_active && cq != 0.0;
    if (s < 2) {
      if (cact) {
        const double kink = xb - st->rc / cq;
        if (isint) {
          t = s ? ceil(kink) : floor(kink);
          ok = true;
        } else {
          t = kink;
          ok = s == 0;
        }
      }
    } else if (s == 2) {
      t = l;
      ok = true;
    } else if (s == 3) {
      t = u;
      ok = true;
    } else if (s == 4 || s == 5) {
      t = (s == 4) ? xb - 1.0 : xb + 1.0;
      ok = isint;
    } else if (s == 6) {
      o.current = true;
      return o;
    }
  }
  if (ok && isfinite(t) && t >= l && t <= u && t != xb) {
    o.t = t;
    o.valid = true;
  }
  return o;
}

// What the roles of k_jump share.
struct JumpCall {
  DevProblem P;
  const double* x;
  const RowState* rs;
  const GatherRow* grow;  // the call's compact row copy (exact data), or null
  const WalkState* st;
  int32_t exact_data, obj_small;
  const int32_t* singles;  // columns of at most one entry
  const int32_t* groups;   // columns of 2 .. kJumpLane entries
  const JumpBinTask* btasks;
  const JumpTask* tasks;
  int32_t n_singles, n_groups, nbtasks, ntasks, n_plain;
  int32_t small_coef;  // every coefficient is an integer in [-127, 127]
  int32_t blk[3];      // end of the workgroups of bins, tasks, groups (the rest: singles)
  double* part;
  long long* bpart;
  double* jv;
  double* js;
};

__device__ __forceinline__ JumpEntry jump_entry(const JumpCall& J, bool exact, int e) {
  // rows from the 8-byte compact copy on exact data (the same values), else
  // the 16-byte row states
  JumpEntry o;
  const int i = gmem(J.P.col_row)[e];
  o.a = gmem(J.P.col_val)[e];
  if (exact) {
    const GatherRow g = gload(gmem(J.grow), (int64_t)i);
    o.r = (double)g.r;
    o.w0 = (float)g.w0;
    o.w1 = g.w1 == kNoTwin ? -1.0f : (float)g.w1;
  } else {
    const RowState q = gload(gmem(J.rs), (int64_t)i);
    o.r = q.r;
    o.w0 = q.w0;
    o.w1 = q.w1;
  }
  return o;
}

__device__ __forceinline__ double add_entry(double v, const JumpEntry& e, double d) {
  const double y = e.r + e.a * d;
  v = v + (double)e.w0 * relu(y);
  if (e.w1 >= 0.0f) v = v + (double)e.w1 * relu(-y);
  return v;
}

// The values a column of at most kJumpLane entries tries, numbered: a narrow
// column off exact data every value of its domain; any other one, per entry
// and then for the cutoff row when it acts on the column, the values at its
// kink (an integer variable: floor and ceiling, widened by one on either side
// for a narrow column; a continuous one: the kink), then l, u and, for an
// integer variable, xbar - 1 and xbar + 1. Every V formed on exact data is an
// exact integer below 2^53, and then those values hold the chosen one of a
// narrow column too (a value strictly between them has neighbours on one line
// through it; a zero slope makes the neighbour towards xbar tie and win, any
// other slope makes a neighbour smaller); the widening keeps a rounding of the
// FP64 kink across an integer from hiding one.
struct JumpTries {
  bool every, isint;
  int per;  // log2 of the values per kink
  int kinks;
  __device__ __forceinline__ int count(double l, double u) const {
    return every ? (int)(u - l) + 1 : (kinks << per) + (isint ? 4 : 2);
  }
  // kink(i): the i-th kink
  template <typename Kink>
  __device__ __forceinline__ double value(int c, double xb, double l, double u, Kink kink) const {
    if (every) return l + (double)c;
    const int i = c >> per;
    if (i < kinks) {
      const double k = kink(i);
      const int o = c & ((1 << per) - 1);
      if (per == 0) return k;
      if (per == 1) return o ? ceil(k) : floor(k);
      return o < 2 ? floor(k) + (double)(o - 1) : ceil(k) + (double)(o - 2);
    }
    const int sp = c - (kinks << per);
    return sp == 0 ? l : (sp == 1 ? u : (sp == 2 ? xb - 1.0 : xb + 1.0));
  }
};

__device__ __forceinline__ JumpTries jump_tries(bool isint, bool narrow, bool exact, int kinks) {
  return JumpTries{narrow && !exact, isint, isint ? (narrow ? 2 : 1) : 0, kinks};
}

// Columns of at most one entry, a lane each.
__device__ __forceinline__ void jump_single(const JumpCall& J, bool exact, int b) {
  const int i = b * 256 + (int)threadIdx.x;
  if (i >= J.n_singles) return;
  const int q = gmem(J.singles)[i];
  const DevProblem& P = J.P;
  const WalkState* st = J.st;
  const int beg = gmem(P.col_ptr)[q], deg = gmem(P.col_ptr)[q + 1] - beg;
  const double xb = gmem(J.x)[q], l = gmem(P.lb)[q], u = gmem(P.ub)[q];
  const bool isint = gmem(P.is_int)[q] != 0;
  const double cq = st->cut_active ? gmem(P.obj)[q] : 0.0;
  const double rc = st->rc, wc = (double)st->wc;
  JumpEntry e{0.0, 1.0, 0.0f, -1.0f};
  if (deg > 0) e = jump_entry(J, exact, beg);
  auto V = [&](double t) {
    const double d = t - xb;
    double v = deg > 0 ? add_entry(0.0, e, d) : 0.0;
    if (cq != 0.0) v = v + wc * relu(rc + cq * d);
    return v;
  };
  const JumpTries T = jump_tries(isint, jump_narrow(isint, l, u), exact, deg + (cq != 0.0 ? 1 : 0));
  const double k0 = deg > 0 ? xb - e.r / e.a : xb - rc / cq;
  const double k1 = cq != 0.0 ? xb - rc / cq : 0.0;
  bool found = false;
  double bt = xb, bv = 0.0;
  const int nc = T.count(l, u);
  for (int c = 0; c < nc; ++c) {
    const double t = T.value(c, xb, l, u, [&](int k) { return k == 0 ? k0 : k1; });
    if (!(isfinite(t) && t >= l && t <= u && t != xb)) continue;
    const double v = V(t);
    if (!found || jump_better(v, t, bv, bt, xb)) {
      found = true;
      bt = t;
      bv = v;
    }
  }
  gmem(J.jv)[q] = found ? bt : xb;
  gmem(J.js)[q] = found ? V(xb) - bv : 0.0;
}

// Columns of 2 .. kJumpLane entries, kJumpLane lanes each: the longest columns
// have 36 candidates of 8 terms, which one lane needs several thousand dependent
// instructions for; the group's lanes take every eighth candidate.
struct JumpGroupSmem {
  JumpEntry e[256];
  double kink[256 + 256 / kJumpLane];
};
__device__ __forceinline__ void jump_group(const JumpCall& J, bool exact, int b, JumpGroupSmem& S) {
  constexpr int G = kJumpLane;
  const int tid = threadIdx.x, g = tid & (G - 1), base = tid & ~(G - 1);
  const int i = b * (256 / G) + tid / G;
  const bool in = i < J.n_groups;
  const int q = gmem(J.groups)[in ? i : 0];
  const DevProblem& P = J.P;
  const WalkState* st = J.st;
  const int beg = gmem(P.col_ptr)[q], deg = gmem(P.col_ptr)[q + 1] - beg;
  const double xb = gmem(J.x)[q], l = gmem(P.lb)[q], u = gmem(P.ub)[q];
  const bool isint = gmem(P.is_int)[q] != 0;
  const double cq = st->cut_active ? gmem(P.obj)[q] : 0.0;
  const double rc = st->rc, wc = (double)st->wc;
  JumpEntry* E = S.e + base;
  double* kink = S.kink + base + base / G;
  if (g < deg) {
    const JumpEntry e = jump_entry(J, exact, beg + g);
    E[g] = e;
    kink[g] = xb - e.r / e.a;
  }
  if (g == 0 && cq != 0.0) kink[deg] = xb - rc / cq;
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  auto V = [&](double t) {
    const double d = t - xb;
    double v = 0.0;
    for (int k = 0; k < deg; ++k) v = add_entry(v, E[k], d);
    if (cq != 0.0) v = v + wc * relu(rc + cq * d);
    return v;
  };
  const JumpTries T = jump_tries(isint, jump_narrow(isint, l, u), exact, deg + (cq != 0.0 ? 1 : 0));
  // the first of the candidates that are best, as trying them one after
  // another finds it
  bool found = false, nan = false;
  double bt = xb, bv = 0.0;
  int bc = 0;
  const int nc = T.count(l, u);
  auto consider = [&](int c) {
    const double t = T.value(c, xb, l, u, [&](int k) { return kink[k]; });
    if (!(isfinite(t) && t >= l && t <= u && t != xb)) return;
    const double v = V(t);
    nan = nan || v != v;
    if (!found || jump_better(v, t, bv, bt, xb)) {
      found = true;
      bt = t;
      bv = v;
      bc = c;
    }
  };
  for (int c = g; c < nc; c += G) consider(c);
  if (__ballot(nan)) {
    // an overflow makes the comparisons depend on the order: one lane tries
    // every candidate in turn
    found = false;
    bt = xb;
    bv = 0.0;
    if (g == 0)
      for (int c = 0; c < nc; ++c) consider(c);
  }
#pragma unroll
  for (int o = 1; o < G; o <<= 1) {
    const double ov = __shfl_xor(bv, o, kWave), ot = __shfl_xor(bt, o, kWave);
    const bool of = __shfl_xor((int)found, o, kWave) != 0;
    const int oc = __shfl_xor(bc, o, kWave);
    if (of && (!found || jump_better(ov, ot, bv, bt, xb) || (ov == bv && ot == bt && oc < bc))) {
      found = true;
      bt = ot;
      bv = ov;
      bc = oc;
    }
  }
  if (g != 0 || !in) return;
  gmem(J.jv)[q] = found ? bt : xb;
  gmem(J.js)[q] = found ? V(xb) - bv : 0.0;
}

__device__ void jump_task(const DevProblem& P, const double* __restrict__ x, const RowState* __restrict__ rs,
                          const WalkState* __restrict__ st, const JumpTask T, double* __restrict__ part,
                          JumpEntry* E) {
  const int lane = threadIdx.x & (kWave - 1);
  const int q = T.q;
  const int beg = P.col_ptr[q], deg = P.col_ptr[q + 1] - beg;
  const double xb = x[q], l = P.lb[q], u = P.ub[q];
  const bool isint = P.is_int[q] != 0;
  const bool narrow = jump_narrow(isint, l, u);
  const JumpCand cd = jump_candidate(P, rs, st, q, beg, deg, xb, l, u, isint, narrow, T.tile * kWave + lane);
  const double d = cd.t - xb;
  const int e0 = beg + T.chunk * kJumpChunk;
  const int e1 = min(beg + deg, e0 + kJumpChunk);
  // each batch of 64 entries goes through this wavefront's LDS slice; every
  // lane then reads entry k at one address (a broadcast)
  double v = 0.0;
  for (int base = e0; base < e1; base += kWave) {
    const int e = base + lane;
    JumpEntry me{0.0, 0.0, 0.0f, -1.0f};
    if (e < e1) {
      const RowState s = rs[P.col_row[e]];
      me.r = s.r;
      me.w0 = s.w0;
      me.w1 = s.w1;
      me.a = P.col_val[e];
    }
    // the previous batch's reads are done before the slice is overwritten
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    E[lane] = me;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    const int cnt = min(kWave, e1 - base);
#pragma unroll 4
    for (int k = 0; k < cnt; ++k) {
      const JumpEntry q = E[k];
      const double y = q.r + q.a * d;
      v = v + (double)q.w0 * relu(y);
      if (q.w1 >= 0.0f) v = v + (double)q.w1 * relu(-y);
    }
  }
  part[(size_t)T.slot * kWave + lane] = v;
}

// floor(n / d) and ceil(n / d) for d > 0 and |n|, |d| < 2^31, clamped to [-1,
// kJumpNarrow + 1] (positions beyond leave every narrow column). kSmall (d <=
// 127): a float product with the reciprocal, within 1.2e-5 of the quotient
// where that is at most 65; 1/512 moves an integer quotient past its own floor
// and any other lies at least 1/127 from an integer, so the results are exact.
// Otherwise one FP64 division: an integer quotient is exact, and any other lies
// at least 1/d from an integer while the rounding moves it by at most |n/d|
// 2^-53 < 2^-22 / d.
template <bool kSmall>
__device__ __forceinline__ int floor_div(long long n, long long d) {
  constexpr float kTop = (float)(kJumpNarrow + 1);
  if constexpr (kSmall)
    return (int)__builtin_amdgcn_fmed3f(
        floorf(__builtin_fmaf((float)n, __builtin_amdgcn_rcpf((float)d), 1.0f / 512.0f)), -1.0f, kTop);
  return (int)fmin(fmax(floor((double)n / (double)d), -1.0), (double)kTop);
}
template <bool kSmall>
__device__ __forceinline__ int ceil_div(long long n, long long d) {
  constexpr float kTop = (float)(kJumpNarrow + 1);
  if constexpr (kSmall)
    return (int)__builtin_amdgcn_fmed3f(
        ceilf(__builtin_fmaf((float)n, __builtin_amdgcn_rcpf((float)d), -1.0f / 512.0f)), -1.0f, kTop);
  return (int)fmin(fmax(ceil((double)n / (double)d), -1.0), (double)kTop);
}

// One term w max(0, c + a p) over positions p = 0 .. W-1 as bin updates:
// from the first positive position on (a > 0), or up to the last one
// (a < 0), the term is w c + w a p. Updates of bin 0 (every term with a < 0
// that is positive at p = 0, and every term with a > 0 positive from p = 0)
// go to the lane's own k0 and s0, added into the bin once per wavefront:
// as LDS atomics they would all hit one address.
template <bool kSmall>
__device__ __forceinline__ void add_ramp(unsigned long long* K, unsigned long long* S, long long& k0, long long& s0,
                                         long long c, long long a, int w, int W) {
  if (w == 0) return;
  const bool up = a > 0;
  // the position from which on (a > 0) or up to which the term is positive
  const int p = up ? floor_div<kSmall>(-c, a) + 1 : ceil_div<kSmall>(c, -a);
  const long long wc = w * c, wa = kSmall ? (long long)(w * (int)a) : w * a;  // small: below 2^16 * 2^7
  if (up ? p <= 0 : p > 0) {
    k0 += wc;
    s0 += wa;
  }
  if (p > 0 && p < W) {
    atomicAdd(&K[p], (unsigned long long)(up ? wc : -wc));
    atomicAdd(&S[p], (unsigned long long)(up ? wa : -wa));
  }
}

template <int kCtrl, int kRowMask>
__device__ __forceinline__ long long dpp_ll(long long v) {  // identity 0
  const unsigned lo = (unsigned)dpp<kCtrl, kRowMask>((int)v, 0);
  const unsigned hi = (unsigned)dpp<kCtrl, kRowMask>((int)(v >> 32), 0);
  return (long long)(((unsigned long long)hi << 32) | lo);
}
// Sums over the lanes up to and with this one.
__device__ __forceinline__ long long wave_scan(long long v) {
  v += dpp_ll<kRowShr1, 0xF>(v);
  v += dpp_ll<kRowShr2, 0xF>(v);
  v += dpp_ll<kRowShr4, 0xF>(v);
  v += dpp_ll<kRowShr8, 0xF>(v);
  v += dpp_ll<kBcast15, 0xA>(v);
  v += dpp_ll<kBcast31, 0xC>(v);
  return v;
}
__device__ __forceinline__ long long wave_total(long long v) {
  v = wave_scan(v);
  const unsigned lo = __builtin_amdgcn_readlane((unsigned)v, 63);
  const unsigned hi = __builtin_amdgcn_readlane((unsigned)(v >> 32), 63);
  return (long long)(((unsigned long long)hi << 32) | lo);
}

// The argmin of a narrow column from its bins (lane p holds bin p of the
// offsets k and slopes sl, summed over the column's chunks): prefix sums
// across the lanes give V(l + p) exactly, the cutoff term is added in
// integers; lane 0 writes the jump value and score. Every V is an integer in
// [0, 2^52], so the smallest is the largest 2^53 - V; of the lanes that hold it
// the nearest below xbar and the nearest above are the two to choose from.
__device__ __forceinline__ void bins_finish(const DevProblem& P, const WalkState* st, int q, double xb, long long k,
                                            long long sl, double* jv, double* js) {
  const int lane = threadIdx.x & (kWave - 1);
  const double l = gmem(P.lb)[q];
  const int W = (int)(gmem(P.ub)[q] - l) + 1;
  const double cq = gmem(P.obj)[q];
  const bool cact = st->cut_active && cq != 0.0;
  k = wave_scan(k);
  sl = wave_scan(sl);
  long long vi = k + (long long)lane * sl;
  const double t = l + (double)lane;
  if (cact) {
    const long long y = (long long)st->rc + (long long)cq * (long long)(t - xb);
    vi += (long long)st->wc * (y > 0 ? y : 0);
  }
  const double v = (double)vi;
  const bool in = lane < W, cur = in && t == xb;
  const double key = in && !cur ? 9007199254740992.0 - v : 0.0;
  const double best = wave_max_pos(key);
  const unsigned long long m = __ballot(key == best && best > 0.0), below = __ballot(t < xb);
  const unsigned long long ml = m & below, mu = m & ~below, m0 = __ballot(cur);
  const double tl = l + (double)(63 - __builtin_clzll(ml | 1ull)), tu = l + (double)__builtin_ctzll(mu | (1ull << 63));
  const bool lower = ml != 0 && (mu == 0 || xb - tl <= tu - xb);
  const double v0 = m0 ? __shfl(v, __builtin_ctzll(m0 | (1ull << 63)), kWave) : 0.0;
  if (lane == 0) {
    gmem(jv)[q] = m ? (lower ? tl : tu) : xb;
    gmem(js)[q] = m ? v0 - (9007199254740992.0 - best) : 0.0;
  }
}

// One wavefront per bins task: the chunk's entries (and the twins of
// equality rows), one per lane, as slope and offset bins of the column's
// positions in the wavefront's own LDS slice. A task's entries lie in one
// eighth of the rows, and the four tasks of a workgroup in the same eighth,
// which the task order places on one XCD, so the row gathers stay in that
// XCD's L2.
struct JumpBinSmem {
  unsigned long long K[4][kWave], S[4][kWave];
};
template <bool kSmall>
__device__ __forceinline__ void jump_bins(const JumpCall& J, int b, JumpBinSmem& M) {
  const int id = b * 4 + (threadIdx.x >> 6);
  if (id >= J.nbtasks) return;  // whole wavefronts leave together
  const int lane = threadIdx.x & (kWave - 1);
  const DevProblem& P = J.P;
  unsigned long long* K = M.K[threadIdx.x >> 6];
  unsigned long long* S = M.S[threadIdx.x >> 6];
  K[lane] = 0ull;
  S[lane] = 0ull;
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  const JumpBinTask T = J.btasks[id];
  if (T.q < 0) return;  // padding of the row-range interleave
  const int q = T.q;
  const double xb = gmem(J.x)[q], l = gmem(P.lb)[q];
  const int W = (int)(P.ub[q] - l) + 1;
  long long k0 = 0, s0 = 0;
  // one entry per lane and step (two in flight measured slower: 40.0 against
  // 37.1 us, 2M entries); rows from the compact copy (exact on this path:
  // integer residuals and weights)
  for (int e = T.e_beg + lane; e < T.e_end; e += kWave) {
    const GatherRow r = gload(gmem(J.grow), (int64_t)gmem(P.col_row)[e]);
    const double a = gmem(P.col_val)[e];
    const long long c = (long long)((double)r.r + a * (l - xb));  // residual at x_q = l: an integer
    const long long ai = (long long)a;
    add_ramp<kSmall>(K, S, k0, s0, c, ai, (int)r.w0, W);
    if (r.w1 != kNoTwin) add_ramp<kSmall>(K, S, k0, s0, -c, -ai, (int)r.w1, W);
  }
  k0 = wave_total(k0);
  s0 = wave_total(s0);
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  const long long k = (long long)K[lane] + (lane == 0 ? k0 : 0), sl = (long long)S[lane] + (lane == 0 ? s0 : 0);
  if (T.slot < 0) {
    bins_finish(P, J.st, q, xb, k, sl, J.jv, J.js);  // the whole column
    return;
  }
  gmem(J.bpart)[(size_t)T.slot * 2 * kWave + lane] = k;
  gmem(J.bpart)[(size_t)T.slot * 2 * kWave + kWave + lane] = sl;
}

// Every column's score up to the combines: the roles of the workgroups by J.blk,
// the longest work first. The bins tasks begin at workgroup 0, which their order
// over the XCDs counts on. The tasks' workgroups stride over every task, or on
// exact data over the first n_plain only (those of columns without a bins form).
// Bounded by its vector instructions (double precision): 1.6e7 of them on 200k
// integer columns of 2M entries, 34 us, where one lane per short column (29 us;
// 111 registers and serial candidates), the bins with double-precision quotients
// and exchanges through LDS (42 us) and an empty tasks launch (5 us) took 76 us
// one after another. Six wavefronts a SIMD: 37.1 us with five, no spills.
__global__ __launch_bounds__(256, 6) void k_jump(JumpCall J) {
  // aligned so that the tasks' loop reads entries by 16 bytes (1785 against 1920 us
  // on 1000 continuous columns of 2500 entries)
  __shared__ union alignas(16) {
    JumpGroupSmem group;
    JumpEntry task[4][kWave];
    JumpBinSmem bins;
  } M;
  const bool exact = jump_exact(J.st, J.exact_data, J.obj_small);
  const int b = blockIdx.x;
  if (b < J.blk[0]) {
    if (!exact) return;
    if (J.small_coef)
      jump_bins<true>(J, b, M.bins);
    else
      jump_bins<false>(J, b, M.bins);
  } else if (b < J.blk[1]) {
    const int nt = exact ? J.n_plain : J.ntasks;
    for (int id = (b - J.blk[0]) * 4 + (threadIdx.x >> 6); id < nt; id += (J.blk[1] - J.blk[0]) * 4)  // whole wavefronts
      jump_task(J.P, J.x, J.rs, J.st, J.tasks[id], J.part, M.task[threadIdx.x >> 6]);
  } else if (b < J.blk[2]) {
    jump_group(J, exact, b - J.blk[1], M.group);
  } else {
    jump_single(J, exact, b - J.blk[2]);
  }
}

constexpr int kJumpInFlight = 16;  // chunk partials per load round of the combines

// A chunked column with a bins form on exact data (one workgroup per such
// column record): each wavefront adds every fourth chunk's bins,
// kJumpInFlight chunks per load round (integer sums, so any order gives the
// same bins), wavefront 0 adds the four partial sums and finishes.
__device__ __forceinline__ void bins_combine(const DevProblem& P, const double* x, const WalkState* st, const JumpCol J,
                                             const long long* __restrict__ bpart, double* jv, double* js) {
  __shared__ long long red[2][3][kWave];
  const int lane = threadIdx.x & (kWave - 1), wv = threadIdx.x >> 6;
  long long k = 0, sl = 0;
  for (int ch0 = wv * kJumpInFlight; ch0 < J.bn; ch0 += 4 * kJumpInFlight) {
    long long kk[kJumpInFlight], ss[kJumpInFlight];
#pragma unroll
    for (int t = 0; t < kJumpInFlight; ++t) {
      const size_t b = (size_t)(J.bfirst + ch0 + t) * 2 * kWave + lane;
      kk[t] = ch0 + t < J.bn ? bpart[b] : 0ll;
      ss[t] = ch0 + t < J.bn ? bpart[b + kWave] : 0ll;
    }
#pragma unroll
    for (int t = 0; t < kJumpInFlight; ++t) {
      k += kk[t];
      sl += ss[t];
    }
  }
  if (wv > 0) {
    red[0][wv - 1][lane] = k;
    red[1][wv - 1][lane] = sl;
  }
  __syncthreads();
  if (wv != 0) return;
  for (int w = 0; w < 3; ++w) {
    k += red[0][w][lane];
    sl += red[1][w][lane];
  }
  bins_finish(P, st, J.q, x[J.q], k, sl, jv, js);
}

__device__ void jump_combine(const DevProblem& P, const double* __restrict__ x, const RowState* __restrict__ rs,
                             const WalkState* __restrict__ st, int32_t exact_data, int32_t obj_small, const JumpCol J,
                             const double* __restrict__ part, double* __restrict__ jv, double* __restrict__ js) {
  const int lane = threadIdx.x & (kWave - 1);
  const int q = J.q;
  const int beg = P.col_ptr[q], deg = P.col_ptr[q + 1] - beg;
  const double xb = x[q], l = P.lb[q], u = P.ub[q];
  const bool isint = P.is_int[q] != 0;
  const bool narrow = jump_narrow(isint, l, u);
  const double cq = P.obj[q];
  const bool cact = st->cut_active && cq != 0.0;
  const double rc = st->rc, wc = (double)st->wc;
  bool found = false;
  double bt = xb, bv = 0.0, v0 = 0.0;
  bool have0 = false;
  // bins form on exact data: finished by its bins task or by bins_combine
  if (J.bn != 0 && jump_exact(st, exact_data, obj_small)) return;
  for (int tile = 0; tile < J.ntiles; ++tile) {
    const JumpCand cd = jump_candidate(P, rs, st, q, beg, deg, xb, l, u, isint, narrow, tile * kWave + lane);
    const int s0 = J.first_slot + tile * J.nchunks;
    // the chunks' partial sums added in chunk order, kJumpInFlight loaded
    // at a time
    double v = part[(size_t)s0 * kWave + lane];
    for (int ch0 = 1; ch0 < J.nchunks; ch0 += kJumpInFlight) {
      double pv[kJumpInFlight];
#pragma unroll
      for (int t = 0; t < kJumpInFlight; ++t)
        if (ch0 + t < J.nchunks) pv[t] = part[(size_t)(s0 + ch0 + t) * kWave + lane];
#pragma unroll
      for (int t = 0; t < kJumpInFlight; ++t)
        if (ch0 + t < J.nchunks) v = v + pv[t];
    }
    if (cact) v = v + wc * relu(rc + cq * (cd.t - xb));
    if (cd.current) {
      v0 = v;
      have0 = true;
    }
    if (cd.valid && (!found || jump_better(v, cd.t, bv, bt, xb))) {
      found = true;
      bt = cd.t;
      bv = v;
    }
  }
  // argmin across the lanes; V(xb) from the lane that evaluated it
#pragma unroll
  for (int o = 1; o < kWave; o <<= 1) {
    const double ov = __shfl_xor(bv, o, kWave), ot = __shfl_xor(bt, o, kWave);
    const bool of = __shfl_xor((int)found, o, kWave) != 0;
    if (of && (!found || jump_better(ov, ot, bv, bt, xb))) {
      found = true;
      bt = ot;
      bv = ov;
    }
  }
  const unsigned long long m0 = __ballot(have0);
  const int l0 = m0 ? __builtin_ctzll(m0) : 0;
  v0 = __shfl(v0, l0, kWave);
  if (lane == 0) {
    jv[q] = found ? bt : xb;
    js[q] = found ? v0 - bv : 0.0;
  }
}

// The first n_chunk workgroups take the chunked columns with a bins form (on
// exact data), the others stride over the column records, one wavefront per
// record: every record, or on exact data only the first n_plain (the columns
// without a bins form).
__global__ __launch_bounds__(256) void k_jump_combine(DevProblem P, const double* __restrict__ x,
                                                      const RowState* __restrict__ rs,
                                                      const WalkState* __restrict__ st,
                                                      int32_t exact_data, int32_t obj_small,
                                                      const JumpCol* __restrict__ cols, int32_t ncols,
                                                      int32_t n_plain, int32_t n_chunk, const double* __restrict__ part,
                                                      const long long* __restrict__ bpart, double* __restrict__ jv,
                                                      double* __restrict__ js) {
  const bool exact = jump_exact(st, exact_data, obj_small);
  if ((int)blockIdx.x < n_chunk) {
    if (exact) bins_combine(P, x, st, cols[n_plain + blockIdx.x], bpart, jv, js);
    return;
  }
  const int nc = exact ? n_plain : ncols;
  const int b = blockIdx.x - n_chunk, nb = gridDim.x - n_chunk;
  for (int id = b * 4 + (threadIdx.x >> 6); id < nc; id += nb * 4)  // whole wavefronts
    jump_combine(P, x, rs, st, exact_data, obj_small, cols[id], part, jv, js);
}

}  // namespace

hipError_t launch_jump(const DevProblem& P, const JumpPlan& L, const double* x, const RowState* rs, const WalkState* st,
                       const GatherRow* grow, int32_t obj_small, double* jv, double* js, hipStream_t s) {
  constexpr int kStrideGrid = 2048;  // most workgroups that stride over tasks or column records
  JumpCall J{};
  J.P = P;
  J.x = x;
  J.rs = rs;
  J.grow = grow;
  J.st = st;
  J.exact_data = grow != nullptr ? 1 : 0;
  J.obj_small = obj_small;
  J.singles = L.singles;
  J.groups = L.groups;
  J.btasks = L.btasks;
  J.tasks = L.tasks;
  J.n_singles = L.n_singles;
  J.n_groups = L.n_groups;
  J.nbtasks = L.n_btasks;
  J.ntasks = L.n_tasks;
  J.n_plain = L.n_plain_tasks;
  J.small_coef = L.small_coef;
  J.part = L.part;
  J.bpart = L.bpart;
  J.jv = jv;
  J.js = js;
  J.blk[0] = grow ? (L.n_btasks + 3) / 4 : 0;
  J.blk[1] = J.blk[0] + std::min((L.n_tasks + 3) / 4, kStrideGrid);
  J.blk[2] = J.blk[1] + (L.n_groups + 256 / kJumpLane - 1) / (256 / kJumpLane);
  const int end = J.blk[2] + (L.n_singles + 255) / 256;
  if (end > 0) hipLaunchKernelGGL(k_jump, dim3((unsigned)end), dim3(256), 0, s, J);
  if (L.n_cols > 0)
    hipLaunchKernelGGL(k_jump_combine, dim3((unsigned)(L.n_chunk_cols + std::min((L.n_cols + 3) / 4, kStrideGrid))),
                       dim3(256), 0, s, P, x, rs, st, J.exact_data, obj_small, L.cols, L.n_cols, L.n_plain_cols,
                       L.n_chunk_cols, L.part, L.bpart, jv, js);
  return hipGetLastError();
}

}  // namespace chap
