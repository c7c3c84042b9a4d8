// Tabu-walk kernels for gfx950: residual from scratch, state initialisation,
// global move selection under tabu/aspiration, sparse move application and
// weight update.
//
// Residuals r_i = sum_k a_ik x_k - b_i are stored per row (section 3.1
// "Memory Considerations", first remark) in the row's '<=' orientation; the
// negated twin of an equality row has residual -r_i. A move of variable j by
// d updates only the rows of column j: r_i += a_ij d. The objective cutoff
// row c^T x <= bc (section 3.2) is kept in the walk state.

#include <climits>
#include <cmath>

#include "call_begin.h"
#include "chap_internal.h"
#include "exact_sum.h"
#include "learned_rows.h"
#include "move_best.h"
#include "narrow_finish.h"

namespace chap {
namespace {


__device__ __forceinline__ double wave_sum_d(double v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, kWave);
  return v;
}

__device__ __forceinline__ long long wave_sum_ll(long long v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, kWave);
  return v;
}

// Sum across a workgroup of 256 threads; every thread gets the total.
__device__ __forceinline__ long long block_sum_ll(long long v, long long* red) {
  v = wave_sum_ll(v);
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  __syncthreads();
  if (lane == 0) red[wv] = v;
  __syncthreads();
  long long t = 0;
  for (int q = 0; q < (int)(blockDim.x >> 6); ++q) t += red[q];
  return t;
}

__device__ __forceinline__ double block_sum_d(double v, double* red) {
  v = wave_sum_d(v);
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  __syncthreads();
  if (lane == 0) red[wv] = v;
  __syncthreads();
  double t = 0.0;
  for (int q = 0; q < (int)(blockDim.x >> 6); ++q) t += red[q];
  return t;
}

__device__ __forceinline__ int viol_change(double r, double r2, double eps) {
  return (r2 > eps ? 1 : 0) - (r > eps ? 1 : 0);
}


// The objective-related part of a walk state, held in registers by every
// lane of one wavefront (uniform values; lane 0 writes them back).
struct ObjState {
  double f, fbest, bc, rc;
  long long V;
  float wc;
  int has_best, copy_best, cut_active, obj_integral;
  __device__ void load(const WalkState* st) {
    f = st->f;
    fbest = st->fbest;
    bc = st->bc;
    rc = st->rc;
    V = st->V;
    wc = st->wc;
    has_best = st->has_best;
    copy_best = st->copy_best;
    cut_active = st->cut_active;
    obj_integral = st->obj_integral;
  }
  __device__ void store(WalkState* st) const {
    st->f = f;
    st->fbest = fbest;
    st->bc = bc;
    st->rc = rc;
    st->V = V;
    st->wc = wc;
    st->has_best = has_best;
    st->copy_best = copy_best;
    st->cut_active = cut_active;
    st->obj_integral = obj_integral;
  }
  // Cutoff residual c^T x - bc: rounded once from the exact sum acc, or (acc
  // null: FP64 sums of the objective are exact) f - bc.
  __device__ double cutoff_residual(const WaveExact* acc) const { return acc ? acc->round_plus(-bc) : f - bc; }
  // Incumbent rule when no normalised row is violated: the point is
  // feasible; record it if it improves the best objective and (re)set the
  // cutoff row c^T x <= f_best - delta (section 3.2).
  __device__ void incumbent_check(double eps, const WaveExact* acc) {
    if (V != 0) return;
    if (!has_best || f < fbest) {
      fbest = f;
      has_best = 1;
      copy_best = 1;
    }
    const double delta = obj_integral ? 1.0 : 1e-4 * fmax(1.0, fabs(fbest));
    bc = fbest - delta;
    cut_active = 1;
    rc = cutoff_residual(acc);
    V = (rc > eps) ? 1 : 0;
  }
};

// Residual from scratch of every stored row, r_i = sum_k a_ik x_k - b_i
// (coefficients from the int8 row copy when the instance has one), with the
// row's products summed one after another in the row's stored
// order (the order of the caller's CSR, as the definition is written). A
// group of kResidualLanes lanes owns a row: the lanes load consecutive
// entries and form their products (coalesced row reads),
// and every lane of the group then adds the products in entry order from
// its neighbours' registers, so the sum is the sequential one bit for bit. On
// instances whose row activities are exact integers (P.sums_exact) the
// order cannot change the sum: each lane adds its own products and the
// group combines the lanes' sums in three exchanges.
// Weights: kWeightsUnit sets every weight to 1,
// kWeightsScatter copies the caller's normalised weights. With grow, the
// compact row copy is written too (all-integer instances); with the
// caller's weights it is checked as well: st->compact_rows, set by the
// state initialisation that runs first, is cleared when a residual or a
// weight (the cutoff's included) does not fit.
constexpr int kResidualLanes = 8;
constexpr int kResidualSteps = 4;
enum { kWeightsUnit, kWeightsScatter };

constexpr int kResidualRound = kResidualLanes * kResidualSteps;

// One row's sum by a group of kResidualLanes lanes, [rb, re) its entries:
// where the row activities are exact (P.sums_exact) each lane's share, added
// up by the caller; otherwise the whole sequential sum on every lane of the
// group. kResidualSteps entries per lane in flight, every load of a round
// issued before its products are summed. kSmall: int8 coefficients and the
// byte copy of x, whose products are exact integers (instances with exact row
// activities); otherwise the FP64 values (the byte copy of x when xc is
// given) and, unless P.sums_exact, the sequential order within the row.
template <bool kSmall>
__device__ __forceinline__ double residual_rounds(const DevProblem& P, const double* x, const int8_t* xc, int g,
                                                  int rb, int re) {
  constexpr int S = kResidualSteps;
  const gptr<const double> val = gmem(P.row_val);
  const gptr<const int8_t> c8 = gmem(P.row_c8);
  const gptr<const int32_t> col = gmem(P.row_col);
  const gptr<const double> xg = gmem(x);
  const gptr<const int8_t> xcg = gmem(xc);
  double sum = 0.0;
  for (int e0 = rb; e0 < re; e0 += kResidualRound) {
    int c[S];
    if constexpr (kSmall) {
      int a[S];
#pragma unroll
      for (int u = 0; u < S; ++u) {
        const int e = e0 + u * kResidualLanes + g;
        const bool in = e < re;
        c[u] = in ? col[e] : 0;
        a[u] = in ? (int)c8[e] : 0;
      }
#pragma unroll
      for (int u = 0; u < S; ++u) sum = sum + (double)(a[u] * (int)xcg[c[u]]);
    } else {
      double a[S], prod[S];
#pragma unroll
      for (int u = 0; u < S; ++u) {
        const int e = e0 + u * kResidualLanes + g;
        const bool in = e < re;
        c[u] = in ? col[e] : 0;
        a[u] = in ? val[e] : 0.0;
      }
#pragma unroll
      for (int u = 0; u < S; ++u) prod[u] = a[u] * (xc ? (double)xcg[c[u]] : xg[c[u]]);
      if (P.sums_exact) {
#pragma unroll
        for (int u = 0; u < S; ++u) sum = sum + prod[u];
      } else {
#pragma unroll
        for (int u = 0; u < S; ++u) {
          const int cnt = min(kResidualLanes, re - (e0 + u * kResidualLanes));
          for (int t = 0; t < cnt; ++t) sum = sum + __shfl(prod[u], t, kResidualLanes);
        }
      }
    }
  }
  return sum;
}

// The sequential sum of one row's products by a whole wavefront, [rb, re) its
// entries (uniform). The products of kWaveSteps x 64 entries are formed side
// by side, every load issued before any is used; each is then read from its
// lane into a scalar register and added in entry order, which costs an add
// and no exchange through LDS. jmoved, xn: the value column jmoved has from
// now on (a move being applied); -1 for none.
constexpr int kWaveSteps = 4;
__device__ __forceinline__ double read_lane(double v, int lane) {
  const unsigned long long u = __double_as_longlong(v);
  const unsigned lo = __builtin_amdgcn_readlane((unsigned)u, lane);
  const unsigned hi = __builtin_amdgcn_readlane((unsigned)(u >> 32), lane);
  return __longlong_as_double(((unsigned long long)hi << 32) | lo);
}

__device__ __forceinline__ double wave_row_sum(const DevProblem& P, const double* x, int rb, int re, int jmoved,
                                               double xn) {
  const int lane = threadIdx.x & (kWave - 1);
  const gptr<const double> val = gmem(P.row_val);
  const gptr<const int32_t> col = gmem(P.row_col);
  const gptr<const double> xg = gmem(x);
  double sum = 0.0;
  for (int e0 = rb; e0 < re; e0 += kWaveSteps * kWave) {
    int c[kWaveSteps];
    double a[kWaveSteps], prod[kWaveSteps];
#pragma unroll
    for (int u = 0; u < kWaveSteps; ++u) {
      const int e = e0 + u * kWave + lane;
      const bool in = e < re;
      c[u] = in ? col[e] : 0;
      a[u] = in ? val[e] : 0.0;
    }
#pragma unroll
    for (int u = 0; u < kWaveSteps; ++u) prod[u] = a[u] * (c[u] == jmoved ? xn : xg[c[u]]);
#pragma unroll
    for (int u = 0; u < kWaveSteps; ++u) {
      const int cnt = min(kWave, re - (e0 + u * kWave));
      int t = 0;
      for (; t + 8 <= cnt; t += 8)
#pragma unroll
        for (int k = 0; k < 8; ++k) sum = sum + read_lane(prod[u], t + k);
      for (; t < cnt; ++t) sum = sum + read_lane(prod[u], t);
    }
  }
  return sum;
}

// Writes row i's residual r and weights (Unit: 1 and the twin's 1;
// Scatter: the caller's w0 and w1) and, with grow, its compact
// copy; with the caller's weights the copy is checked as well: the state
// initialisation has run and checked the cutoff weight, and a residual or
// weight that does not fit clears st->compact_rows.
template <int kWeights>
__device__ __forceinline__ void write_residual(int64_t i, double r, float w0, float w1, bool twin,
                                               RowState* __restrict__ rs, GatherRow* __restrict__ grow,
                                               WalkState* st_w) {
  RowState q;
  q.r = r;
  q.w0 = w0;
  q.w1 = twin ? w1 : -1.0f;
  if constexpr (kWeights == kWeightsUnit) {
    q.w0 = 1.0f;
    q.w1 = twin ? 1.0f : -1.0f;
    if (grow) {
      GatherRow cr;
      cr.r = (int32_t)r;
      cr.w0 = 1;
      cr.w1 = twin ? (uint16_t)1 : kNoTwin;
      grow[i] = cr;
    }
  } else if (grow) {
    const bool ok = r == floor(r) && fabs(r) <= 2147483647.0 && q.w0 == floorf(q.w0) && q.w0 >= 0.0f &&
                    q.w0 < 65535.0f && (q.w1 < 0.0f || (q.w1 == floorf(q.w1) && q.w1 < 65535.0f));
    if (!ok) st_w->compact_rows = 0;  // every writer stores the same value
    GatherRow cr;
    cr.r = ok ? (int32_t)r : 0;
    cr.w0 = ok ? (uint16_t)q.w0 : 0;
    cr.w1 = (ok && q.w1 >= 0.0f) ? (uint16_t)q.w1 : kNoTwin;
    grow[i] = cr;
  }
  rs[i] = q;
}

// Rows of more than kResLongRow entries are left to the grid's last
// workgroups, one wavefront per row of P.long_rows: with eight lanes the
// longest rows set the kernel's time (general instance of 100k columns and
// rows of up to 346 entries: 32 us before).
template <int kWeights>
__global__ __launch_bounds__(256) void k_residual(DevProblem P, int32_t group_blocks, const double* __restrict__ x,
                                                  const int8_t* __restrict__ xc, const WalkState* st,
                                                  uint32_t epoch, RowState* __restrict__ rs,
                                                  const int32_t* __restrict__ nidx, const uint8_t* __restrict__ pair,
                                                  const float* __restrict__ w, GatherRow* __restrict__ grow) {
  WalkState* st_w = const_cast<WalkState*>(st);
  const bool small = xc != nullptr && st->x_misfit != epoch;
  const bool wave = (int)blockIdx.x >= group_blocks;
  const int lanes = wave ? kWave : kResidualLanes;
  const int g = threadIdx.x & (lanes - 1);
  int64_t i = ((int64_t)(blockIdx.x - (wave ? group_blocks : 0)) * blockDim.x + threadIdx.x) / lanes;
  if (wave) {
    if (i >= P.n_long_rows) return;  // whole wavefronts leave together
    i = __builtin_amdgcn_readfirstlane(P.long_rows[i]);
  }
  if (i >= P.ms) return;  // whole groups leave together
  const int rb = P.row_ptr[i], re = P.row_ptr[i + 1];
  if (!wave && P.long_rows && re - rb > kResLongRow) return;
  // lane 0 writes the row: its right-hand side and weights are loaded first
  // and arrive while the entries are read
  double rhs = 0.0;
  float w0 = 1.0f, w1 = -1.0f;
  bool twin = false;
  if (g == 0) {
    rhs = P.row_rhs[i];
    twin = pair[i] != 0;
    if constexpr (kWeights == kWeightsScatter) {
      const int k = nidx[i];
      w0 = w[k];
      if (twin) w1 = w[k + 1];
    }
  }
  double sum;
  if (wave && !P.sums_exact) {
    sum = wave_row_sum(P, x, __builtin_amdgcn_readfirstlane(rb), __builtin_amdgcn_readfirstlane(re), -1, 0.0);
  } else if (wave) {
    sum = 0.0;
    for (int e = rb + g; e < re; e += kWave) sum = sum + P.row_val[e] * x[P.row_col[e]];
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) sum = sum + __shfl_xor(sum, o, kWave);
  } else {
    sum = (P.row_c8 && small && P.sums_exact) ? residual_rounds<true>(P, x, xc, g, rb, re)
                                              : residual_rounds<false>(P, x, small ? xc : nullptr, g, rb, re);
    if (P.sums_exact) {
#pragma unroll
      for (int o = 1; o < kResidualLanes; o <<= 1) sum = sum + __shfl_xor(sum, o, kResidualLanes);
    }
  }
  if (g == 0) write_residual<kWeights>(i, sum - rhs, w0, w1, twin, rs, grow, st_w);
}

// Row sums of one workgroup's P.rb_rows rows with x held in LDS: the
// byte copy of x is swept in kResXBlock-column blocks (the next block's
// bytes loaded into registers while the current one is used), and the
// group's entries of each block (int8 coefficient, word = row in group and
// column in block) add their products into int32 LDS sums (exact: the
// layout exists only where every row's byte-range activity fits). This
// trades the one random L2 request per nonzero of k_residual for whole-line
// reads of x. A call whose point does not fit the byte copy sums the rows
// from x as k_residual does.
constexpr int kResBlockedThreads = 1024;
static_assert(kResXBlock == (1 << 17) && kResGroupRows <= (1 << 15), "entry word: row << 17 | column");
template <int kWeights>
__global__ __launch_bounds__(kResBlockedThreads) void k_residual_blocked(
    DevProblem P, const double* __restrict__ x, const int8_t* __restrict__ xc, const WalkState* st, uint32_t epoch,
    RowState* __restrict__ rs, const int32_t* __restrict__ nidx, const uint8_t* __restrict__ pair,
    const float* __restrict__ w, GatherRow* __restrict__ grow) {
  __shared__ int32_t acc[kResGroupRows];
  __shared__ __align__(16) int8_t xs[kResXBlock];
  WalkState* st_w = const_cast<WalkState*>(st);
  const int64_t i0 = (int64_t)blockIdx.x * P.rb_rows;
  const int rows = (int)min((int64_t)P.rb_rows, (int64_t)P.ms - i0);
  const bool small = st->x_misfit != epoch;
  if (small) {
    constexpr int kV = kResXBlock / 16 / kResBlockedThreads;  // 16-byte words of a block per thread
    constexpr int kE = 4;                                      // entries per thread in flight
    const int4* __restrict__ xv = (const int4*)xc;
    const gptr<const int8_t> xb = gmem(xc);
    const gptr<const uint32_t> ent = gmem(P.rb_ent);
    const gptr<const int8_t> c8 = gmem(P.rb_c8);
    const int nxb = P.rb_nxb;
    const int32_t* seg = P.rb_seg + (int64_t)blockIdx.x * nxb;
    for (int t = threadIdx.x; t < rows; t += kResBlockedThreads) acc[t] = 0;
    // block b's bytes below n: whole 16-byte words, then the single bytes of
    // the last one (words past n are neither loaded nor read)
    int4 pre[kV];
    auto load_block = [&](int b) {
      const int64_t c0 = (int64_t)b * kResXBlock;
      const int bytes = (int)min((int64_t)kResXBlock, (int64_t)P.n - c0);
#pragma unroll
      for (int v = 0; v < kV; ++v) {
        const int t = threadIdx.x + v * kResBlockedThreads;
        if (16 * t + 16 <= bytes) {
          pre[v] = xv[c0 / 16 + t];
        } else if (16 * t < bytes) {
          int32_t part[4] = {0, 0, 0, 0};
          for (int k = 0; 16 * t + k < bytes; ++k)
            part[k >> 2] |= (int32_t)(uint8_t)xb[c0 + 16 * t + k] << (8 * (k & 3));
          pre[v] = make_int4(part[0], part[1], part[2], part[3]);
        }
      }
    };
    auto store_block = [&](int b) {
      const int bytes = (int)min((int64_t)kResXBlock, (int64_t)P.n - (int64_t)b * kResXBlock);
#pragma unroll
      for (int v = 0; v < kV; ++v) {
        const int t = threadIdx.x + v * kResBlockedThreads;
        if (16 * t < bytes) ((int4*)xs)[t] = pre[v];
      }
    };
    int b = 0;
    while (b < nxb && seg[b] == seg[b + 1]) ++b;  // blocks without entries are skipped
    if (b < nxb) load_block(b);
    while (b < nxb) {
      int nb = b + 1;
      while (nb < nxb && seg[nb] == seg[nb + 1]) ++nb;
      __syncthreads();  // the previous block's readers are done
      store_block(b);
      if (nb < nxb) load_block(nb);  // in flight while this block is used
      __syncthreads();
      const int e_end = seg[b + 1];
      for (int e0 = seg[b] + threadIdx.x; e0 < e_end; e0 += kE * kResBlockedThreads) {
        uint32_t wd[kE];
        int a[kE];
#pragma unroll
        for (int u = 0; u < kE; ++u) {
          const int e = e0 + u * kResBlockedThreads;
          wd[u] = e < e_end ? ent[e] : 0u;
          a[u] = e < e_end ? (int)c8[e] : 0;
        }
#pragma unroll
        for (int u = 0; u < kE; ++u)
          if (a[u] != 0) atomicAdd(&acc[wd[u] >> 17], a[u] * (int)xs[wd[u] & (kResXBlock - 1)]);
      }
      b = nb;
    }
    __syncthreads();
    for (int t = threadIdx.x; t < rows; t += kResBlockedThreads) {
      const int64_t i = i0 + t;
      float w0 = 1.0f, w1 = -1.0f;
      const bool twin = pair[i] != 0;
      if constexpr (kWeights == kWeightsScatter) {
        const int k = nidx[i];
        w0 = w[k];
        if (twin) w1 = w[k + 1];
      }
      write_residual<kWeights>(i, (double)acc[t] - P.row_rhs[i], w0, w1, twin, rs, grow, st_w);
    }
  } else {
    // kResidualLanes lanes per row, rows of the group one group of lanes
    // after another (the FP64 path of k_residual)
    const int g = threadIdx.x & (kResidualLanes - 1);
    for (int t = threadIdx.x / kResidualLanes; t < rows; t += kResBlockedThreads / kResidualLanes) {
      const int64_t i = i0 + t;
      double sum = residual_rounds<false>(P, x, nullptr, g, P.row_ptr[i], P.row_ptr[i + 1]);
#pragma unroll
      for (int o = 1; o < kResidualLanes; o <<= 1) sum = sum + __shfl_xor(sum, o, kResidualLanes);
      if (g != 0) continue;
      float w0 = 1.0f, w1 = -1.0f;
      const bool twin = pair[i] != 0;
      if constexpr (kWeights == kWeightsScatter) {
        const int k = nidx[i];
        w0 = w[k];
        if (twin) w1 = w[k + 1];
      }
      write_residual<kWeights>(i, sum - P.row_rhs[i], w0, w1, twin, rs, grow, st_w);
    }
  }
}

// Start point of a seeded walk (internal order): with seed > 0 an integer
// variable with finite bounds starts at l + (h mod (u - l + 1)), h the
// (j+1)-th SplitMix64 output of the seed for original index j; every other
// variable starts at 0 clamped into its bounds.
__global__ __launch_bounds__(256) void k_start_point(DevProblem P, uint64_t seed, double* __restrict__ x,
                                                     int8_t* __restrict__ xc) {
  const int q = blockIdx.x * blockDim.x + threadIdx.x;
  if (q >= P.n) return;
  const double l = P.lb[q], u = P.ub[q];
  double v;
  if (seed != 0 && P.is_int[q] && isfinite(l) && isfinite(u)) {
    const uint64_t h = splitmix64(seed, (uint64_t)P.perm[q]);
    const uint64_t width = (uint64_t)(u - l) + 1;
    v = l + (double)(h % width);
  } else {
    v = 0.0;
    if (v < l) v = l;
    if (v > u) v = u;
  }
  x[q] = v;
  if (xc) xc[q] = (int8_t)v;  // an integer within [l, u] (byte copies are kept only then)
}

__global__ __launch_bounds__(256) void k_stage_x(const int32_t* __restrict__ perm, const double* __restrict__ src,
                                                 double* __restrict__ dst, int8_t* __restrict__ xc, WalkState* st,
                                                 uint32_t epoch, int32_t n, SingleInit init) {
  const int q = blockIdx.x * blockDim.x + threadIdx.x;
  if (q == 0 && init.cutoff_w) single_state(st, init);
  if (q >= n) return;
  const double v = src[perm[q]];
  dst[q] = v;
  if (xc) stage_byte(v, q, xc, st, epoch);
}

constexpr int kInitCopies = 16;

// f = c^T x and V = violated rows as grid reductions; the last workgroup
// writes the walk state. With objacc (objectives whose FP64 sums may be
// inexact) every workgroup adds its products exactly into a fixed-point sum
// in LDS, the last one adds the workgroups' sums, keeps the result in objacc
// and rounds f and the cutoff residual from it; otherwise the FP64 sum is
// exact and its order does not matter.
__global__ __launch_bounds__(256) void k_state_init(DevProblem P, const double* __restrict__ x,
                                                    const RowState* __restrict__ rs, WalkState* st,
                                                    double* partial, uint32_t* ticket, long long* objacc,
                                                    int64_t iters, int32_t tenure, int32_t obj_integral,
                                                    double cutoff_rhs, const float* cutoff_w,
                                                    int32_t check_incumbent, int32_t need_obj, int32_t need_v) {
  __shared__ double redd[4];
  __shared__ long long redl[4];
  // kInitCopies private sums (lane l uses copy l mod kInitCopies): values of
  // one magnitude meet in the same limbs, and one copy would queue every lane
  // of a wavefront at the same three addresses
  __shared__ long long lacc[kInitCopies][kExactLimbs + 1];
  __shared__ uint32_t last;
  long long* plimb = (long long*)(partial + 2 * kInitBlocks);
  const double eps = P.eps;
  const int gt = blockIdx.x * blockDim.x + threadIdx.x;
  const int gs = gridDim.x * blockDim.x;
  if (objacc) {
    for (int t = threadIdx.x; t < kInitCopies * (kExactLimbs + 1); t += blockDim.x) (&lacc[0][0])[t] = 0;
    __syncthreads();
  }
  long long* mine = lacc[threadIdx.x & (kInitCopies - 1)];
  // kU items per thread and step, every load issued before any is used
  constexpr int kU = 4;
  double f = 0.0;
  const int n_obj = need_obj ? P.n : 0;
  for (int j0 = gt; j0 < n_obj; j0 += kU * gs) {
    double c[kU], xv[kU];
#pragma unroll
    for (int u = 0; u < kU; ++u) {
      const int j = j0 + u * gs;
      c[u] = j < n_obj ? P.obj[j] : 0.0;
      xv[u] = j < n_obj ? x[j] : 0.0;
    }
#pragma unroll
    for (int u = 0; u < kU; ++u) {
      if (c[u] == 0.0) continue;
      if (objacc) {
        double p, e;
        exact_product(c[u], xv[u], p, e);
        exact_atomic_add(mine, p);
        exact_atomic_add(mine, e);
      } else {
        f += c[u] * xv[u];
      }
    }
  }
  long long v = 0;
  const int m_v = need_v ? P.ms : 0;
  for (int i0 = gt; i0 < m_v; i0 += kU * gs) {
    RowState q[kU];
#pragma unroll
    for (int u = 0; u < kU; ++u) {
      const int i = i0 + u * gs;
      q[u] = i < m_v ? rs[i] : RowState{0.0, 0.0f, -1.0f};
    }
#pragma unroll
    for (int u = 0; u < kU; ++u) {
      v += (q[u].r > eps) ? 1 : 0;
      if (q[u].w1 >= 0.0f && -q[u].r > eps) v += 1;
    }
  }
  f = block_sum_d(f, redd);
  v = block_sum_ll(v, redl);
  if (threadIdx.x == 0) {
    partial[2 * blockIdx.x] = f;
    partial[2 * blockIdx.x + 1] = (double)v;
  }
  if (objacc) {
    __syncthreads();
    for (int t = threadIdx.x; t < kExactLimbs; t += blockDim.x) {
      long long sum = 0;
      for (int c = 0; c < kInitCopies; ++c) sum += lacc[c][t];
      plimb[blockIdx.x * kExactLimbs + t] = sum;
    }
  }
  __threadfence();
  __syncthreads();
  if (threadIdx.x == 0) last = atomicAdd(ticket, 1u);
  __syncthreads();
  if (last != gridDim.x - 1) return;
  __threadfence();
  if (objacc) {
    // the workgroups' sums: thread t adds limb t mod kExactLimbs of every
    // third workgroup, then the three shares of a limb are added
    constexpr int kShares = 256 / kExactLimbs;
    const int limb = threadIdx.x % kExactLimbs, share = threadIdx.x / kExactLimbs;
    long long sum = 0;
    if (share < kShares) {
#pragma unroll 8
      for (unsigned b = share; b < gridDim.x; b += kShares) sum += plimb[b * kExactLimbs + limb];
      lacc[share][limb] = sum;
    }
    __syncthreads();
    if (threadIdx.x < kExactLimbs) {
      sum = lacc[0][threadIdx.x];
      for (int c = 1; c < kShares; ++c) sum += lacc[c][threadIdx.x];
      lacc[0][threadIdx.x] = sum;
    }
    __syncthreads();
  }
  if (threadIdx.x >= 64) return;
  // one wavefront finishes; every lane computes the same values. The FP64 sums
  // are exact (of f unless objacc replaces it, and of counts), so their order
  // does not matter.
  double ft = 0.0, vt = 0.0;
  for (unsigned b = threadIdx.x; b < gridDim.x; b += 64) {
    ft += partial[2 * b];
    vt += partial[2 * b + 1];
  }
  ft = wave_sum_d(ft);
  vt = wave_sum_d(vt);
  WaveExact acc;
  if (objacc) {
    acc.a = lacc[0][threadIdx.x];
    acc.b = threadIdx.x < kExactLimbs - 64 ? lacc[0][64 + threadIdx.x] : 0;
    acc.normalize();
    acc.store(objacc);
    ft = acc.round_nearest();
  }
  ObjState o;
  o.f = ft;
  o.fbest = HUGE_VAL;
  o.has_best = 0;
  o.copy_best = 0;
  o.obj_integral = obj_integral;
  o.V = (long long)vt;
  o.wc = cutoff_w ? *cutoff_w : 1.0f;
  o.bc = 0.0;
  o.rc = 0.0;
  o.cut_active = 0;
  if (isfinite(cutoff_rhs)) {
    o.cut_active = 1;
    o.bc = cutoff_rhs;
    o.rc = o.cutoff_residual(objacc ? &acc : nullptr);
    if (o.rc > eps) o.V += 1;
  }
  // the start point is the first candidate for the best infeasible point
  const long long v_orig = (long long)vt;
  if (check_incumbent) o.incumbent_check(eps, objacc ? &acc : nullptr);
  if (threadIdx.x != 0) return;
  st->inf_V = v_orig > 0 ? v_orig : LLONG_MAX;
  st->inf_k = v_orig > 0 ? -1 : -2;
  *ticket = 0u;
  o.store(st);
  reset_state(st, iters, tenure, o.wc);
}

// A finished walk's state in the caller's order: x and, with an incumbent,
// best_x by the column permutation, the residuals and weights of the normalised
// rows (an equality row's twin has residual -r and the second weight), the
// cutoff row last; the walk's record and its trace as they are (only the points
// without o.resid). Bounded by the
// scattered 8-byte stores; the host did the same in 5 ms at 2M columns, after
// reading both points and the row states.
__global__ __launch_bounds__(256) void k_state_out(int32_t n, int32_t m, int32_t mp, const int32_t* __restrict__ perm,
                                                   const int32_t* __restrict__ nidx, const uint8_t* __restrict__ pair,
                                                   const double* __restrict__ x, const double* __restrict__ best_x,
                                                   const RowState* __restrict__ rs,
                                                   const WalkState* __restrict__ st,
                                                   const chap_trace_record* __restrict__ trace, int64_t iters,
                                                   StateOut o) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x, stride = (int64_t)gridDim.x * blockDim.x;
  const bool best = st->has_best != 0;
  for (int64_t q = i; q < n; q += stride) {
    const int j = perm[q];
    o.x[j] = x[q];
    if (best) o.best[j] = best_x[q];
  }
  if (!o.resid) return;
  for (int64_t k = i; k < m; k += stride) {
    const RowState r = rs[k];
    const int t = nidx[k];
    o.resid[t] = r.r;
    o.w[t] = r.w0;
    if (pair[k]) {
      o.resid[t + 1] = -r.r;
      o.w[t + 1] = r.w1;
    }
  }
  if (i == 0) {
    o.resid[mp] = st->cut_active ? st->rc : 0.0;
    o.w[mp] = st->wc;
  }
  if (o.st) {
    static_assert(sizeof(WalkState) % 8 == 0 && sizeof(chap_trace_record) % 8 == 0, "whole words");
    const long long* a = (const long long*)st;
    for (int64_t k = i; k < (int64_t)(sizeof(WalkState) / 8); k += stride) ((long long*)o.st)[k] = a[k];
    const long long* b = (const long long*)trace;
    for (int64_t k = i; k < iters * (int64_t)(sizeof(chap_trace_record) / 8); k += stride) ((long long*)o.trace)[k] = b[k];
  }
}

// Best positive score overall and among non-tabu variables of the columns the
// pass did not record itself (from C.scan_from on), ties to the lowest
// original index; one record per workgroup. The pending copy of a new
// incumbent (flagged by the previous iteration, before this iteration's move
// changes x) is done here too for those columns.
//
// With `combine` the long narrow columns' scores are not in s yet: the
// workgroups past argmax_blocks combine their partial bins, one wavefront
// per column (which writes the column's score), beside the scan, which
// skips their index range.
__global__ __launch_bounds__(256) void k_argmax(const WalkCtx* __restrict__ walks, const int32_t* __restrict__ off,
                                                int32_t nw, int32_t combine) {
  int lb;
  const int w_ = block_walk(off, nw, lb);
  if (w_ < 0) return;
  const WalkCtx& C = walks[w_];
  const WalkState* st = C.st;
  const bool active = st->k < st->iters;
  if (lb == 0 && threadIdx.x == 0) snapshot(C.st, active);
  if (!active) return;
  const int64_t k = st->k;
  BestPair best;
  const int ncc = combine ? C.plan.n_chunk_cols : 0;
  const int cq0 = ncc > 0 ? C.plan.chunk_cols[0].col : 0;
  if (lb >= C.argmax_blocks) {
    const int idx = (lb - C.argmax_blocks) * 4 + (int)(threadIdx.x >> 6);
    if (idx < ncc) {
      int q;
      const double v = combine_col(C, idx, threadIdx.x & 63, &q);
      if ((threadIdx.x & 63) == 0 && v > 0.0)
        best.offer(v, gmem(C.P.perm)[q], q, k <= (int64_t)gmem((const int32_t*)C.tabu)[q]);
    }
  } else {
    scan_scores(C, k, st->copy_best != 0, C.scan_from + lb * (int)blockDim.x + (int)threadIdx.x,
                C.argmax_blocks * (int)blockDim.x, best, [&](int q) { return (uint32_t)(q - cq0) < (uint32_t)ncc; });
  }
  block_record<4>(best, C.best + C.group_rec + lb);
}

// ---------------------------------------------------------------------------
// k_step: the rest of an iteration in one launch.
//
// Selection: every workgroup reduces the iteration's best-move records (a few
// hundred to a few thousand of 32 bytes) for itself, so that no kernel boundary
// stands between the choice and its application. Every input of the choice is
// left alone until the walk's last workgroup ends the iteration: the records,
// the snapshot of the iteration and its violated rows, x, xhat and s.
//
// Tabu/aspiration: a tabu overall best is taken only if its move leaves no
// violated row; since a move changes at most one violation per normalised
// entry of its column, that is impossible while V exceeds the column's entry
// count, and the column is only scanned otherwise, then by workgroup 0. The
// others must not change rows that it still reads: those that could share the
// application wait for its choice (one word of the walk state) and then take
// shares of it as they come, workgroup 0 too, so that every share is done whether
// or not a waiting workgroup gave up. Where the outcomes ask for few workgroups
// nobody waits (share_min). With all of it left to workgroup 0 a reweight of 1M
// rows made an iteration 134 us, now 33; a move of 20k rows summed again took 658
// us, now 80.
//
// Application: the move's rows, or the weights of every violated row (a
// reweight), over as many workgroups as their number asks for; the others
// leave. With recompute = 0 the rows are updated as r += a_ij d, exact on
// all-integer data; otherwise each touched row is summed again from scratch so
// the kept residual equals its definition bit for bit.
//
// End of the iteration (objective, cutoff row, incumbent rule, trace, k + 1)
// by one wavefront of the workgroup that finishes last, found by one 64-bit
// atomic that counts workgroups and sums their violation changes; a move of
// one workgroup needs no atomic. No fence: the last workgroup reads nothing
// that another one wrote except that word.
//
// Bound: latency. One launch replaces four (5 us each at the least in a graph:
// selection, application, end, and the scan of s where the pass records its
// best moves itself).
// ---------------------------------------------------------------------------

constexpr int kStepWaves = kStepThreads / kWave;

struct StepSmem {
  MoveRecord rec[kStepWaves];
  int red[kStepWaves];
  long long total;
  unsigned long long word;
  int last;
};

// WalkState::choice. A waiting workgroup asks at most kStepPolls times, half a
// microsecond apart (a scan takes about 1.5 us per 1024 entries), and then leaves.
enum { kChoiceNone = 0, kChoiceAll = 1, kChoiceFree = 2 };  // no move, the overall best, the best not tabu
constexpr int kStepPolls = 4096;
constexpr int kChoiceShift = 22;
constexpr unsigned long long kChoiceShares = (1ull << kChoiceShift) - 1;
__device__ __forceinline__ unsigned long long choice_tag(int64_t k) { return (unsigned long long)(k + 1) << (kChoiceShift + 2); }
__device__ __forceinline__ bool choice_of(unsigned long long word, int64_t k) {
  return word >> (kChoiceShift + 2) == choice_tag(k) >> (kChoiceShift + 2);
}

// The choice of iteration k as workgroup 0 stores it, or -1. Whole workgroup.
__device__ __forceinline__ int step_await(WalkState* st, int64_t k, StepSmem& S) {
  if (threadIdx.x == 0) {
    unsigned long long w = 0;
    for (int i = 0; i < kStepPolls; ++i) {
      w = __hip_atomic_load(&st->choice, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (choice_of(w, k)) break;
      __builtin_amdgcn_s_sleep(16);
    }
    S.word = w;
  }
  __syncthreads();
  return choice_of(S.word, k) ? (int)(S.word >> kChoiceShift) & 3 : -1;
}

// The next share of the application. Whole workgroup.
__device__ __forceinline__ int step_share(WalkState* st, StepSmem& S) {
  __syncthreads();
  if (threadIdx.x == 0) S.word = atomicAdd(&st->choice, 1ull);
  __syncthreads();
  return (int)(S.word & kChoiceShares);
}

// Sum over the workgroup (a thread's violation changes fit 32 bits, and so do
// a wavefront's).
__device__ __forceinline__ long long step_sum(int v, StepSmem& S) {
  v = wave_sum_int(v);
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  __syncthreads();
  if (lane == 0) S.red[wv] = v;
  __syncthreads();
  long long t = 0;
#pragma unroll
  for (int w = 0; w < kStepWaves; ++w) t += S.red[w];
  return t;
}

// Violation change of column q moved by d, one workgroup.
__device__ long long step_violations(const WalkCtx& C, int q, double d, StepSmem& S) {
  const DevProblem& P = C.P;
  const WalkState* st = C.st;
  const double eps = P.eps;
  int mine = 0;
  for (int e = P.col_ptr[q] + (int)threadIdx.x; e < P.col_ptr[q + 1]; e += kStepThreads) {
    const RowState r = C.rs[P.col_row[e]];
    const double r2 = r.r + P.col_val[e] * d;
    mine += viol_change(r.r, r2, eps);
    if (r.w1 >= 0.0f) mine += viol_change(-r.r, -r2, eps);
  }
  long long dv = step_sum(mine, S);
  if (st->cut_active) {
    const double c = P.obj[q];
    if (c != 0.0) dv += viol_change(st->rc, st->rc + c * d, eps);
  }
  return dv;
}

struct StepMove {
  int64_t k;
  int q, j, kind;  // internal and original column (-1: none), trace kind
  double x_old, x_new, score;
  double c;  // objective coefficient of the moved column
};

// What the end of the iteration needs of the state as it was before it, read
// by wavefront 0 of every workgroup while the records arrive (nobody changes
// it before the last workgroup of the walk does).
struct StepState {
  ObjState o;
  WaveExact acc;
  long long inf_V;
  int tenure;
};

// Ends the iteration, one wavefront (the exact objective sum is spread over
// its lanes); lane 0 writes. dV: violation change of the rows.
__device__ __forceinline__ void step_finish(const WalkCtx& C, const StepMove& M, long long dV, StepState& T) {
  WalkState* st = C.st;
  const int lane = threadIdx.x & (kWave - 1);
  const double eps = C.P.eps;
  ObjState& o = T.o;
  o.copy_best = 0;  // a pending copy was done by the kernels before
  o.V += dV;
  const bool exact = C.objacc != nullptr;
  WaveExact& acc = T.acc;
  const double c = M.c;
  if (M.q >= 0) {
    if (c != 0.0) {
      double r2 = 0.0;
      if (exact) {
        double p, e;
        exact_product(c, M.x_new, p, e);
        acc.add(p);
        acc.add(e);
        exact_product(c, M.x_old, p, e);
        acc.add(-p);
        acc.add(-e);
        acc.normalize();
        acc.store(C.objacc);
        o.f = acc.round_nearest();
        if (o.cut_active) r2 = o.cutoff_residual(&acc);
      } else {
        const double d = M.x_new - M.x_old;
        r2 = o.rc + c * d;
        o.f = o.f + c * d;
      }
      if (o.cut_active) {
        o.V += viol_change(o.rc, r2, eps);
        o.rc = r2;
      }
    }
  } else if (M.kind != kStallKind && o.cut_active && o.rc > eps) {
    o.wc = o.wc + 1.0f;
  }
  const long long V = o.V;
  const double f = o.f;
  const long long v_orig = V - ((o.cut_active && o.rc > eps) ? 1 : 0);
  // the next iteration may rescore only the columns of the moved column's
  // rows when this step changed nothing else the scores depend on: no
  // reweight, no cutoff residual change, no incumbent (which moves the
  // cutoff row)
  const int aff = (M.q >= 0 && !(o.cut_active && c != 0.0) && V != 0) ? 1 : 0;
  o.incumbent_check(eps, exact ? &acc : nullptr);
  if (lane != 0) return;
  chap_trace_record* t = C.trace + M.k;
  t->iter = M.k;
  t->var = M.j;
  t->kind = M.kind;
  t->x_old = M.x_old;
  t->x_new = M.x_new;
  t->score = M.score;
  t->viol = V;
  t->obj = f;
  if (M.q >= 0) {
    C.x[M.q] = M.x_new;
    C.tabu[M.q] = (int32_t)(M.k + T.tenure);
    if (v_orig > 0 && v_orig < T.inf_V) {
      st->inf_V = v_orig;
      st->inf_k = M.k;
    }
  }
  o.store(st);
  st->mv_j = M.q;
  st->mv_new = M.x_new;
  st->aff_ok = aff;
  st->dV = 0ull;
  st->k = M.k + 1;
}

// lc: null for an iteration over every column (no admissible move: a
// reweight); else a proposal iteration over nrec records (no admissible move:
// a stall, which makes no reweight and idles the rest of its block). kShare: some
// walk may share an application (the code for it costs a walk of one workgroup
// 0.15 us an iteration).
template <bool kShare>
__global__ __launch_bounds__(kStepThreads) void k_step(const WalkCtx* __restrict__ walks,
                                                       const int32_t* __restrict__ off, int32_t nw,
                                                       const LearnCtx* lc, int32_t nrec) {
  int lb;
  const int w_ = block_walk(off, nw, lb);
  if (w_ < 0) return;
  const WalkCtx& C = walks[w_];
  const DevProblem& P = C.P;
  WalkState* st = C.st;
  const int64_t k = st->sel_k;
  if (k < 0) return;
  __shared__ StepSmem S;
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wv = tid >> 6;
  const double eps = P.eps;
  // ---- selection
  if (!lc) nrec = C.group_rec + C.argmax_blocks + C.argmax_comb;
  StepState T;
  if (wv == 0) {
    T.o.load(st);
    if (C.objacc) T.acc.load(C.objacc);
    T.inf_V = st->inf_V;
    T.tenure = st->tenure;
  }
  BestPair b;
  {
    const gptr<const MoveRecord> rec = gmem((const MoveRecord*)C.best);
    // kU records per thread and step, every load issued before any is used
    constexpr int kU = 4;
    for (int i0 = tid; i0 < nrec; i0 += kU * kStepThreads) {
      MoveRecord r[kU];
#pragma unroll
      for (int u = 0; u < kU; ++u) {
        const int i = min(i0 + u * kStepThreads, nrec - 1);
        r[u].s_all = rec[i].s_all;
        r[u].s_free = rec[i].s_free;
        r[u].j_all = rec[i].j_all;
        r[u].q_all = rec[i].q_all;
        r[u].j_free = rec[i].j_free;
        r[u].q_free = rec[i].q_free;
      }
#pragma unroll
      for (int u = 0; u < kU; ++u) b.offer(r[u]);  // the last record may be offered again
    }
    // wavefronts without a record (and their slots) hold none
    const int used = min(kStepWaves, (nrec + kWave - 1) / kWave);
    if (wv < used) {
      b.wave_reduce();
      if (lane == 0) S.rec[wv] = b.record();
    }
    __syncthreads();
    b = BestPair();
    if (lane < used) b.offer(S.rec[lane]);
    b.wave_reduce();
  }
  StepMove M{k, -1, -1, lc ? kStallKind : 2, 0.0, 0.0, 0.0, 0.0};
  const int qa = b.all.q;
  const gptr<const double> x = gmem((const double*)C.x), xhat = gmem((const double*)C.xhat),
                           sc = gmem((const double*)C.s);
  // the workgroups that the move of a column of deg entries, or (none) an
  // outcome without a move, is divided among. A row summed again: by a wavefront
  // while that leaves few rounds, else by kResidualLanes lanes (a short row leaves
  // most of a wavefront idle)
  auto deg_of = [&](int q) { return P.col_ptr[q + 1] - P.col_ptr[q]; };
  auto rows_by_wave = [&](int deg) { return deg <= C.apply_blocks * kStepWaves * 2; };
  auto blocks_of = [&](bool none, int deg) {
    if (none) return lc ? 1 : C.apply_blocks;
    const int per = C.recompute ? (rows_by_wave(deg) ? kStepWaves : kStepThreads / kResidualLanes) : kStepThreads;
    return max(1, min(C.apply_blocks, (deg + per - 1) / per));
  };
  bool solo = false;    // workgroup 0 does the whole iteration
  bool shares = false;  // the application's shares are taken as the workgroups come
  if (qa >= 0 && b.all.j == b.free.j) {
    M.q = qa;
    M.j = b.all.j;
    M.kind = 0;
  } else if (qa >= 0) {
    const int64_t V = st->sel_V;
    const int deg = deg_of(qa);
    const int64_t bound = 2 * (int64_t)deg + 1;
    int choice = b.free.q >= 0 ? kChoiceFree : kChoiceNone;
    if (__builtin_expect(V <= bound, 0)) {  // out of the way of the other iterations' code
      const bool none = b.free.q < 0;
      const int least = share_min(C);
      int most = 1;
      if (kShare && C.apply_blocks >= least)
        most = max(blocks_of(false, deg), blocks_of(none, none ? 0 : deg_of(b.free.q)));
      shares = most >= least;
      solo = !shares;
      if (lb >= (shares ? most : 1)) return;
      if (lb == 0) {
        if (V + step_violations(C, qa, xhat[qa] - x[qa], S) == 0) choice = kChoiceAll;
        if (shares && tid == 0)
          __hip_atomic_store(&st->choice, choice_tag(k) | (unsigned long long)choice << kChoiceShift, __ATOMIC_RELAXED,
                             __HIP_MEMORY_SCOPE_AGENT);
      } else {
        choice = step_await(st, k, S);
        if (choice < 0) return;
      }
    }
    if (choice == kChoiceAll) {
      M.q = qa;
      M.j = b.all.j;
      M.kind = 1;
    } else if (choice == kChoiceFree) {
      M.q = b.free.q;
      M.j = b.free.j;
      M.kind = 0;
    }
  }
  if (M.q >= 0 && lc) M.kind += kProposalKind;
  // ---- application
  int beg = 0, end = 0;
  if (M.q >= 0) {  // one round of loads
    beg = P.col_ptr[M.q];
    end = P.col_ptr[M.q + 1];
    M.x_old = x[M.q];
    M.x_new = xhat[M.q];
    M.score = sc[M.q];
    M.c = gmem(P.obj)[M.q];
  }
  const bool resum = M.q >= 0 && C.recompute;
  const bool by_wave = resum && rows_by_wave(end - beg);
  const int nb = solo ? 1 : blocks_of(M.q < 0, end - beg);
  RowState* rs = C.rs;
  // one share of the application; this thread's violation changes
  auto apply = [&](int share) {
    const int gt = share * kStepThreads + tid, gs = nb * kStepThreads;
    int dv = 0;  // this thread's violation changes
    if (resum) {
      // every touched row is summed again in its stored order (products side by
      // side, added in entry order); its state and right-hand side q, rhs
      auto update = [&](int i, RowState q, double rhs, double acc) {
        const double r2 = acc - rhs;
        rs[i].r = r2;
        if (C.grow) C.grow[i].r = (int32_t)r2;
        dv += viol_change(q.r, r2, eps);
        if (q.w1 >= 0.0f) dv += viol_change(-q.r, -r2, eps);
      };
      if (by_wave) {
        for (int e = __builtin_amdgcn_readfirstlane(beg + gt / kWave); e < end; e += gs / kWave) {
          const int i = __builtin_amdgcn_readfirstlane(P.col_row[e]);
          const RowState q = rs[i];
          const double rhs = P.row_rhs[i];
          const double acc = wave_row_sum(P, C.x, __builtin_amdgcn_readfirstlane(P.row_ptr[i]),
                                          __builtin_amdgcn_readfirstlane(P.row_ptr[i + 1]), M.q, M.x_new);
          if (lane == 0) update(i, q, rhs, acc);
        }
      } else {
        const int g = gt & (kResidualLanes - 1);
        for (int e = beg + gt / kResidualLanes; e < end; e += gs / kResidualLanes) {
          const int i = P.col_row[e];
          double acc = 0.0;
          const int rb = P.row_ptr[i], re = P.row_ptr[i + 1];
          for (int e0 = rb; e0 < re; e0 += kResidualLanes) {
            const int f = e0 + g;
            double prod = 0.0;
            if (f < re) {
              const int c = P.row_col[f];
              prod = P.row_val[f] * ((c == M.q) ? M.x_new : x[c]);
            }
            const int cnt = min(kResidualLanes, re - e0);
            for (int t = 0; t < cnt; ++t) acc = acc + __shfl(prod, t, kResidualLanes);
          }
          if (g == 0) update(i, rs[i], P.row_rhs[i], acc);
        }
      }
    } else if (M.q >= 0) {
      const double d = M.x_new - M.x_old;
      for (int e = beg + gt; e < end; e += gs) {
        const int i = P.col_row[e];
        const RowState q = rs[i];
        const double r2 = q.r + P.col_val[e] * d;
        rs[i].r = r2;
        if (C.grow) C.grow[i].r = (int32_t)r2;
        dv += viol_change(q.r, r2, eps);
        if (q.w1 >= 0.0f) dv += viol_change(-q.r, -r2, eps);
      }
    } else if (M.kind != kStallKind) {
      constexpr int kU = 4;  // rows per thread and step, loaded before any is used
      for (int64_t i0 = gt; i0 < P.ms; i0 += (int64_t)kU * gs) {
        RowState q[kU];
#pragma unroll
        for (int u = 0; u < kU; ++u) {
          const int64_t i = i0 + (int64_t)u * gs;
          q[u] = i < P.ms ? rs[i] : RowState{0.0, 0.0f, -1.0f};
        }
#pragma unroll
        for (int u = 0; u < kU; ++u) {
          const int64_t i = i0 + (int64_t)u * gs;
          if (q[u].r > eps) {
            rs[i].w0 = q[u].w0 + 1.0f;
            if (C.grow) C.grow[i].w0 = (uint16_t)(q[u].w0 + 1.0f);
          }
          if (q[u].w1 >= 0.0f && -q[u].r > eps) {
            rs[i].w1 = q[u].w1 + 1.0f;
            if (C.grow) C.grow[i].w1 = (uint16_t)(q[u].w1 + 1.0f);
          }
        }
      }
    }
    return dv;
  };
  // adds a share's violation changes; true where all shares are done, with the sum
  auto all_done = [&](int dv, long long& dV) {
    dV = step_sum(dv, S);
    if (nb == 1) return true;
    if (tid == 0) {
      const unsigned long long mine = ((unsigned long long)dV << 16) + 1ull;
      const unsigned long long sum = atomicAdd(&st->dV, mine) + mine;
      S.last = (int)(sum & 0xFFFFull) == nb;
      S.total = (long long)sum >> 16;
    }
    __syncthreads();
    dV = S.total;
    return S.last != 0;
  };
  long long dV;
  int share = kShare && shares ? step_share(st, S) : lb;
  while (true) {
    if (share >= nb) return;
    if (all_done(apply(share), dV)) break;
    if (!kShare || __builtin_expect(!shares, 1)) return;
    share = step_share(st, S);
  }
  // ---- the workgroup of the last share ends the iteration
  if (wv != 0) return;
  step_finish(C, M, dV, T);
  if (lc && lane == 0) {
    if (M.q >= 0) {
      learned::after_move(C, *lc, M.q, M.x_new, k);
    } else {
      lc->ls->stalls += 1;
      lc->ls->idle = 1;
    }
  }
}

__global__ __launch_bounds__(64) void k_subset_none(const WalkCtx* __restrict__ walks,
                                                    const LearnCtx* __restrict__ lc) {
  WalkState* st = walks[0].st;
  if (threadIdx.x == 0) snapshot(st, st->k < st->iters && !lc->ls->idle);
}

__global__ __launch_bounds__(256) void k_copy_best(const double* __restrict__ x, double* __restrict__ best_x,
                                                   const WalkState* st, int32_t n) {
  if (!st->copy_best) return;
  const int gs = gridDim.x * blockDim.x;
  for (int j = blockIdx.x * blockDim.x + threadIdx.x; j < n; j += gs) best_x[j] = x[j];
}

__device__ __forceinline__ int copy_blocks(int32_t n) { return max(1, min((int)(((int64_t)n + 255) / 256), 256)); }

__global__ __launch_bounds__(256) void k_copy_best_batch(const WalkCtx* __restrict__ walks,
                                                         const int32_t* __restrict__ off, int32_t nw) {
  int lb;
  const int w_ = block_walk(off, nw, lb);
  if (w_ < 0) return;
  const WalkCtx& C = walks[w_];
  if (!C.st->copy_best) return;
  const int gs = copy_blocks(C.P.n) * blockDim.x;
  for (int q = lb * blockDim.x + threadIdx.x; q < C.P.n; q += gs) C.best_x[q] = C.x[q];
}

__global__ __launch_bounds__(256) void k_gather(const int32_t* __restrict__ perm, const double* __restrict__ src,
                                                double* __restrict__ dst, int32_t n) {
  const int q = blockIdx.x * blockDim.x + threadIdx.x;
  if (q < n) dst[q] = src[perm[q]];
}

// da[j] = a[inv[j]], db[j] = b[inv[j]] (internal order -> caller's order),
// written in the caller's order so that the stores are coalesced.
__global__ __launch_bounds__(256) void k_gather2(const int32_t* __restrict__ inv, const double* __restrict__ a,
                                                 const double* __restrict__ b, double* __restrict__ da,
                                                 double* __restrict__ db, int32_t n) {
  const int j = blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= n) return;
  const int q = inv[j];
  da[j] = a[q];
  db[j] = b[q];
}

// Planned permutation, first pass: workgroup c sorts input chunk c by output
// block in LDS, then writes the sorted chunk to its runs' staging slots
// (consecutive slots within a run). kArrays (1 or 2) arrays side by side,
// sharing the plan's index loads.
constexpr int kPermRunsThreads = 1024;
constexpr int kPermPlaceThreads = 512;
template <int kArrays>
__global__ __launch_bounds__(kPermRunsThreads) void k_perm_runs(PermPlan pl, const double* __restrict__ in0,
                                                                const double* __restrict__ in1,
                                                                double* __restrict__ st0, double* __restrict__ st1) {
  __shared__ double lds[kArrays][kPermChunk];
  constexpr int kU = kPermChunk / kPermRunsThreads;
  const double* in[2] = {in0, in1};
  double* st[2] = {st0, st1};
  const int64_t base = (int64_t)blockIdx.x * kPermChunk;
  const int cnt = (int)min((int64_t)kPermChunk, (int64_t)pl.n - base);
  double v[kArrays][kU];
  int pos[kU];
#pragma unroll
  for (int u = 0; u < kU; ++u) {
    const int t = threadIdx.x + u * kPermRunsThreads;
    if (t < cnt) {
      pos[u] = pl.lpos[base + t];
#pragma unroll
      for (int a = 0; a < kArrays; ++a) v[a][u] = in[a][base + t];
    }
  }
#pragma unroll
  for (int u = 0; u < kU; ++u)
    if (threadIdx.x + u * kPermRunsThreads < cnt)
#pragma unroll
      for (int a = 0; a < kArrays; ++a) lds[a][pos[u]] = v[a][u];
  __syncthreads();
#pragma unroll
  for (int u = 0; u < kU; ++u) {
    const int t = threadIdx.x + u * kPermRunsThreads;
    if (t < cnt) pos[u] = pl.sdst[base + t];
  }
#pragma unroll
  for (int u = 0; u < kU; ++u) {
    const int t = threadIdx.x + u * kPermRunsThreads;
    if (t < cnt)
#pragma unroll
      for (int a = 0; a < kArrays; ++a) st[a][pos[u]] = lds[a][t];
  }
}

// Second pass: workgroup b places output block b's values (contiguous in
// staging) at their offsets in LDS and writes the block, kArrays arrays side
// by side. With xc, the byte copy of array 0 as in k_stage_x.
template <int kArrays>
__global__ __launch_bounds__(kPermPlaceThreads) void k_perm_place(PermPlan pl, const double* __restrict__ st0,
                                                                  const double* __restrict__ st1,
                                                                  double* __restrict__ out0, double* __restrict__ out1,
                                                                  int8_t* __restrict__ xc, WalkState* ws,
                                                                  uint32_t epoch, SingleInit init) {
  if (blockIdx.x == 0 && threadIdx.x == 0 && init.cutoff_w) single_state(ws, init);
  __shared__ double lds[kArrays][kPermBlock];
  constexpr int kU = kPermBlock / kPermPlaceThreads;
  const double* st[2] = {st0, st1};
  double* out[2] = {out0, out1};
  const int64_t base = (int64_t)blockIdx.x * kPermBlock;
  const int cnt = (int)min((int64_t)kPermBlock, (int64_t)pl.n - base);
  double v[kArrays][kU];
  int pos[kU];
#pragma unroll
  for (int u = 0; u < kU; ++u) {
    const int t = threadIdx.x + u * kPermPlaceThreads;
    if (t < cnt) {
      pos[u] = pl.dl[base + t];
#pragma unroll
      for (int a = 0; a < kArrays; ++a) v[a][u] = st[a][base + t];
    }
  }
#pragma unroll
  for (int u = 0; u < kU; ++u)
    if (threadIdx.x + u * kPermPlaceThreads < cnt)
#pragma unroll
      for (int a = 0; a < kArrays; ++a) lds[a][pos[u]] = v[a][u];
  __syncthreads();
  bool misfit = false;
#pragma unroll
  for (int u = 0; u < kU; ++u) {
    const int t = threadIdx.x + u * kPermPlaceThreads;
    if (t < cnt) {
#pragma unroll
      for (int a = 0; a < kArrays; ++a) out[a][base + t] = lds[a][t];
      if (xc) {
        const double x = lds[0][t];
        const bool fits = x == floor(x) && x >= -128.0 && x <= 127.0;
        xc[base + t] = fits ? (int8_t)x : (int8_t)0;
        misfit = misfit || !fits;
      }
    }
  }
  if (misfit) ws->x_misfit = epoch;  // every writer stores the same value
}

inline int blocks_for(int64_t work, int cap) {
  int64_t b = (work + 255) / 256;
  if (b < 1) b = 1;
  if (b > cap) b = cap;
  return (int)b;
}


// ---------------------------------------------------------------------------
// Affected rescoring. The best shift of column q depends on x_q, its bounds,
// the residuals and weights of its rows and, when the cutoff row is active,
// that row's residual and weight. A move of column j* with no reweight and
// no change of the cutoff row changes only the residuals of j*'s rows, so
// only x_j* and the columns sharing one of those rows need a new score.
// ---------------------------------------------------------------------------

// One workgroup: lists the affected columns, splits the list into its
// lane-group columns and the rest, with the rest's subset chunk offsets
// (ceil(entries / kSubsetChunk) chunks per binary or narrow column, none for a
// general one), and skips the full pass. When the step was not a plain move,
// the list is longer than cap, a listed column has no subset form, or the
// chunks exceed sub_cap, the iteration scores every column: through the
// split of all columns when there is one, else through the full pass. Points
// the subset record and the group list at the lists it takes and clears the
// count.
__global__ __launch_bounds__(256) void k_aff_plan(const WalkCtx* __restrict__ walks, LearnCtx* __restrict__ lc,
                                                  AffLists A) {
  const WalkCtx& C = walks[0];
  WalkState* st = C.st;
  LearnCtx& L = *lc;
  if (st->k >= st->iters) return;
  __shared__ int wsum[4];
  __shared__ int carry, bad, n_other, n_s, n_mark;
  const int tid = threadIdx.x;
  // the affected columns: the moved column and the columns of its rows
  // (stamp[q] = iteration + 1 marks a column already listed; stamps are
  // cleared when the walk starts); at most cap are listed, all are counted.
  // The rows' entries are taken as one flat range (prefix of the row
  // lengths in LDS), so every thread's stamps are in flight at once; a
  // column of more than kAffRows rows is left to the full scoring.
  __shared__ int rpre[kAffRows + 1];
  __shared__ int rrow[kAffRows];
  __shared__ int lst[kRescoreCapMax];  // the affected list
  __shared__ int olst[kRescoreCapMax];  // its columns outside the lane-group range
  if (tid == 0) n_mark = 0;
  __syncthreads();
  if (st->aff_ok) {
    const DevProblem& P = C.P;
    const int32_t tag = (int32_t)st->k + 1;
    const int q0 = st->mv_j;
    const int beg = P.col_ptr[q0], deg = P.col_ptr[q0 + 1] - beg;
    if (deg > kAffRows) {
      if (tid == 0) n_mark = A.cap + 1;
    } else {
      const int lane = tid & 63, wv = tid >> 6;
      int len = 0;
      if (tid < deg) {
        const int i = P.col_row[beg + tid];
        rrow[tid] = i;
        len = P.row_ptr[i + 1] - P.row_ptr[i];
      }
      int inc = len;
#pragma unroll
      for (int o = 1; o < kWave; o <<= 1) {
        const int y = __shfl_up(inc, o, kWave);
        if (lane >= o) inc += y;
      }
      if (lane == 63) wsum[wv] = inc;
      __syncthreads();
      int off = inc - len;
      for (int k = 0; k < wv; ++k) off += wsum[k];
      if (tid < deg) rpre[tid] = off;
      if (tid == deg - 1) rpre[deg] = off + len;
      if (deg == 0 && tid == 0) rpre[0] = 0;
      __syncthreads();
      const int total = rpre[deg];
      auto push = [&](int q) {
        if (atomicExch(&A.stamp[q], tag) != tag) {
          const int k = atomicAdd(&n_mark, 1);
          if (k < A.cap) lst[k] = q;
        }
      };
      if (tid == 0) push(q0);
      for (int f = tid; f < total; f += 256) {
        int lo = 0, hi = deg - 1;
        while (lo < hi) {
          const int mid = (lo + hi + 1) >> 1;
          if (rpre[mid] <= f)
            lo = mid;
          else
            hi = mid - 1;
        }
        push(P.row_col[P.row_ptr[rrow[lo]] + (f - rpre[lo])]);
      }
    }
  }
  __syncthreads();
  const int n_list = st->aff_ok ? n_mark : 0;
  const bool listed = st->aff_ok && n_list <= A.cap;
  const int g0 = C.plan.grp_col[0], g1 = C.plan.grp_col[kGroupClasses];
  if (tid == 0) {
    carry = 0;
    bad = 0;
    n_other = 0;
    n_s = 0;
  }
  __syncthreads();
  if (listed) {
    for (int i = tid; i < n_list; i += 256) {
      const int q = lst[i];
      if (q >= g0 && q < g1) {
        A.slist[atomicAdd(&n_s, 1)] = q;
      } else {
        if (L.cls[q] == SUB_NONE) bad = 1;
        const int k = atomicAdd(&n_other, 1);
        olst[k] = q;
        A.olist[k] = q;
      }
    }
    __syncthreads();
    const int n_o = n_other;
    const int lane = tid & 63, wv = tid >> 6;
    for (int base = 0; base < n_o; base += 256) {
      const int i = base + tid;
      int c = 0;
      if (i < n_o) {
        const int q = olst[i];
        const uint8_t cl = L.cls[q];
        const int e = C.P.col_ptr[q + 1] - C.P.col_ptr[q];
        c = (cl == SUB_GENERAL || cl == SUB_NONE) ? 0 : max(1, (e + kSubsetChunk - 1) / kSubsetChunk);
      }
      int inc = c;
#pragma unroll
      for (int o = 1; o < kWave; o <<= 1) {
        const int y = __shfl_up(inc, o, kWave);
        if (lane >= o) inc += y;
      }
      if (lane == 63) wsum[wv] = inc;
      __syncthreads();
      int off = carry + inc - c;
      for (int k = 0; k < wv; ++k) off += wsum[k];
      if (i < n_o) A.ooff[i] = off;
      __syncthreads();
      if (tid == 255) carry = off + c;
      __syncthreads();
    }
  }
  if (tid != 0) return;
  const bool subset = listed && !bad && carry <= A.sub_cap;
  if (subset) {
    A.ooff[n_other] = carry;
    L.sel[0] = A.olist;
    L.sub_off = A.ooff;
    L.ls->tk[0].count = n_other;
    L.ls->tk[0].chunks = carry;
    L.ls->idle = 0;
    A.run->slist = A.slist;
    A.run->n_s = n_s;
    st->pass_skip = 1;
    st->aff_iters += 1;
  } else if (A.full_olist) {
    L.sel[0] = const_cast<int32_t*>(A.full_olist);
    L.sub_off = const_cast<int32_t*>(A.full_ooff);
    L.ls->tk[0].count = A.n_full_o;
    L.ls->tk[0].chunks = A.full_chunks;
    L.ls->idle = 0;
    A.run->n_s = -1;
    st->pass_skip = 1;
  } else {
    L.ls->tk[0].count = 0;
    L.ls->tk[0].chunks = 0;
    L.ls->idle = 1;
    A.run->n_s = 0;
    st->pass_skip = 0;
  }
}


// ---------------------------------------------------------------------------
// Diversity restarts of batched walks (section 3.1 "Parallel Tabu Search
// Instances": walks whose points come too close to another walk's restart).
// ---------------------------------------------------------------------------

__global__ __launch_bounds__(64) void k_set_iters(const WalkCtx* __restrict__ walks, int32_t nw, int64_t iters_end) {
  const int w = blockIdx.x * blockDim.x + threadIdx.x;
  if (w < nw) walks[w].st->iters = iters_end;
}

// One workgroup per task: discrete variables of the task's column range at
// which the two points differ, added into dist[pair].
__global__ __launch_bounds__(256) void k_hamming(const HamTask* __restrict__ tasks, int32_t* __restrict__ dist) {
  const HamTask T = tasks[blockIdx.x];
  __shared__ long long red[4];
  long long c = 0;
  for (int q = T.begin + (int)threadIdx.x; q < T.end; q += (int)blockDim.x)
    c += (T.is_int[q] != 0 && T.xa[q] != T.xb[q]) ? 1 : 0;
  c = block_sum_ll(c, red);
  if (threadIdx.x == 0 && c != 0) atomicAdd(&dist[T.pair], (int32_t)c);
}

__global__ void k_restart_fix(WalkState* st, RestartKeep keep) {
  if (threadIdx.x != 0) return;
  const bool improved = st->has_best && st->copy_best;  // the restart point is a new incumbent
  if (!improved) {
    st->has_best = keep.has_best;
    st->fbest = keep.fbest;
    st->copy_best = 0;
  }
  st->k = keep.k;
  const bool fresh = st->inf_k != -2;  // the restart point is infeasible
  if (keep.inf_k != -2 && (!fresh || keep.inf_V <= st->inf_V)) {
    st->inf_V = keep.inf_V;
    st->inf_k = keep.inf_k;
  } else if (fresh) {
    st->inf_k = keep.k - 1;
  }
}

}  // namespace

namespace {

inline int32_t residual_groups(int32_t ms) { return (int32_t)(((int64_t)ms * kResidualLanes + 255) / 256); }

// k_residual's workgroups: the rows' lane groups, then the long rows' wavefronts
inline dim3 residual_grid(const DevProblem& P) {
  return dim3((unsigned)(residual_groups(P.ms) + (P.n_long_rows + 3) / 4));
}

}  // namespace

// The x-block kernel where the problem has its row layout and the call has
// a byte copy of x (its own fallback covers a point that does not fit).
inline bool residual_blocked(const DevProblem& P, const int8_t* xc) { return P.rb_ent != nullptr && xc != nullptr; }

inline dim3 residual_blocked_grid(const DevProblem& P) {
  return dim3((unsigned)(((int64_t)P.ms + P.rb_rows - 1) / P.rb_rows));
}

hipError_t launch_residual_unit(const DevProblem& P, const uint8_t* pair, const double* x, const int8_t* xc,
                                const WalkState* st, uint32_t epoch, RowState* rs, GatherRow* grow,
                                hipStream_t stream) {
  if (P.ms > 0 && residual_blocked(P, xc))
    hipLaunchKernelGGL(k_residual_blocked<kWeightsUnit>, residual_blocked_grid(P), dim3(kResBlockedThreads), 0,
                       stream, P, x, xc, st, epoch, rs, nullptr, pair, nullptr, grow);
  else if (P.ms > 0)
    hipLaunchKernelGGL(k_residual<kWeightsUnit>, residual_grid(P), dim3(256), 0, stream, P,
                       residual_groups(P.ms), x, xc, st, epoch, rs,
                       nullptr, pair, nullptr, grow);
  return hipGetLastError();
}

hipError_t launch_residual_scatter(const DevProblem& P, const int32_t* nidx, const uint8_t* pair, const float* w,
                                   const double* x, const int8_t* xc, const WalkState* st, uint32_t epoch,
                                   RowState* rs, hipStream_t stream, GatherRow* grow) {
  if (P.ms > 0 && residual_blocked(P, xc))
    hipLaunchKernelGGL(k_residual_blocked<kWeightsScatter>, residual_blocked_grid(P), dim3(kResBlockedThreads), 0,
                       stream, P, x, xc, st, epoch, rs, nidx, pair, w, grow);
  else if (P.ms > 0)
    hipLaunchKernelGGL(k_residual<kWeightsScatter>, residual_grid(P), dim3(256), 0, stream, P,
                       residual_groups(P.ms), x, xc, st, epoch,
                       rs, nidx, pair, w, grow);
  return hipGetLastError();
}

hipError_t launch_start_point(const DevProblem& P, uint64_t seed, double* x, int8_t* xc, hipStream_t stream) {
  if (P.n > 0) hipLaunchKernelGGL(k_start_point, dim3((P.n + 255) / 256), dim3(256), 0, stream, P, seed, x, xc);
  return hipGetLastError();
}

hipError_t launch_stage_x(const int32_t* perm, const double* src, double* dst, int8_t* xc, WalkState* st,
                          uint32_t epoch, int32_t n, const SingleInit& init, hipStream_t stream) {
  if (n > 0 || init.cutoff_w)
    hipLaunchKernelGGL(k_stage_x, dim3((unsigned)std::max(1, (n + 255) / 256)), dim3(256), 0, stream, perm, src, dst,
                       xc, st, epoch, n, init);
  return hipGetLastError();
}

hipError_t launch_state_init(const DevProblem& P, const double* x, const RowState* rs, WalkState* st,
                             double* partial, uint32_t* ticket, long long* objacc, int64_t iters, int32_t tenure,
                             int32_t obj_integral, double cutoff_rhs, const float* cutoff_w, int check_incumbent,
                             int count_violated, hipStream_t stream) {
  // a single pass needs neither V nor, without a cutoff row, f
  const int32_t need_v = (check_incumbent || count_violated) ? 1 : 0;
  const int32_t need_obj = (check_incumbent || std::isfinite(cutoff_rhs)) ? 1 : 0;
  const int64_t work = std::max<int64_t>(need_obj ? P.n : 0, need_v ? P.ms : 0);
  const int blocks = work > 0 ? blocks_for((work + 3) / 4, kInitBlocks) : 1;
  hipLaunchKernelGGL(k_state_init, dim3(blocks), dim3(256), 0, stream, P, x, rs, st, partial, ticket, objacc, iters,
                     tenure, obj_integral, cutoff_rhs, cutoff_w, check_incumbent, need_obj, need_v);
  return hipGetLastError();
}

static hipError_t launch_step(const BatchLaunch& L, const LearnCtx* lc, int32_t nrec, hipStream_t stream) {
  const dim3 grid((unsigned)L.grid[KS_STEP]);
  if (L.step_shares)
    hipLaunchKernelGGL(k_step<true>, grid, dim3(kStepThreads), 0, stream, L.walks, L.off[KS_STEP], L.nw, lc, nrec);
  else
    hipLaunchKernelGGL(k_step<false>, grid, dim3(kStepThreads), 0, stream, L.walks, L.off[KS_STEP], L.nw, lc, nrec);
  return hipGetLastError();
}

hipError_t launch_walk_step(const BatchLaunch& L, hipStream_t stream, bool combine) {
  const int nw = L.nw;
  const int32_t comb = (combine && pass_defers_combine(L)) ? 1 : 0;
  if (L.total[KS_ARGMAX] > 0)
    hipLaunchKernelGGL(k_argmax, dim3((unsigned)L.grid[KS_ARGMAX]), dim3(256), 0, stream, L.walks, L.off[KS_ARGMAX],
                       nw, comb);
  return launch_step(L, nullptr, 0, stream);
}

hipError_t launch_subset_step(const BatchLaunch& L, const LearnCtx* lc, int32_t nrec, hipStream_t stream) {
  return launch_step(L, lc, nrec, stream);
}

hipError_t launch_subset_none(const WalkCtx* C, const LearnCtx* L, hipStream_t s) {
  hipLaunchKernelGGL(k_subset_none, dim3(1), dim3(64), 0, s, C, L);
  return hipGetLastError();
}

hipError_t launch_affected(const WalkCtx* C, LearnCtx* L, const AffLists& A, hipStream_t s) {
  hipLaunchKernelGGL(k_aff_plan, dim3(1), dim3(256), 0, s, C, L, A);
  return hipGetLastError();
}

hipError_t launch_set_iters(const BatchLaunch& L, int64_t iters_end, hipStream_t s) {
  hipLaunchKernelGGL(k_set_iters, dim3((unsigned)((L.nw + 63) / 64)), dim3(64), 0, s, L.walks, L.nw, iters_end);
  return hipGetLastError();
}

hipError_t launch_hamming(const HamTask* tasks, int32_t ntasks, int32_t* dist, hipStream_t s) {
  if (ntasks > 0) hipLaunchKernelGGL(k_hamming, dim3((unsigned)ntasks), dim3(256), 0, s, tasks, dist);
  return hipGetLastError();
}

hipError_t launch_restart_fix(WalkState* st, const RestartKeep& keep, hipStream_t s) {
  hipLaunchKernelGGL(k_restart_fix, dim3(1), dim3(64), 0, s, st, keep);
  return hipGetLastError();
}

hipError_t launch_copy_best_batch(const BatchLaunch& L, hipStream_t stream) {
  hipLaunchKernelGGL(k_copy_best_batch, dim3((unsigned)L.grid[KS_COPY]), dim3(256), 0, stream, L.walks,
                     L.off[KS_COPY], L.nw);
  return hipGetLastError();
}

hipError_t launch_gather(const int32_t* perm, const double* src, double* dst, int32_t n, hipStream_t stream) {
  if (n > 0) hipLaunchKernelGGL(k_gather, dim3((n + 255) / 256), dim3(256), 0, stream, perm, src, dst, n);
  return hipGetLastError();
}

hipError_t launch_stage_x_plan(const PermPlan& plan, const double* src, double* dst, int8_t* xc, WalkState* st,
                               uint32_t epoch, double* stage, const SingleInit& init, hipStream_t stream) {
  if (plan.n > 0) {
    const unsigned nc = (unsigned)((plan.n + kPermChunk - 1) / kPermChunk);
    const unsigned nb = (unsigned)((plan.n + kPermBlock - 1) / kPermBlock);
    hipLaunchKernelGGL(k_perm_runs<1>, dim3(nc), dim3(kPermRunsThreads), 0, stream, plan, src, nullptr, stage,
                       nullptr);
    hipLaunchKernelGGL(k_perm_place<1>, dim3(nb), dim3(kPermPlaceThreads), 0, stream, plan, stage, nullptr, dst,
                       nullptr, xc, st, epoch, init);
  }
  return hipGetLastError();
}

hipError_t launch_gather2_plan(const PermPlan& plan, const double* a, const double* b, double* da, double* db,
                               double* stage, hipStream_t stream) {
  if (plan.n > 0) {
    const unsigned nc = (unsigned)((plan.n + kPermChunk - 1) / kPermChunk);
    const unsigned nb = (unsigned)((plan.n + kPermBlock - 1) / kPermBlock);
    double* stage_b = stage + plan.n;
    hipLaunchKernelGGL(k_perm_runs<2>, dim3(nc), dim3(kPermRunsThreads), 0, stream, plan, a, b, stage, stage_b);
    hipLaunchKernelGGL(k_perm_place<2>, dim3(nb), dim3(kPermPlaceThreads), 0, stream, plan, stage, stage_b, da, db,
                       nullptr, nullptr, 0u, SingleInit());
  }
  return hipGetLastError();
}

hipError_t launch_gather2(const int32_t* inv, const double* a, const double* b, double* da, double* db, int32_t n,
                          hipStream_t stream) {
  if (n > 0) hipLaunchKernelGGL(k_gather2, dim3((n + 255) / 256), dim3(256), 0, stream, inv, a, b, da, db, n);
  return hipGetLastError();
}

hipError_t launch_state_out(const DevProblem& P, const int32_t* nidx, const uint8_t* pair, int32_t mp,
                            const WalkCtx& c, int64_t iters, const StateOut& o, hipStream_t stream) {
  hipLaunchKernelGGL(k_state_out, dim3(blocks_for(std::max(1, std::max(P.n, P.ms)), 4096)), dim3(256), 0, stream, P.n,
                     P.ms, mp, P.perm, nidx, pair, c.x, c.best_x, c.rs, c.st, c.trace, iters, o);
  return hipGetLastError();
}

hipError_t launch_copy_best(const double* x, double* best_x, WalkState* st, int32_t n, hipStream_t stream) {
  hipLaunchKernelGGL(k_copy_best, dim3(blocks_for(n, 1024)), dim3(256), 0, stream, x, best_x, st, n);
  return hipGetLastError();
}

}  // namespace chap
