// Learned candidate proposal for one tabu walk on gfx950.
//
// The paper scores every column exactly in every iteration (section 3.1,
// "Scoring Functions"). Here a network ranks the columns and only its top K
// get the exact best shift; a full pass every few iterations (or after a
// proposal iteration without an admissible move) is the fallback, the judge
// of the network and the source of its training pairs. Every move taken is
// still an exact best shift under the tabu and aspiration rules.
//
// Stored feature rows (16 bfloat16 per column, internal order):
//   0 weighted violated share   sum_{viol} w / sum w over the column's rows
//   1 log2(1 + stored entries)
//   2 c_j / max |c|
//   3 s_last / sum w, clamped to [-4, 4] (score at the last full pass)
//   4 binary  5 general integer  6 continuous
//   7 position (x - l) / (u - l) (0.5 for an infinite bound, 0 for l = u)
//   8 log2(1 + min(u - l, 2^20)) (20 for an infinite bound)
//   9 unweighted violated share
//  10 violated mass: sum_{viol} |a| min(r, 1000) / (1000 sum |a|)
//  11 sign(xhat_last - x)
//  12..13 (storage) int32 iteration of the column's last move
//  15 log2(1 + moves of the column)
// Inputs 12..14 of the network are formed when a row is read: the tabu age
// min(k - last move, 1024) / 1024, min(k - last full pass, 64) / 64, and the
// violated fraction V / m'. Inputs 0, 3, 9, 10 are refreshed at full passes
// only; 7, 11, 12, 15 change with the column's own moves. Every value is
// computed in FP64 and rounded once to bfloat16.
//
// Top-K: scores become order-preserving 32-bit keys (0 = never proposed); a
// three-digit radix select (11, 11, 10 bits) finds the K-th key, and an
// order-preserving compaction lists the selected columns in ascending
// internal index (equal keys: lowest index first). Each kernel of the select
// re-derives the digits chosen so far from the histograms of the earlier
// kernels (a few kilobytes from L2), so no single-workgroup kernel sits
// between them; a last one puts the list together.

#include <climits>
#include <cmath>

#include "chap_internal.h"
#include "learned_rows.h"
#include "mlp_core.h"
#include "move_best.h"

namespace chap {
namespace {

using namespace mlp;
using namespace learned;

constexpr int kBlock = 256;

// Order-preserving key of a finite score; never 0.
__device__ __forceinline__ uint32_t order_key(float y) {
  const uint32_t u = __float_as_uint(y);
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

__device__ __forceinline__ bool active(const WalkState* st, const LearnState* ls) {
  return st->k < st->iters && !ls->idle;
}

// Inputs 13 and 14, the same for every column at one iteration.
struct Globals {
  short since;  // bfloat16 bits of min(k - k_last_full, 64) / 64
  short vfrac;  // bfloat16 bits of V / m'
};

__device__ __forceinline__ Globals globals(int64_t k, int64_t k_last_full, int64_t V, int32_t mp) {
  Globals G;
  G.since = (short)d2bf((double)min(k - k_last_full, (int64_t)64) / 64.0);
  G.vfrac = (short)d2bf((double)V / (double)max(mp, 1));
  return G;
}

// The network inputs of column q in B layout (inputs 4g..4g+3 of this lane's
// group) at iteration k. The tabu age min(k - last, 1024) / 1024 is a
// multiple of 2^-10 in [0, 1], exact in FP64 before its single rounding.
__device__ __forceinline__ bf16x4 assemble(const uint16_t* __restrict__ feat, int q, int g, int64_t k,
                                           const Globals& G) {
  const bf16x4 raw = *(const bf16x4*)(feat + (int64_t)q * 16 + 4 * g);
  if (g != 3) return raw;
  const int32_t last = (int32_t)(((uint32_t)(uint16_t)raw[1] << 16) | (uint32_t)(uint16_t)raw[0]);
  const int64_t age = min(k - (int64_t)last, kAgeCap);
  bf16x4 x;
  x[0] = (short)d2bf((double)age * (1.0 / (double)kAgeCap));
  x[1] = G.since;
  x[2] = G.vfrac;
  x[3] = raw[3];
  return x;
}

// ---------------------------------------------------------------------------
// Stored rows
// ---------------------------------------------------------------------------

// Static inputs and initial dynamic state of every column: never moved, or
// the given last-move iterations and move counts (original order).
__global__ __launch_bounds__(256) void k_learn_init(const WalkCtx* __restrict__ walks,
                                                    const LearnCtx* __restrict__ lc, int32_t n,
                                                    const int32_t* __restrict__ last_move,
                                                    const int32_t* __restrict__ moves) {
  const WalkCtx& C = walks[0];
  const LearnCtx& L = *lc;
  const DevProblem& P = C.P;
  const int q = blockIdx.x * blockDim.x + threadIdx.x;
  if (q >= n) return;
  uint16_t* row = L.feat + (int64_t)q * 16;
  const double l = P.lb[q], u = P.ub[q];
  const bool isint = P.is_int[q] != 0;
  const bool isbin = isint && l == 0.0 && u == 1.0;
  const int deg = P.col_ptr[q + 1] - P.col_ptr[q];
  for (int t = 0; t < 16; ++t) row[t] = 0;
  row[1] = d2bf(log2(1.0 + (double)deg));
  row[2] = d2bf(L.c_max > 0.0 ? P.obj[q] / L.c_max : 0.0);
  row[4] = d2bf(isbin ? 1.0 : 0.0);
  row[5] = d2bf(isint && !isbin ? 1.0 : 0.0);
  row[6] = d2bf(isint ? 0.0 : 1.0);
  row[7] = d2bf(position(C.x[q], l, u));
  row[8] = d2bf((isfinite(l) && isfinite(u)) ? log2(1.0 + fmin(u - l, 1048576.0)) : 20.0);
  const int j = P.perm[q];
  const int32_t mv = moves ? moves[j] : 0;
  set_last_move(row, last_move ? last_move[j] : kNeverMoved);
  row[15] = d2bf(log2(1.0 + (double)mv));
  L.moves[q] = mv;
  L.xhat_last[q] = C.x[q];
}

// Contributions of stored entry e to the six refresh sums.
__device__ __forceinline__ void refresh_entry(const DevProblem& P, const RowState* rs, int e, double* v) {
  const RowState r = rs[P.col_row[e]];
  const double a = fabs(P.col_val[e]);
  const double eps = P.eps;
  v[0] += (double)r.w0;
  v[3] += 1.0;
  v[4] += a;
  if (r.r > eps) {
    v[1] += (double)r.w0;
    v[2] += 1.0;
    v[5] += a * fmin(r.r, 1000.0);
  }
  if (r.w1 >= 0.0f) {
    const double r1 = -r.r;
    v[0] += (double)r.w1;
    v[3] += 1.0;
    v[4] += a;
    if (r1 > eps) {
      v[1] += (double)r.w1;
      v[2] += 1.0;
      v[5] += a * fmin(r1, 1000.0);
    }
  }
}

// Inputs 0, 3, 7, 9, 10, 11 of column q from its six sums; xhat_last := xhat.
__device__ __forceinline__ void refresh_write(const WalkCtx& C, const LearnCtx& L, int q, const double* v) {
  uint16_t* row = L.feat + (int64_t)q * 16;
  const double sw = v[0], swv = v[1], nv = v[2], ne = v[3], sa = v[4], sav = v[5];
  const double x = C.x[q], xh = C.xhat[q];
  row[0] = d2bf(sw > 0.0 ? swv / sw : 0.0);
  row[3] = d2bf(sw > 0.0 ? fmin(fmax(C.s[q] / sw, -4.0), 4.0) : 0.0);
  row[7] = d2bf(position(x, C.P.lb[q], C.P.ub[q]));
  row[9] = d2bf(ne > 0.0 ? nv / ne : 0.0);
  row[10] = d2bf(sa > 0.0 ? sav / (1000.0 * sa) : 0.0);
  row[11] = d2bf(sign_of(xh - x));
  L.xhat_last[q] = xh;
}

// Short proposable columns: eight lanes per column, fixed-order sums.
__global__ __launch_bounds__(256) void k_refresh_short(const WalkCtx* __restrict__ walks,
                                                       const LearnCtx* __restrict__ lc) {
  const WalkCtx& C = walks[0];
  const LearnCtx& L = *lc;
  if (!L.ls->train_active) return;
  const int sub = threadIdx.x & 7;
  const int64_t groups = (int64_t)gridDim.x * (blockDim.x >> 3);
  for (int64_t idx = (int64_t)blockIdx.x * (blockDim.x >> 3) + (threadIdx.x >> 3); idx < L.n_ref_short;
       idx += groups) {
    const int q = L.ref_short[idx];
    double v[6] = {0, 0, 0, 0, 0, 0};
    for (int e = C.P.col_ptr[q] + sub; e < C.P.col_ptr[q + 1]; e += 8) refresh_entry(C.P, C.rs, e, v);
#pragma unroll
    for (int t = 0; t < 6; ++t)
#pragma unroll
      for (int o = 1; o < 8; o <<= 1) v[t] += __shfl_xor(v[t], o, kWave);
    if (sub == 0) refresh_write(C, L, q, v);
  }
}

__device__ __forceinline__ double block_sum(double v, double* red) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, kWave);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  double t = 0.0;
  for (int w = 0; w < (int)(blockDim.x >> 6); ++w) t += red[w];
  return t;
}

// Chunks of long proposable columns: one workgroup per chunk (grid-stride),
// partial sums per chunk.
__global__ __launch_bounds__(256) void k_refresh_chunks(const WalkCtx* __restrict__ walks,
                                                        const LearnCtx* __restrict__ lc) {
  const WalkCtx& C = walks[0];
  const LearnCtx& L = *lc;
  if (!L.ls->train_active) return;
  __shared__ double red[4];
  for (int t = blockIdx.x; t < L.n_ref_chunks; t += gridDim.x) {
    const ChunkTask T = L.ref_chunks[t];
    double v[6] = {0, 0, 0, 0, 0, 0};
    for (int e = T.e_beg + threadIdx.x; e < T.e_end; e += blockDim.x) refresh_entry(C.P, C.rs, e, v);
    double out[6];
    for (int k = 0; k < 6; ++k) out[k] = block_sum(v[k], red);
    if (threadIdx.x == 0)
      for (int k = 0; k < 6; ++k) L.ref_parts[T.slot].v[k] = out[k];
  }
}

// Long proposable columns: sums of their chunks in order.
__global__ __launch_bounds__(256) void k_refresh_combine(const WalkCtx* __restrict__ walks,
                                                         const LearnCtx* __restrict__ lc) {
  const WalkCtx& C = walks[0];
  const LearnCtx& L = *lc;
  if (!L.ls->train_active) return;
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= L.n_ref_cols) return;
  const ChunkCol cc = L.ref_cols[i];
  double v[6] = {0, 0, 0, 0, 0, 0};
  for (int k = 0; k < cc.nparts; ++k)
    for (int t = 0; t < 6; ++t) v[t] += L.ref_parts[cc.first + k].v[t];
  refresh_write(C, L, cc.col, v);
}

// Start of a block of iterations (full evaluation first).
__global__ void k_learn_begin(const WalkCtx* __restrict__ walks, const LearnCtx* __restrict__ lc) {
  const WalkCtx& C = walks[0];
  LearnState* ls = lc->ls;
  if (threadIdx.x != 0) return;
  WalkState* st = C.st;
  if (st->k < st->iters) {
    ls->idle = 0;
    ls->train_active = 1;
    ls->k_last_full = st->k;
  } else {
    ls->idle = 1;
    ls->train_active = 0;
  }
}

// ---------------------------------------------------------------------------
// Radix top-K
// ---------------------------------------------------------------------------

// Sums over the lanes up to and with this one, by DPP.
__device__ __forceinline__ uint32_t wave_scan(uint32_t u) {
  int v = (int)u;
  v += dpp<kRowShr1, 0xF>(v, 0);
  v += dpp<kRowShr2, 0xF>(v, 0);
  v += dpp<kRowShr4, 0xF>(v, 0);
  v += dpp<kRowShr8, 0xF>(v, 0);
  v += dpp<kBcast15, 0xA>(v, 0);
  v += dpp<kBcast31, 0xC>(v, 0);
  return (uint32_t)v;
}

struct Select {
  bool all;          // at most K nonzero keys: take every nonzero key
  uint32_t prefix;   // digits chosen so far (levels below `upto`)
  int rem;           // keys still to take under the prefix
  uint32_t thresh;   // final key T (upto == 3)
  int need_eq;       // keys == T to take (upto == 3)
};

// The histograms of a selection: the first digit's in kHistCopies copies (the
// scores share few first digits, so the scoring workgroups would queue at one
// copy: 12 ns each), then the other digits'.
constexpr int kHistCopies = 8;
static_assert((kHistCopies + 2) * kRadixBins == kHistStride, "as allocated");
__device__ __forceinline__ int hist_of(int which, int level) {
  return which * kHistStride + (level == 0 ? 0 : kHistCopies + level - 1) * kRadixBins;
}

// A thread's bins of one histogram: kBinsPer neighbours, thread 0 the highest.
constexpr int kBinsPer = kRadixBins / kBlock;
struct Bins {
  uint32_t c[kBinsPer];
};
template <int kCopies>
__device__ __forceinline__ Bins load_bins(const uint32_t* __restrict__ h) {
  static_assert(kBinsPer == 8, "two 16-byte loads");
  const uint4* p = (const uint4*)(h + kRadixBins - kBinsPer * ((int)threadIdx.x + 1));
  Bins B{};
#pragma unroll
  for (int c = 0; c < kCopies; ++c, p += kRadixBins / 4) {
    const uint4 lo = p[0], hi = p[1];
    const uint32_t v[kBinsPer] = {hi.w, hi.z, hi.y, hi.x, lo.w, lo.z, lo.y, lo.x};
#pragma unroll
    for (int t = 0; t < kBinsPer; ++t) B.c[t] += v[t];
  }
  return B;
}

// Whole workgroup (256 threads): the bin of a histogram (bins from the top)
// that holds the rem-th largest key; *left = rank of that key inside the bin.
__device__ void find_digit(const Bins& B, int rem, int* digit, int* left, uint32_t* total) {
  __shared__ uint32_t part[kBlock / kWave];
  __shared__ int res[2];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  uint32_t sum = 0;
#pragma unroll
  for (int t = 0; t < kBinsPer; ++t) sum += B.c[t];
  const uint32_t inc = wave_scan(sum);
  __syncthreads();
  if (lane == kWave - 1) part[wv] = inc;
  if (tid == 0) {
    res[0] = 0;
    res[1] = 0;
  }
  __syncthreads();
  uint32_t before_w = 0, all = 0;
  for (int w = 0; w < kBlock / kWave; ++w) {
    if (w < wv) before_w += part[w];
    all += part[w];
  }
  const uint32_t hi = before_w + inc, lo = hi - sum;
  if (lo < (uint32_t)rem && hi >= (uint32_t)rem) {
    uint32_t cum = lo;
#pragma unroll
    for (int t = 0; t < kBinsPer; ++t) {
      if (cum < (uint32_t)rem && cum + B.c[t] >= (uint32_t)rem) {
        res[0] = kRadixBins - 1 - (tid * kBinsPer + t);
        res[1] = rem - (int)cum;
      }
      cum += B.c[t];
    }
  }
  __syncthreads();
  *digit = res[0];
  *left = res[1];
  *total = all;
}

// Digits of levels < kUpto (3: the final threshold) from the histograms of the
// earlier kernels, which load_levels() has read: the loads do not depend on
// the digits, so one wait covers them all. Whole workgroup.
template <int kUpto>
struct Levels {
  Bins b[kUpto];
};
template <int kUpto>
__device__ __forceinline__ Levels<kUpto> load_levels(const LearnCtx& L, int which) {
  Levels<kUpto> V;
  V.b[0] = load_bins<kHistCopies>(L.hist + hist_of(which, 0));
#pragma unroll
  for (int t = 1; t < kUpto; ++t) V.b[t] = load_bins<1>(L.hist + hist_of(which, t));
  return V;
}
template <int kUpto>
__device__ Select derive(const Levels<kUpto>& V, int K) {
  Select S{false, 0u, K, 0u, 0};
  int d, left;
  uint32_t total;
  find_digit(V.b[0], K, &d, &left, &total);
  if (total <= (uint32_t)K) {
    S.all = true;
    return S;
  }
  S.prefix = (uint32_t)d;
  S.rem = left;
  if constexpr (kUpto >= 2) {
    find_digit(V.b[1], S.rem, &d, &left, &total);
    S.prefix = (S.prefix << 11) | (uint32_t)d;
    S.rem = left;
  }
  if constexpr (kUpto >= 3) {
    find_digit(V.b[2], S.rem, &d, &left, &total);
    S.thresh = (S.prefix << 10) | (uint32_t)d;
    S.need_eq = left;
  }
  return S;
}

__device__ __forceinline__ void flush_hist(uint32_t* lds, uint32_t* global) {
  __syncthreads();
  for (int b = threadIdx.x; b < kRadixBins; b += blockDim.x) {
    const uint32_t c = lds[b];
    if (c) atomicAdd(&global[b], c);
  }
}

// Network score key of every column plus the first-digit histogram; also the
// pending incumbent copy (before this iteration's move changes x).
__global__ __launch_bounds__(256) void k_learn_score(const WalkCtx* __restrict__ walks,
                                                     const LearnCtx* __restrict__ lc, const float* __restrict__ w,
                                                     const uint16_t* __restrict__ wb, int32_t n) {
  const WalkCtx& C = walks[0];
  const LearnCtx& L = *lc;
  const WalkState* st = C.st;
  if (!active(st, L.ls)) return;
  __shared__ uint32_t hist[kRadixBins];
  for (int b = threadIdx.x; b < kRadixBins; b += blockDim.x) hist[b] = 0;
  if (st->copy_best)
    for (int q = blockIdx.x * blockDim.x + threadIdx.x; q < n; q += gridDim.x * blockDim.x) C.best_x[q] = C.x[q];
  __syncthreads();
  Weights W;
  load_weights(wb, w, W);
  const int l = threadIdx.x & 63, g = l >> 4, r = l & 15;
  const int64_t k = st->k;
  const Globals Gl = globals(k, L.ls->k_last_full, st->V, L.mp);
  const int ntiles = (n + 15) / 16;
  const int stride = gridDim.x * 4;
  const bf16x4 zero = {0, 0, 0, 0};
  // a ring of kScoreDepth tiles per wavefront: the inputs of the tile
  // kScoreDepth steps ahead are loaded while the current one is computed
  constexpr int kScoreDepth = 8;
  const int tile0 = blockIdx.x * 4 + (threadIdx.x >> 6);
  bf16x4 ring[kScoreDepth];
#pragma unroll
  for (int d = 0; d < kScoreDepth; ++d) {
    const int t = tile0 + d * stride;
    ring[d] = (t < ntiles && t * 16 + r < n) ? assemble(L.feat, t * 16 + r, g, k, Gl) : zero;
  }
  for (int base = tile0; base < ntiles; base += kScoreDepth * stride) {
#pragma unroll
    for (int d = 0; d < kScoreDepth; ++d) {
      const int t = base + d * stride;
      if (t >= ntiles) break;
      const bf16x4 x = ring[d];
      const int tn = t + kScoreDepth * stride;
      ring[d] = (tn < ntiles && tn * 16 + r < n) ? assemble(L.feat, tn * 16 + r, g, k, Gl) : zero;
      Acts A;
      forward(W, x, A);
      const int q = t * 16 + r;
      if (l < 16 && q < n) {
        const uint32_t key = L.cls[q] != SUB_NONE ? order_key(A.y) : 0u;
        L.keys[0][q] = key;
        if (key) atomicAdd(&hist[key >> 21], 1u);
      }
    }
  }
  flush_hist(hist, L.hist + hist_of(0, 0) + (blockIdx.x & (kHistCopies - 1)) * kRadixBins);
}

// Label keys (exact scores of the full pass) plus their first-digit histogram.
__global__ __launch_bounds__(256) void k_label_keys(const WalkCtx* __restrict__ walks,
                                                    const LearnCtx* __restrict__ lc, int32_t n) {
  const WalkCtx& C = walks[0];
  const LearnCtx& L = *lc;
  if (!active(C.st, L.ls)) return;
  __shared__ uint32_t hist[kRadixBins];
  for (int b = threadIdx.x; b < kRadixBins; b += blockDim.x) hist[b] = 0;
  __syncthreads();
  for (int q = blockIdx.x * blockDim.x + threadIdx.x; q < n; q += gridDim.x * blockDim.x) {
    const uint32_t key = L.cls[q] != SUB_NONE ? order_key((float)C.s[q]) : 0u;
    L.keys[1][q] = key;
    if (key) atomicAdd(&hist[key >> 21], 1u);
  }
  flush_hist(hist, L.hist + hist_of(1, 0) + (blockIdx.x & (kHistCopies - 1)) * kRadixBins);
}

__device__ __forceinline__ uint32_t digit_of(uint32_t key, int level) {
  return level == 1 ? ((key >> 10) & 0x7FFu) : (key & 0x3FFu);
}

__device__ __forceinline__ uint32_t prefix_of(uint32_t key, int level) {
  return level == 1 ? (key >> 21) : (key >> 10);
}

// A thread's keys of a tile of kTopkChunk columns: four, then every fourth
// workgroup width on (zero past the end; the array is padded to whole fours).
constexpr int kKeysPer = kTopkChunk / kBlock;

// Histogram of digit kLevel (1 or 2) over keys that match the digits above, a
// tile of kTopkChunk columns per workgroup and step, its keys asked for before
// the digits are derived.
template <int kLevel>
__global__ __launch_bounds__(kBlock) void k_topk_hist(const WalkCtx* __restrict__ walks,
                                                      const LearnCtx* __restrict__ lc, int32_t which, int32_t n) {
  const WalkCtx& C = walks[0];
  const LearnCtx& L = *lc;
  if (!active(C.st, L.ls)) return;
  const Levels<kLevel> V = load_levels<kLevel>(L, which);
  const uint32_t* keys = L.keys[which];
  uint4 v[kKeysPer / 4];
  auto load = [&](int beg) {
#pragma unroll
    for (int t = 0; t < kKeysPer / 4; ++t) {
      const int q = beg + (t * kBlock + (int)threadIdx.x) * 4;
      v[t] = q < n ? *(const uint4*)(keys + q) : uint4{0u, 0u, 0u, 0u};
    }
  };
  load(blockIdx.x * kTopkChunk);
  __shared__ uint32_t hist[kRadixBins];
  for (int b = threadIdx.x; b < kRadixBins; b += kBlock) hist[b] = 0;
  const Select S = derive<kLevel>(V, L.K[which]);
  if (S.all) return;
  for (int beg = blockIdx.x * kTopkChunk; beg < n; beg += gridDim.x * kTopkChunk) {
    if (beg != (int)blockIdx.x * kTopkChunk) load(beg);
#pragma unroll
    for (int t = 0; t < kKeysPer / 4; ++t) {
      const int q = beg + (t * kBlock + (int)threadIdx.x) * 4;
      const uint32_t k4[4] = {v[t].x, v[t].y, v[t].z, v[t].w};
#pragma unroll
      for (int u = 0; u < 4; ++u)
        if (q + u < n && k4[u] && prefix_of(k4[u], kLevel) == S.prefix) atomicAdd(&hist[digit_of(k4[u], kLevel)], 1u);
    }
  }
  flush_hist(hist, L.hist + hist_of(which, kLevel));
}

__device__ __forceinline__ bool take_above(uint32_t key, const Select& S) {
  return key != 0u && (S.all || key > S.thresh);
}

__device__ __forceinline__ bool take_equal(uint32_t key, const Select& S) {
  return !S.all && key == S.thresh;
}

// Appends the c2 first columns of the proposal set to the set log as the set
// of the current iteration (one workgroup; no-op without the log).
__device__ void log_set(const WalkCtx& C, const LearnCtx& L, int c2) {
  if (L.set_off == nullptr) return;
  const int64_t k = C.st->k;
  const int64_t pos = L.ls->set_pos;
  const bool fits = pos + c2 <= L.set_log_cap;
  if (fits)
    for (int i = threadIdx.x; i < c2; i += blockDim.x) L.set_log[pos + i] = C.P.perm[L.sel[0][i]];
  __syncthreads();
  if (threadIdx.x == 0) {
    const int64_t end = fits ? pos + c2 : pos;
    L.set_off[k] = pos;
    L.set_off[k + 1] = end;
    L.ls->set_pos = end;
  }
}

// A proposal iteration that keeps the last proposal set: logs it again.
__global__ __launch_bounds__(256) void k_keep_set(const WalkCtx* __restrict__ walks,
                                                  const LearnCtx* __restrict__ lc) {
  const WalkCtx& C = walks[0];
  const LearnCtx& L = *lc;
  if (!active(C.st, L.ls)) return;
  log_set(C, L, L.ls->tk[0].count);
}

// Index of the chunk that holds item i of an exclusive prefix off[0..nc].
__device__ __forceinline__ int chunk_of(const int32_t* off, int nc, int i) {
  int lo = 0, hi = nc - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (off[mid] <= i)
      lo = mid;
    else
      hi = mid - 1;
  }
  return lo;
}

// Store of 8 bytes past the caches of this XCD (an atomic store of device scope):
// once it has completed, any other workgroup can load it after invalidating its
// own caches.
__device__ __forceinline__ void put_agent(uint2* p, uint2 v) {
  __hip_atomic_store((unsigned long long*)p, (unsigned long long)v.y << 32 | v.x, __ATOMIC_RELAXED,
                     __HIP_MEMORY_SCOPE_AGENT);
}
constexpr int kWaitStores = 0x0F70;  // s_waitcnt vmcnt(0)

// The selection in ascending column order and its end, in one launch. Every
// workgroup compacts its chunk of columns (kTopkChunk times L.topk_tiles)
// into its part of L.stage: the keys above the threshold from the front, each
// with the number of equal ones before it, the equal ones from the back with
// the number of greater ones before them (no more than the selection can
// take). The last to arrive adds the chunks' counts, so that every staged key
// knows its place, and writes the selected columns; for the proposal set also
// the subset-pass chunk offsets and the set log; then it clears the histograms
// and the ticket for the next selection. What the workgroups hand over goes past
// their L2 (put_agent), so none of them needs a release fence, which would write
// back what the scoring left there: with one the whole iteration took 63, 97 and
// 194 us on 200k, 700k and 2M columns, without 60, 82 and 141. (A launch of its
// own for the list: 59, 78 and 135, but 2.5 us more in each iteration that does
// nothing after a stall.)
__global__ __launch_bounds__(kBlock) void k_topk_take(const WalkCtx* __restrict__ walks,
                                                      const LearnCtx* __restrict__ lc, int32_t which, int32_t full,
                                                      int32_t n) {
  const WalkCtx& C = walks[0];
  const LearnCtx& L = *lc;
  if (!active(C.st, L.ls)) return;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const Levels<3> V = load_levels<3>(L, which);
  const uint32_t* keys = L.keys[which];
  const int chunk = kTopkChunk * L.topk_tiles;
  const int beg = blockIdx.x * chunk;
  uint4 v[kKeysPer / 4];
  auto load = [&](int tile) {
#pragma unroll
    for (int t = 0; t < kKeysPer / 4; ++t) {
      const int q = beg + tile * kTopkChunk + tid * kKeysPer + 4 * t;
      v[t] = q < n ? *(const uint4*)(keys + q) : uint4{0u, 0u, 0u, 0u};
    }
  };
  load(0);
  const Select S = derive<3>(V, L.K[which]);
  __shared__ uint32_t sg[4], se[4];
  __shared__ uint32_t last;
  uint2* stage = L.stage + (int64_t)blockIdx.x * chunk;
  uint32_t gt_base = 0, eq_base = 0;  // of the tiles before this one
  for (int tile = 0; tile < L.topk_tiles; ++tile) {
    if (tile > 0) load(tile);
    const int q0 = beg + tile * kTopkChunk + tid * kKeysPer;
    uint32_t mg = 0, me = 0;  // this thread's keys above and equal, a bit each
#pragma unroll
    for (int t = 0; t < kKeysPer / 4; ++t) {
      const uint32_t k4[4] = {v[t].x, v[t].y, v[t].z, v[t].w};
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const bool in = q0 + 4 * t + u < n;
        mg |= (in && take_above(k4[u], S) ? 1u : 0u) << (4 * t + u);
        me |= (in && take_equal(k4[u], S) ? 1u : 0u) << (4 * t + u);
      }
    }
    const uint32_t gt = __popc(mg), eq = __popc(me);
    const uint32_t ig = wave_scan(gt), ie = wave_scan(eq);
    __syncthreads();  // the tile before has read sg and se
    if (lane == kWave - 1) {
      sg[wv] = ig;
      se[wv] = ie;
    }
    __syncthreads();
    uint32_t og = gt_base + ig - gt, oe = eq_base + ie - eq;
    for (int k = 0; k < kBlock / kWave; ++k) {
      if (k < wv) {
        og += sg[k];
        oe += se[k];
      }
      gt_base += sg[k];
      eq_base += se[k];
    }
    for (uint32_t m = mg; m; m &= m - 1) {
      const int b = __builtin_ctz(m);
      const uint32_t below = (1u << b) - 1u;
      put_agent(stage + og + __popc(mg & below), uint2{(uint32_t)(q0 + b), oe + __popc(me & below)});
    }
    for (uint32_t m = me; m; m &= m - 1) {
      const int b = __builtin_ctz(m);
      const uint32_t below = (1u << b) - 1u;
      const uint32_t e = oe + __popc(me & below);
      if (e >= (uint32_t)S.need_eq) break;
      put_agent(stage + chunk - 1 - e, uint2{(uint32_t)(q0 + b), og + __popc(mg & below)});
    }
  }
  if (tid == 0) put_agent(L.wg_cnt + blockIdx.x, uint2{gt_base, eq_base});
  // the staged keys and the counts have reached memory (they went past the L2)
  // before the workgroup takes its ticket; the fence keeps the stores above the
  // wait
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
  __builtin_amdgcn_s_waitcnt(kWaitStores);
  __syncthreads();
  uint32_t* ticket = L.hist + 2 * kHistStride;
  if (tid == 0) last = atomicAdd(ticket, 1u);
  __syncthreads();
  if (last != gridDim.x - 1) return;
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");

  // exclusive prefixes of the chunks' counts
  __shared__ int32_t pg[kTopkChunks + 1], pe[kTopkChunks + 1];
  __shared__ int32_t pc[kTopkMax];  // subset-pass chunks of the selected columns
  constexpr int kPer = kTopkChunks / kBlock;
  const int nc = gridDim.x;
  uint2 c[kPer];
  uint32_t cg = 0, ce = 0;
#pragma unroll
  for (int t = 0; t < kPer; ++t) {
    const int b = tid * kPer + t;
    c[t] = b < nc ? L.wg_cnt[b] : uint2{0u, 0u};
    cg += c[t].x;
    ce += c[t].y;
  }
  uint32_t ag = wave_scan(cg), ae = wave_scan(ce);
  if (lane == kWave - 1) {
    sg[wv] = ag;
    se[wv] = ae;
  }
  __syncthreads();
  ag -= cg;
  ae -= ce;
  for (int k = 0; k < wv; ++k) {
    ag += sg[k];
    ae += se[k];
  }
#pragma unroll
  for (int t = 0; t < kPer; ++t) {
    pg[tid * kPer + t] = (int32_t)ag;
    pe[tid * kPer + t] = (int32_t)ae;
    ag += c[t].x;
    ae += c[t].y;
  }
  if (tid == kBlock - 1) pg[kTopkChunks] = (int32_t)ag;
  __syncthreads();
  const int above = pg[kTopkChunks];
  const int count = above + (S.all ? 0 : S.need_eq);
  int32_t* out = L.sel[which];
  constexpr int kU = 4;  // staged keys in flight per thread
  for (int i0 = tid; i0 < count; i0 += kU * kBlock) {
    uint2 k[kU];
    int pos[kU];
#pragma unroll
    for (int u = 0; u < kU; ++u) {
      const int i = i0 + u * kBlock;
      if (i >= count) break;
      const bool eq = i >= above;
      const int j = eq ? i - above : i;
      const int b = chunk_of(eq ? pe : pg, nc, j);
      const int o = j - (eq ? pe[b] : pg[b]);
      k[u] = L.stage[(int64_t)b * chunk + (eq ? chunk - 1 - o : o)];
      pos[u] = eq ? j + pg[b] : i;
      if (!eq) k[u].y += pe[b];
    }
#pragma unroll
    for (int u = 0; u < kU; ++u) {
      const int i = i0 + u * kBlock;
      if (i >= count) break;
      // equal: after the greater ones before it; greater: after the equal ones
      // before it that are taken
      const int at = pos[u] + (i >= above ? (int)k[u].y : min((int)k[u].y, S.all ? 0 : S.need_eq));
      const int q = (int)k[u].x;
      out[at] = q;
      if (which == 0) {
        const int e = C.P.col_ptr[q + 1] - C.P.col_ptr[q];
        pc[at] = L.cls[q] == SUB_GENERAL ? 0 : max(1, (e + kSubsetChunk - 1) / kSubsetChunk);
      }
    }
  }
  __syncthreads();
  if (which == 0) {
    // exclusive prefix of the columns' chunk counts, a run of columns a thread
    const int per = (count + kBlock - 1) / kBlock;
    const int i0 = min(count, tid * per), i1 = min(count, i0 + per);
    uint32_t sum = 0;
    for (int i = i0; i < i1; ++i) sum += (uint32_t)pc[i];
    const uint32_t inc = wave_scan(sum);
    if (lane == kWave - 1) sg[wv] = inc;
    __syncthreads();
    int off = (int)(inc - sum);
    for (int k = 0; k < wv; ++k) off += (int)sg[k];
    for (int i = i0; i < i1; ++i) {
      L.sub_off[i] = off;
      off += pc[i];
    }
    if (tid == kBlock - 1) {
      L.sub_off[count] = off;
      L.ls->tk[0].chunks = off;
    }
    // proposal-set log (original indices); a full evaluation records an empty range
    log_set(C, L, full ? 0 : count);
  }
  if (tid == 0) {
    L.ls->tk[which].count = count;
    *ticket = 0u;
  }
  // every reader of the histograms has taken its ticket
  uint4* H = (uint4*)(L.hist + which * kHistStride);
  for (int b = tid; b < kHistStride / 4; b += kBlock) H[b] = uint4{0u, 0u, 0u, 0u};
}

// ---------------------------------------------------------------------------
// Training pairs, judge, features
// ---------------------------------------------------------------------------

// Materialised training inputs and targets of a full evaluation: the top T
// columns by exact score and T random proposable columns; target =
// max(s, 0) / max_j s_j (0 when no score is positive). Also appends them to
// the pair log. One workgroup.
__global__ __launch_bounds__(256) void k_learn_pairs(const WalkCtx* __restrict__ walks,
                                                     const LearnCtx* __restrict__ lc) {
  const WalkCtx& C = walks[0];
  const LearnCtx& L = *lc;
  const WalkState* st = C.st;
  if (!active(st, L.ls)) return;
  __shared__ double red[4];
  const int T2 = 2 * L.T;
  const int cnt = L.ls->tk[1].count;
  const int64_t ev = L.ls->evals;
  double smax = 0.0;
  for (int i = threadIdx.x; i < cnt; i += blockDim.x) smax = fmax(smax, C.s[L.sel[1][i]]);
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) smax = fmax(smax, __shfl_xor(smax, o, kWave));
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  if (lane == 0) red[wv] = smax;
  __syncthreads();
  smax = fmax(fmax(red[0], red[1]), fmax(red[2], red[3]));
  const int64_t k = st->k;
  const Globals Gl = globals(k, L.ls->k_last_full, st->V, L.mp);
  const int64_t logged = L.ls->logged;
  const bool log = L.log_feat != nullptr && logged + T2 <= L.log_cap;
  for (int i = threadIdx.x; i < T2; i += blockDim.x) {
    int q;
    if (i < L.T && i < cnt)
      q = L.sel[1][i];
    else
      q = L.elig_list[splitmix64(L.seed, (uint64_t)(ev * T2 + i)) % (uint64_t)L.n_elig];
    const double tgt = smax > 0.0 ? fmax(C.s[q], 0.0) / smax : 0.0;
    L.pair_tgt[i] = (float)tgt;
    if (log) L.log_tgt[logged + i] = (float)tgt;
    for (int gg = 0; gg < 4; ++gg) {
      const bf16x4 x = assemble(L.feat, q, gg, k, Gl);
      for (int t = 0; t < 4; ++t) {
        L.pair_feat[(int64_t)i * 16 + 4 * gg + t] = (uint16_t)x[t];
        if (log) L.log_feat[(logged + i) * 16 + 4 * gg + t] = (uint16_t)x[t];
      }
    }
  }
  __syncthreads();
  if (threadIdx.x == 0 && log) L.ls->logged = logged + T2;
}

// Judge of a full evaluation (was its move in the network's proposal set?)
// and the stored-row update of the move. Runs after the iteration's end.
__global__ void k_learn_judge(const WalkCtx* __restrict__ walks, const LearnCtx* __restrict__ lc) {
  const WalkCtx& C = walks[0];
  const LearnCtx& L = *lc;
  const WalkState* st = C.st;
  if (threadIdx.x != 0 || st->sel_k < 0) return;
  LearnState* ls = L.ls;
  ls->evals += 1;
  const int q = st->mv_j;
  if (q < 0) return;
  after_move(C, L, q, st->mv_new, st->sel_k);
  const int32_t* set = L.sel[0];
  int lo = 0, hi = ls->tk[0].count - 1;
  while (lo <= hi) {
    const int mid = (lo + hi) >> 1;
    if (set[mid] == q) {
      ls->hits += 1;
      return;
    }
    if (set[mid] < q)
      lo = mid + 1;
    else
      hi = mid - 1;
  }
}

// All 16 inputs of every column in original order (zeros for columns that
// are never proposed).
__global__ __launch_bounds__(256) void k_learn_features_out(const WalkCtx* __restrict__ walks,
                                                            const LearnCtx* __restrict__ lc, int32_t n, int64_t k,
                                                            int64_t k_last_full, uint16_t* __restrict__ out) {
  const WalkCtx& C = walks[0];
  const LearnCtx& L = *lc;
  const int q = blockIdx.x * blockDim.x + threadIdx.x;
  if (q >= n) return;
  uint16_t* o = out + (int64_t)C.P.perm[q] * 16;
  const bool ok = L.cls[q] != SUB_NONE;
  const Globals Gl = globals(k, k_last_full, C.st->V, L.mp);
  for (int gg = 0; gg < 4; ++gg) {
    const bf16x4 x = assemble(L.feat, q, gg, k, Gl);
    for (int t = 0; t < 4; ++t) o[4 * gg + t] = ok ? (uint16_t)x[t] : 0;
  }
}

inline int grid_for(int64_t work, int per_block, int cap) {
  int64_t b = (work + per_block - 1) / per_block;
  return (int)std::max<int64_t>(1, std::min<int64_t>(b, cap));
}

hipError_t topk(const WalkCtx* C, const LearnCtx* L, const LearnCtx& Lh, int which, int full, int32_t n,
                hipStream_t s) {
  const int hb = grid_for(n, kTopkChunk, 1024);
  hipLaunchKernelGGL(k_topk_hist<1>, dim3(hb), dim3(kBlock), 0, s, C, L, which, n);
  hipLaunchKernelGGL(k_topk_hist<2>, dim3(hb), dim3(kBlock), 0, s, C, L, which, n);
  hipLaunchKernelGGL(k_topk_take, dim3(Lh.nwg), dim3(kBlock), 0, s, C, L, which, (int32_t)full, n);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_learn_init(const WalkCtx* C, const LearnCtx* L, const LearnCtx& Lh, int32_t n,
                             const int32_t* last_move, const int32_t* moves, hipStream_t s) {
  if (n > 0) hipLaunchKernelGGL(k_learn_init, dim3((n + 255) / 256), dim3(256), 0, s, C, L, n, last_move, moves);
  return hipGetLastError();
}

hipError_t launch_learn_refresh(const WalkCtx* C, const LearnCtx* L, const LearnCtx& Lh, hipStream_t s) {
  if (Lh.n_ref_short > 0)
    hipLaunchKernelGGL(k_refresh_short, dim3(grid_for(Lh.n_ref_short, 32, 8192)), dim3(256), 0, s, C, L);
  if (Lh.n_ref_chunks > 0) {
    hipLaunchKernelGGL(k_refresh_chunks, dim3(std::min(Lh.n_ref_chunks, 4096)), dim3(256), 0, s, C, L);
    hipLaunchKernelGGL(k_refresh_combine, dim3((Lh.n_ref_cols + 255) / 256), dim3(256), 0, s, C, L);
  }
  return hipGetLastError();
}

hipError_t launch_learn_begin(const WalkCtx* C, const LearnCtx* L, hipStream_t s) {
  hipLaunchKernelGGL(k_learn_begin, dim3(1), dim3(64), 0, s, C, L);
  return hipGetLastError();
}

hipError_t launch_learn_propose(const WalkCtx* C, const LearnCtx* L, const LearnCtx& Lh, const ModelDev& M,
                                int32_t n, int full_iteration, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  // three workgroups a CU, as many as are resident; two while that leaves a
  // wavefront few tiles, as each workgroup adds its turn at the histogram's bins.
  // An iteration with 512 and 768 of them: 57.6 and 58.5 us on 200k columns, 78.4
  // and 77.2 on 700k, 149 and 134 on 2M (1024: 149, 1536: 140)
  hipLaunchKernelGGL(k_learn_score, dim3(grid_for(n, 64, n < (1 << 19) ? 512 : 768)), dim3(256), 0, s, C, L, M.w, M.wb, n);
  return topk(C, L, Lh, 0, full_iteration, n, s);
}

hipError_t launch_learn_train(const WalkCtx* C, const LearnCtx* L, const LearnCtx& Lh, const ModelDev& M,
                              int32_t n, int32_t steps, float lr, hipStream_t s) {
  if (n <= 0 || (steps <= 0 && Lh.log_feat == nullptr)) return hipSuccess;
  hipLaunchKernelGGL(k_label_keys, dim3(grid_for(n, 256 * 16, 1024)), dim3(256), 0, s, C, L, n);
  hipError_t e = topk(C, L, Lh, 1, 1, n, s);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_learn_pairs, dim3(1), dim3(256), 0, s, C, L);
  for (int32_t t = 0; t < steps; ++t) {
    e = launch_mlp_grad_guarded(M, &Lh.ls->train_active, Lh.pair_feat, Lh.pair_tgt, 2 * (int64_t)Lh.T, s);
    if (e != hipSuccess) return e;
    e = launch_mlp_reduce_guarded(M, &Lh.ls->train_active, 2 * (int64_t)Lh.T, lr, s);
    if (e != hipSuccess) return e;
  }
  return hipGetLastError();
}

hipError_t launch_learn_keep_set(const WalkCtx* C, const LearnCtx* L, hipStream_t s) {
  hipLaunchKernelGGL(k_keep_set, dim3(1), dim3(256), 0, s, C, L);
  return hipGetLastError();
}

hipError_t launch_learn_judge(const WalkCtx* C, const LearnCtx* L, hipStream_t s) {
  hipLaunchKernelGGL(k_learn_judge, dim3(1), dim3(64), 0, s, C, L);
  return hipGetLastError();
}

hipError_t launch_learn_features_out(const WalkCtx* C, const LearnCtx* L, int32_t n, int64_t k, int64_t k_last_full,
                                     uint16_t* out, hipStream_t s) {
  if (n > 0)
    hipLaunchKernelGGL(k_learn_features_out, dim3((n + 255) / 256), dim3(256), 0, s, C, L, n, k, k_last_full, out);
  return hipGetLastError();
}

}  // namespace chap
