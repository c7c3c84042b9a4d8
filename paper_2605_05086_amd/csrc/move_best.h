// Best moves: the highest positive score overall and among the columns not
// tabu (ties to the lowest original index), as scoring and scanning kernels
// reduce and record them for the move selection.
#pragma once

#include <hip/hip_runtime.h>

#include <climits>

#include "chap_internal.h"

namespace chap {

__device__ __forceinline__ bool better(double sa, int ja, double sb, int jb) {
  return sa > sb || (sa == sb && ja < jb);
}

// Reductions across a wavefront by DPP (no LDS exchange): rows of 16 lanes
// first, then the last lane of a row into the next rows; lane 63 ends with the
// value of all lanes, which every lane then reads. Lanes a step has no source
// for get the identity `id`.
template <int kCtrl, int kRowMask>
__device__ __forceinline__ int dpp(int v, int id) {
  return __builtin_amdgcn_update_dpp(id, v, kCtrl, kRowMask, 0xF, false);
}
template <int kCtrl, int kRowMask>
__device__ __forceinline__ double dpp_d(double v) {  // identity 0.0
  const long long u = __double_as_longlong(v);
  const unsigned lo = (unsigned)dpp<kCtrl, kRowMask>((int)u, 0);
  const unsigned hi = (unsigned)dpp<kCtrl, kRowMask>((int)(u >> 32), 0);
  return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}
constexpr int kRowShr1 = 0x111, kRowShr2 = 0x112, kRowShr4 = 0x114, kRowShr8 = 0x118, kBcast15 = 0x142,
              kBcast31 = 0x143;

// Maximum of values >= 0.
__device__ __forceinline__ double wave_max_pos(double v) {
  v = fmax(v, dpp_d<kRowShr1, 0xF>(v));
  v = fmax(v, dpp_d<kRowShr2, 0xF>(v));
  v = fmax(v, dpp_d<kRowShr4, 0xF>(v));
  v = fmax(v, dpp_d<kRowShr8, 0xF>(v));
  v = fmax(v, dpp_d<kBcast15, 0xA>(v));
  v = fmax(v, dpp_d<kBcast31, 0xC>(v));
  const long long u = __double_as_longlong(v);
  const unsigned lo = __builtin_amdgcn_readlane((unsigned)u, 63);
  const unsigned hi = __builtin_amdgcn_readlane((unsigned)(u >> 32), 63);
  return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

__device__ __forceinline__ int wave_min_int(int v) {
  v = min(v, dpp<kRowShr1, 0xF>(v, INT_MAX));
  v = min(v, dpp<kRowShr2, 0xF>(v, INT_MAX));
  v = min(v, dpp<kRowShr4, 0xF>(v, INT_MAX));
  v = min(v, dpp<kRowShr8, 0xF>(v, INT_MAX));
  v = min(v, dpp<kBcast15, 0xA>(v, INT_MAX));
  v = min(v, dpp<kBcast31, 0xC>(v, INT_MAX));
  return __builtin_amdgcn_readlane(v, 63);
}

__device__ __forceinline__ int wave_sum_int(int v) {
  v += dpp<kRowShr1, 0xF>(v, 0);
  v += dpp<kRowShr2, 0xF>(v, 0);
  v += dpp<kRowShr4, 0xF>(v, 0);
  v += dpp<kRowShr8, 0xF>(v, 0);
  v += dpp<kBcast15, 0xA>(v, 0);
  v += dpp<kBcast31, 0xC>(v, 0);
  return __builtin_amdgcn_readlane(v, 63);
}

// Running best (score desc, original index asc) with the internal index.
struct Best {
  double s = 0.0;
  int j = INT_MAX;  // original index
  int q = -1;       // internal index
  __device__ __forceinline__ void offer(double s2, int j2, int q2) {
    if (better(s2, j2, s, j)) {
      s = s2;
      j = j2;
      q = q2;
    }
  }
  // Best of the wavefront on every lane: the maximum score, the lowest index
  // among the lanes that hold it, that lane's column.
  __device__ __forceinline__ void wave_reduce() {
    const double m = wave_max_pos(s);
    const int mj = wave_min_int(s == m ? j : INT_MAX);
    const int l = __builtin_ctzll(__ballot(s == m && j == mj));
    q = __builtin_amdgcn_readlane(q, l);
    s = m;
    j = mj;
  }
};

// One record of the move selection (MoveRecord in device memory).
struct BestPair {
  Best all, free;  // free: not tabu
  __device__ __forceinline__ void offer(double s, int j, int q, bool tabu) {
    all.offer(s, j, q);
    if (!tabu) free.offer(s, j, q);
  }
  __device__ __forceinline__ void offer(const MoveRecord& r) {
    all.offer(r.s_all, r.j_all, r.q_all);
    free.offer(r.s_free, r.j_free, r.q_free);
  }
  __device__ __forceinline__ void wave_reduce() {
    all.wave_reduce();
    free.wave_reduce();
  }
  __device__ __forceinline__ MoveRecord record() const {
    return MoveRecord{all.s, free.s, all.j, all.q, free.j, free.q};
  }
};

// Best of a workgroup of kWaves wavefronts into *out (every thread calls it).
template <int kWaves>
__device__ __forceinline__ void block_record(BestPair b, MoveRecord* out) {
  __shared__ MoveRecord rec[kWaves];
  b.wave_reduce();
  if ((threadIdx.x & (kWave - 1)) == 0) rec[threadIdx.x >> 6] = b.record();
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < kWaves; ++w) b.offer(rec[w]);
    *out = b.record();
  }
}

// The same where every lane holds at most one column (score 0: none): the
// second reduction is needed only where a scoring column is tabu.
template <int kWaves>
__device__ __forceinline__ void block_record_one(double s, int j, int q, bool tabu, MoveRecord* out) {
  __shared__ MoveRecord rec[kWaves];
  BestPair b;
  if (s > 0.0) b.offer(s, j, q, tabu);
  b.all.wave_reduce();
  if (__any(tabu && s > 0.0))
    b.free.wave_reduce();
  else
    b.free = b.all;
  if ((threadIdx.x & (kWave - 1)) == 0) rec[threadIdx.x >> 6] = b.record();
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < kWaves; ++w) b.offer(rec[w]);
    *out = b.record();
  }
}

// The kept scores of columns gt, gt + gs, ... of a walk into `best`, but for
// those with mark(q) (read beside the score); with `copy` also the pending copy
// of a new incumbent for all of them. kU columns per thread and step, every load
// issued before any is used.
template <typename Mark>
__device__ __forceinline__ void scan_scores(const WalkCtx& C, int64_t k, bool copy, int gt, int gs, BestPair& best,
                                            Mark mark) {
  const gptr<const double> s = gmem((const double*)C.s);
  const gptr<const int32_t> tabu = gmem((const int32_t*)C.tabu);
  const gptr<const int32_t> perm = gmem(C.P.perm);
  const int32_t n = C.P.n;
  if (copy) {
    const gptr<const double> x = gmem((const double*)C.x);
    const gptr<double> best_x = gmem(C.best_x);
    for (int q = gt; q < n; q += gs) best_x[q] = x[q];
  }
  constexpr int kU = 8;
  for (int64_t q0 = gt; q0 < n; q0 += (int64_t)kU * gs) {
    double v[kU];
    int j[kU], tb[kU];
    bool skip[kU];
#pragma unroll
    for (int u = 0; u < kU; ++u) {
      const int64_t q = q0 + (int64_t)u * gs;
      v[u] = 0.0;
      if (q < n) {
        v[u] = s[q];
        j[u] = perm[q];
        tb[u] = tabu[q];
        skip[u] = mark((int)q);
      }
    }
#pragma unroll
    for (int u = 0; u < kU; ++u) {
      const int64_t q = q0 + (int64_t)u * gs;
      if (q < n && v[u] > 0.0 && !skip[u]) best.offer(v[u], j[u], (int)q, k <= (int64_t)tb[u]);
    }
  }
}

// The iteration the move selection that follows belongs to, and its violated
// rows: the selection's workgroups read this copy, which none of them writes
// (one thread of a kernel before it does).
__device__ __forceinline__ void snapshot(WalkState* st, bool active) {
  st->sel_k = active ? st->k : -1;
  st->sel_V = st->V;
}

}  // namespace chap
