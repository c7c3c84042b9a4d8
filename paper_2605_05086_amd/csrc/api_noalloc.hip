// chap_best_shift_noalloc: the single best-shift pass for callers that cannot
// allocate device memory (code under HIP graph capture, serving loops,
// harnesses that forbid hipMalloc). Every per-call buffer of the pass (the
// point in internal order and its byte copy, row states and their compact
// copy, walk state, set-up partials, the exact objective sum, staged records,
// long-column partials and sort scratch, the launch record) is carved from
// one file-scope device array, `scratch`, of kNoAllocBytes per GPU; the
// kernels are the ones chap_best_shift runs, launched one by one on the
// caller's stream (no graph, no side streams, no events).

#include <mutex>
#include <string>

#include "call_begin.h"
#include "chap_internal.h"

using namespace chap;

namespace {

constexpr int kMaxDevices = 64;

static __device__ __align__(256) unsigned char scratch[kNoAllocBytes];

std::mutex g_mu;
void* g_scratch[kMaxDevices] = {};   // device address of `scratch` on each device
uint32_t g_epoch[kMaxDevices] = {};  // call counter per device (byte copies of x)

// First kernel of a call: the walk record into scratch, the set-up ticket
// cleared, the state of a call without a cutoff row (workgroup 0), and the
// point in internal order with its byte copy.
__global__ __launch_bounds__(256) void k_noalloc_begin(WalkCtx r, WalkCtx* dst, uint32_t* ticket,
                                                       SingleInit init, const int32_t* __restrict__ perm,
                                                       const double* __restrict__ src, double* __restrict__ x,
                                                       int8_t* __restrict__ xc, WalkState* st, uint32_t epoch,
                                                       int32_t n) {
  static_assert(sizeof(WalkCtx) % 4 == 0, "copied as 32-bit words");
  if (blockIdx.x == 0) {
    const uint32_t* from = reinterpret_cast<const uint32_t*>(&r);
    uint32_t* out = reinterpret_cast<uint32_t*>(dst);
    for (int i = threadIdx.x; i < (int)(sizeof(WalkCtx) / 4); i += blockDim.x) out[i] = from[i];
    if (threadIdx.x == 0) {
      *ticket = 0u;
      if (init.cutoff_w) single_state(st, init);
    }
  }
  const int q = blockIdx.x * blockDim.x + threadIdx.x;
  if (q >= n) return;
  const double v = src[perm[q]];
  x[q] = v;
  if (xc) stage_byte(v, q, xc, st, epoch);
}

// Hands out 256-byte aligned pieces of [base, base + cap); used + size
// report what a call needs, whether or not it fits.
struct Carve {
  unsigned char* base;
  size_t cap;
  size_t used = 0;
  template <typename T>
  T* take(size_t count) {
    const size_t at = (used + 255) & ~(size_t)255;
    used = at + std::max<size_t>(count, 1) * sizeof(T);
    return used <= cap ? reinterpret_cast<T*>(base + at) : nullptr;
  }
};

// Every per-call buffer of a pass over p: the walk context's, and the set-up's.
struct Buffers {
  int8_t* xc;
  double* partial;
  long long* objacc;
  WalkCtx* rec;
  uint32_t* ticket;
};

Buffers carve(const chap_problem* p, int64_t stage_ent, Carve& cv, WalkCtx& c) {
  const size_t n = (size_t)p->n, m = (size_t)p->m;
  const PassPlan& plan = p->plan;
  c.x = cv.take<double>(n);
  c.xhat = cv.take<double>(n);
  c.s = cv.take<double>(n);
  c.rs = cv.take<RowState>(m);
  c.grow = p->compact_ok ? cv.take<GatherRow>(m) : nullptr;
  c.st = cv.take<WalkState>(1);
  c.partials = cv.take<ChunkPartial>((size_t)plan.n_partials);
  c.long_pos = cv.take<double>((size_t)plan.long_scratch);
  c.long_delta = cv.take<double>((size_t)plan.long_scratch);
  c.long_marker = cv.take<int32_t>((size_t)plan.long_scratch);
  c.stage_rec = cv.take<uint64_t>((size_t)stage_ent);
  Buffers b;
  b.xc = p->x_small ? cv.take<int8_t>(n) : nullptr;
  b.partial = cv.take<double>(kInitPartial);
  b.objacc = p->obj_fast ? nullptr : cv.take<long long>(kExactLimbs);
  b.rec = cv.take<WalkCtx>(1);
  b.ticket = cv.take<uint32_t>(1);
  return b;
}

int scratch_of_device(int dev, void** out) {
  if (dev < 0 || dev >= kMaxDevices) return fail(CHAP_EINVAL, "chap_best_shift_noalloc: device index out of range");
  std::lock_guard<std::mutex> lock(g_mu);
  if (!g_scratch[dev]) {
    void* ptr = nullptr;
    const hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !ptr)
      return fail(CHAP_EHIP, std::string("hipGetSymbolAddress(scratch): ") + hipGetErrorString(e));
    g_scratch[dev] = ptr;
  }
  *out = g_scratch[dev];
  return CHAP_OK;
}

}  // namespace

namespace chap {

size_t noalloc_bytes(const chap_problem* p, int64_t stage_ent) {
  Carve cv{nullptr, 0};
  WalkCtx c{};
  (void)carve(p, stage_ent, cv, c);
  return cv.used;
}

}  // namespace chap

extern "C" {

int chap_best_shift_noalloc(chap_problem* p, const double* d_x, const float* d_w, double cutoff_rhs,
                            double* d_shift, double* d_score, void* hip_stream) {
  if (!p) return fail(CHAP_EINVAL, "chap_best_shift_noalloc: null problem");
  if (p->n > 0 && (!d_x || !d_shift || !d_score))
    return fail(CHAP_EINVAL, "chap_best_shift_noalloc: null device array");
  if (!d_w) return fail(CHAP_EINVAL, "chap_best_shift_noalloc: null weights");
  if (std::isnan(cutoff_rhs)) return fail(CHAP_EINVAL, "chap_best_shift_noalloc: cutoff_rhs is NaN");
  int dev = 0;
  CHAP_HIP(hipGetDevice(&dev));
  if (dev != p->device)
    return fail(CHAP_EINVAL, "chap_best_shift_noalloc: the problem lives on device " + std::to_string(p->device) +
                                 ", device " + std::to_string(dev) + " is current");
  void* base = nullptr;
  int rc = scratch_of_device(dev, &base);
  if (rc != CHAP_OK) return rc;
  const int32_t n = p->n;
  Carve cv{(unsigned char*)base, kNoAllocBytes};
  WalkCtx c{};
  c.P = p->dev;
  c.plan = p->plan;
  const Buffers b = carve(p, p->plan.n_stage_ent, cv, c);
  if (cv.used > cv.cap)
    return fail(CHAP_EINVAL, "chap_best_shift_noalloc: this problem needs " + std::to_string(cv.used) +
                                 " bytes of scratch, more than the " + std::to_string(kNoAllocBytes) +
                                 " the entry point holds per device (use chap_best_shift)");
  BatchLaunch L;
  L.nw = 1;
  L.walks = b.rec;
  L.stage_pairs = c.plan.stage_pairs;
  for (int k = 0; k < KS_COUNT; ++k) {
    L.total[k] = kernel_blocks(c, k);
    L.grid[k] = L.total[k];
  }
  L.compact = p->compact_ok ? 2 : 0;
  L.caller_weights = 1;
  hipStream_t s = (hipStream_t)hip_stream;
  uint32_t epoch;
  {
    std::lock_guard<std::mutex> lock(g_mu);
    epoch = ++g_epoch[dev] == 0 ? ++g_epoch[dev] : g_epoch[dev];  // never 0
  }
  const bool cut = std::isfinite(cutoff_rhs);
  SingleInit init;
  if (!cut) {
    init.cutoff_w = d_w + p->mp;
    init.obj_integral = p->obj_integral;
  }
  hipLaunchKernelGGL(k_noalloc_begin, dim3((unsigned)std::max(1, (n + 255) / 256)), dim3(256), 0, s, c, b.rec,
                     b.ticket, init, p->dev.perm, d_x, c.x, b.xc, c.st, epoch, n);
  CHAP_HIP(hipGetLastError());
  if (cut)
    CHAP_HIP(launch_state_init(p->dev, c.x, c.rs, c.st, b.partial, b.ticket, b.objacc, 1, 0, p->obj_integral,
                               cutoff_rhs, d_w + p->mp, 0, 0, s));
  CHAP_HIP(launch_residual_scatter(p->dev, p->d_nidx, p->d_pair, d_w, c.x, b.xc, c.st, epoch, c.rs, s, c.grow));
  if (n > 0) CHAP_HIP(launch_pass(L, s, nullptr, false));
  CHAP_HIP(launch_gather2(p->d_inv, c.xhat, c.s, d_shift, d_score, n, s));
  return CHAP_OK;
}

size_t chap_best_shift_noalloc_max_bytes(void) { return kNoAllocBytes; }

}  // extern "C"
