// Inference and training kernels of the candidate-proposal network on
// gfx950 matrix cores (see mlp_core.h for the operand layout).
//
// Training minimises the mean squared error over a batch. The backward pass
// keeps the forward orientation: the output-layer signal g2 = W3^T g3 masked
// by the ReLU gate is already in B layout, so dL/dh1 = W2^T g2 is one more
// set of MFMAs with W2^T as the A operand. The weight gradients contract over
// the samples of a tile, which need the samples along k: the tile's g2, h1,
// g1 and inputs are transposed through LDS for those products. Every sum is
// taken in a fixed order (lanes, waves, workgroups), so a gradient is
// reproducible bit for bit.

#include <algorithm>

#include "chap_internal.h"
#include "mlp_core.h"

namespace chap {
namespace {

using namespace mlp;

constexpr int kWaves = 4;

// Loads the inputs of sample `row` in B layout (inputs 4g..4g+3), zero when
// the sample does not exist.
__device__ __forceinline__ bf16x4 load_inputs(const uint16_t* __restrict__ feat, int64_t row, bool valid) {
  const int g = (threadIdx.x & 63) >> 4;
  const bf16x4 zero = {0, 0, 0, 0};
  return valid ? *(const bf16x4*)(feat + row * kIn + 4 * g) : zero;
}

__global__ __launch_bounds__(256) void k_mlp_forward(const float* __restrict__ w, const uint16_t* __restrict__ wb,
                                                     const uint16_t* __restrict__ feat, int64_t n,
                                                     float* __restrict__ out) {
  Weights W;
  load_weights(wb, w, W);
  const int l = threadIdx.x & 63, r = l & 15;
  const int64_t ntiles = (n + 15) / 16;
  const int64_t stride = (int64_t)gridDim.x * kWaves;
  for (int64_t tile = (int64_t)blockIdx.x * kWaves + (threadIdx.x >> 6); tile < ntiles; tile += stride) {
    const int64_t row = tile * 16 + r;
    Acts A;
    forward(W, load_inputs(feat, row, row < n), A);
    if (l < 16 && row < n) out[row] = A.y;
  }
}

// Sum over the 16 lanes of a lane group (same g), fixed butterfly order: lane
// distances 1, 2, 4, 8 (the mirrors reach the same sums once four and eight
// neighbours agree), by DPP.
template <int kCtrl>
__device__ __forceinline__ float dpp_add(float v) {
  return v + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), kCtrl, 0xF, 0xF, true));
}
__device__ __forceinline__ float group16_sum(float v) {
  v = dpp_add<0xB1>(v);   // quad_perm [1, 0, 3, 2]
  v = dpp_add<0x4E>(v);   // quad_perm [2, 3, 0, 1]
  v = dpp_add<0x141>(v);  // row_half_mirror
  return dpp_add<0x140>(v);  // row_mirror
}

// The wavefront's own LDS slice, written and then read by its lanes.
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Per-workgroup gradient partials of the mean squared error over `nb`
// samples. Sample i is row i of (feat, target), or row
// splitmix64(seed, base + i) mod rows when `sample` is set. inv_nb = 1/nb.
// Writes partials[blockIdx.x][p] for every parameter p. With `advance`, an Adam
// step follows: its counter and the powers beta1^t, beta2^t (FP64) advance here.
// Bounded by the latency of one round (a batch of 1024 is 16 workgroups of four
// tiles): inputs are asked for before the weights, the next round's during this
// one, W2^T comes in operand layout, and the wavefronts' sums meet in LDS in one
// step; 9.2 us at 1024 samples, 16 before (W2^T by 64 two-byte loads a lane,
// wavefronts adding into one LDS copy in turn, exchanges through LDS).
struct GradSmem {
  uint16_t g2[kWaves][kHid * 16];
  uint16_t h1[kWaves][kHid * 16];
  uint16_t g1[kWaves][kHid * 16];
  uint16_t x[kWaves][kIn * 16];
  alignas(16) float sum[kWaves][kNParamPad];
};
__global__ __launch_bounds__(256) void k_mlp_grad(const float* __restrict__ w, const uint16_t* __restrict__ wb,
                                                  const uint16_t* __restrict__ feat,
                                                  const float* __restrict__ target, int64_t rows, int64_t nb,
                                                  int32_t sample, uint64_t seed, uint64_t base, float inv_nb,
                                                  float* __restrict__ partials, double* __restrict__ adam,
                                                  int32_t advance, const int32_t* active) {
  if (active && !*active) return;
  __shared__ GradSmem S;
  const int l = threadIdx.x & 63, g = l >> 4, r = l & 15;
  const int wv = threadIdx.x >> 6;
  if (advance && blockIdx.x == 0 && threadIdx.x == 0) {
    adam[0] *= kAdamBeta1;
    adam[1] *= kAdamBeta2;
    adam[2] += 1.0;
  }
  // inputs and target of this lane's sample of a round
  const int64_t ntiles = (nb + 15) / 16;
  const int64_t stride = (int64_t)gridDim.x * kWaves;
  auto load_sample = [&](int64_t tile, bf16x4& x, float& t) {
    const int64_t i = tile * 16 + r;
    const bool valid = i < nb;
    int64_t row = i;
    if (valid && sample) row = (int64_t)(splitmix64(seed, base + (uint64_t)i) % (uint64_t)rows);
    x = load_inputs(feat, row, valid);
    t = l < 16 && valid ? target[row] : 0.0f;
  };
  bf16x4 x;
  float tgt;
  load_sample((int64_t)blockIdx.x * kWaves + wv, x, tgt);
  Weights W;
  load_weights(wb, w, W);
  // W2^T in A layout: element (i = r, k = 4g + t) of block (ib, ob) is W2[16ob + 4g + t][16ib + r]
  bf16x4 a2t[4][4];
  float w3r[4][4];  // W3[16o + 4g + t] as FP32 (bfloat16 values)
#pragma unroll
  for (int ib = 0; ib < 4; ++ib)
#pragma unroll
    for (int ob = 0; ob < 4; ++ob) a2t[ib][ob] = *(const bf16x4*)(wb + kOffW2T + ((ib * 4 + ob) * 64 + l) * 4);
#pragma unroll
  for (int o = 0; o < 4; ++o) {
    const bf16x4 w3 = *(const bf16x4*)(wb + kOffW3 + 16 * o + 4 * g);
#pragma unroll
    for (int t = 0; t < 4; ++t) w3r[o][t] = bf2f((uint16_t)w3[t]);
  }

  const f32x4 zero4 = {0.0f, 0.0f, 0.0f, 0.0f};
  f32x4 accW2[4][4], accW1[4];
  float accW3[4][4], accB2[4][4], accB1[4][4], accB3 = 0.0f;
#pragma unroll
  for (int a = 0; a < 4; ++a) {
    accW1[a] = zero4;
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      accW2[a][b] = zero4;
      accW3[a][b] = 0.0f;
      accB2[a][b] = 0.0f;
      accB1[a][b] = 0.0f;
    }
  }

  // tiles past the end are all-zero samples with a zero output signal
  for (int64_t base_tile = (int64_t)blockIdx.x * kWaves; base_tile < ntiles; base_tile += stride) {
    const bool valid = (base_tile + wv) * 16 + r < nb;
    const bf16x4 x0 = x;
    const float t0 = tgt;
    if (base_tile + stride < ntiles) load_sample(base_tile + stride + wv, x, tgt);
    Acts A;
    forward(W, x0, A);
    // output signal g3 = 2 (y - t) / nb of sample r, broadcast to its column
    float g3 = 0.0f;
    if (l < 16 && valid) g3 = 2.0f * (A.y - t0) * inv_nb;
    g3 = __shfl(g3, r, 64);
    if (l < 16) accB3 += g3;
    // output layer and g2 = W3 g3 gated by z2 > 0
    bf16x4 g2b[4];
#pragma unroll
    for (int o = 0; o < 4; ++o) {
      float v[4];
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        accW3[o][t] += g3 * bf2f((uint16_t)A.h2[o][t]);
        v[t] = (A.z2[o][t] > 0.0f) ? g3 * w3r[o][t] : 0.0f;
        accB2[o][t] += v[t];
      }
      g2b[o] = to_bf16x4(v[0], v[1], v[2], v[3]);
    }
    // dL/dh1 = W2^T g2, gated by z1 > 0
    bf16x4 g1b[4];
#pragma unroll
    for (int ib = 0; ib < 4; ++ib) {
      f32x4 acc = zero4;
#pragma unroll
      for (int ob = 0; ob < 4; ++ob) acc = mma(a2t[ib][ob], g2b[ob], acc);
      float v[4];
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        v[t] = (A.z1[ib][t] > 0.0f) ? acc[t] : 0.0f;
        accB1[ib][t] += v[t];
      }
      g1b[ib] = to_bf16x4(v[0], v[1], v[2], v[3]);
    }
    // transpose the tile through LDS: unit-major rows of 16 samples
#pragma unroll
    for (int b = 0; b < 4; ++b)
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const int u = 16 * b + 4 * g + t;
        S.g2[wv][u * 16 + r] = (uint16_t)g2b[b][t];
        S.h1[wv][u * 16 + r] = (uint16_t)A.h1[b][t];
        S.g1[wv][u * 16 + r] = (uint16_t)g1b[b][t];
      }
#pragma unroll
    for (int t = 0; t < 4; ++t) S.x[wv][(4 * g + t) * 16 + r] = (uint16_t)x0[t];
    wave_sync();
    // dW2[o][i] += sum_s g2[o][s] h1[i][s];  dW1[h][f] += sum_s g1[h][s] x[f][s]
    bf16x4 h1t[4];
#pragma unroll
    for (int ib = 0; ib < 4; ++ib) h1t[ib] = *(const bf16x4*)&S.h1[wv][(16 * ib + r) * 16 + 4 * g];
#pragma unroll
    for (int ob = 0; ob < 4; ++ob) {
      const bf16x4 g2t = *(const bf16x4*)&S.g2[wv][(16 * ob + r) * 16 + 4 * g];
#pragma unroll
      for (int ib = 0; ib < 4; ++ib) accW2[ob][ib] = mma(g2t, h1t[ib], accW2[ob][ib]);
    }
    const bf16x4 xt = *(const bf16x4*)&S.x[wv][r * 16 + 4 * g];
#pragma unroll
    for (int hb = 0; hb < 4; ++hb) {
      const bf16x4 g1t = *(const bf16x4*)&S.g1[wv][(16 * hb + r) * 16 + 4 * g];
      accW1[hb] = mma(g1t, xt, accW1[hb]);
    }
    wave_sync();
  }
  // lane-group sums of the per-lane accumulators
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      accW3[a][t] = group16_sum(accW3[a][t]);
      accB2[a][t] = group16_sum(accB2[a][t]);
      accB1[a][t] = group16_sum(accB1[a][t]);
    }
  accB3 = group16_sum(accB3);
  // workgroup sum in wave order
  float* sum = S.sum[wv];
#pragma unroll
  for (int ob = 0; ob < 4; ++ob)
#pragma unroll
    for (int ib = 0; ib < 4; ++ib)
#pragma unroll
      for (int t = 0; t < 4; ++t) sum[kOffW2 + (16 * ob + 4 * g + t) * kHid + 16 * ib + r] = accW2[ob][ib][t];
#pragma unroll
  for (int hb = 0; hb < 4; ++hb)
#pragma unroll
    for (int t = 0; t < 4; ++t) sum[kOffW1 + (16 * hb + 4 * g + t) * kIn + r] = accW1[hb][t];
  if (r == 0) {
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        sum[kOffW3 + 16 * a + 4 * g + t] = accW3[a][t];
        sum[kOffB2 + 16 * a + 4 * g + t] = accB2[a][t];
        sum[kOffB1 + 16 * a + 4 * g + t] = accB1[a][t];
      }
  }
  if (l == 0) sum[kOffB3] = accB3;
  __syncthreads();
  float* mine = partials + (int64_t)blockIdx.x * kNParamPad;
  for (int p = 4 * threadIdx.x; p < kNParam; p += 4 * blockDim.x) {  // whole fours: both rows are padded
    f32x4 v = zero4;
#pragma unroll
    for (int w2 = 0; w2 < kWaves; ++w2) v += *(const f32x4*)&S.sum[w2][p];
    *(f32x4*)&mine[p] = v;
  }
}

// The operand copies of parameter p: its bfloat16 value, and a W2 entry's place
// in the transposed layout.
__device__ __forceinline__ void store_bf16(uint16_t* wb, int p, float v) {
  const uint16_t h = f2bf(v);
  wb[p] = h;
  if (p >= kOffW2 && p < kOffB2) {
    const int o = (p - kOffW2) / kHid, i = (p - kOffW2) % kHid;
    wb[kOffW2T + (((i >> 4) * 4 + (o >> 4)) * 64 + ((o >> 2) & 3) * 16 + (i & 15)) * 4 + (o & 3)] = h;
  }
}

constexpr int kReduceThreads = 64;   // one wavefront, so that the parameters spread over many CUs
constexpr int kReduceInFlight = 16;  // partials loaded at a time

// Sums the partials in workgroup order into grad; with `update`, one Adam
// step on the FP32 parameters and a fresh bfloat16 copy. omb1 and omb2 are
// 1 - beta1 and 1 - beta2 rounded once from FP64.
__global__ __launch_bounds__(kReduceThreads) void k_mlp_reduce(float* __restrict__ w, uint16_t* __restrict__ wb,
                                                    float* __restrict__ m, float* __restrict__ v,
                                                    const double* __restrict__ adam, float* __restrict__ grad,
                                                    const float* __restrict__ partials, int32_t nparts,
                                                    int32_t update, float lr, float beta1, float omb1, float beta2,
                                                    float omb2, float eps, const int32_t* active) {
  if (active && !*active) return;
  const int p = blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= kNParam) return;
  float gsum = 0.0f;
  for (int b0 = 0; b0 < nparts; b0 += kReduceInFlight) {
    float v[kReduceInFlight];
#pragma unroll
    for (int k = 0; k < kReduceInFlight; ++k)
      v[k] = b0 + k < nparts ? partials[(int64_t)(b0 + k) * kNParamPad + p] : 0.0f;
#pragma unroll
    for (int k = 0; k < kReduceInFlight; ++k)
      if (b0 + k < nparts) gsum += v[k];
  }
  grad[p] = gsum;
  if (!update) return;
  const float mo = beta1 * m[p] + omb1 * gsum;
  const float vo = beta2 * v[p] + omb2 * gsum * gsum;
  m[p] = mo;
  v[p] = vo;
  const float c1 = (float)(1.0 - adam[0]);
  const float c2 = (float)(1.0 - adam[1]);
  const float mh = mo / c1;
  const float vh = vo / c2;
  const float nw = w[p] - lr * mh / (sqrtf(vh) + eps);
  w[p] = nw;
  store_bf16(wb, p, nw);
}

__global__ __launch_bounds__(256) void k_mlp_bf16_copy(const float* __restrict__ w, uint16_t* __restrict__ wb) {
  const int p = blockIdx.x * blockDim.x + threadIdx.x;
  if (p < kNParam) store_bf16(wb, p, w[p]);
}

}  // namespace

hipError_t launch_mlp_forward(const ModelDev& M, const uint16_t* feat, int64_t n, float* out, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  const int64_t tiles = (n + 15) / 16;
  const int64_t blocks = std::min<int64_t>((tiles + kWaves - 1) / kWaves, 4096);
  hipLaunchKernelGGL(k_mlp_forward, dim3((unsigned)blocks), dim3(256), 0, s, M.w, M.wb, feat, n, out);
  return hipGetLastError();
}

int32_t mlp_grad_blocks(int64_t nb) {
  const int64_t tiles = (nb + 15) / 16;
  return (int32_t)std::max<int64_t>(1, std::min<int64_t>((tiles + kWaves - 1) / kWaves, kGradBlocks));
}

hipError_t grad_impl(const ModelDev& M, const int32_t* active, const uint16_t* feat, const float* target,
                     int64_t rows, int64_t nb, int sample, int advance, uint64_t seed, uint64_t base, hipStream_t s) {
  const int32_t blocks = mlp_grad_blocks(nb);
  hipLaunchKernelGGL(k_mlp_grad, dim3((unsigned)blocks), dim3(256), 0, s, M.w, M.wb, feat, target, rows, nb,
                     (int32_t)sample, seed, base, (float)(1.0 / (double)nb), M.partials, M.adam, (int32_t)advance,
                     active);
  return hipGetLastError();
}

hipError_t reduce_impl(const ModelDev& M, const int32_t* active, int64_t nb, int update, float lr, hipStream_t s) {
  hipLaunchKernelGGL(k_mlp_reduce, dim3((kNParam + kReduceThreads - 1) / kReduceThreads), dim3(kReduceThreads), 0, s,
                     M.w, M.wb, M.m, M.v, M.adam, M.grad, M.partials, mlp_grad_blocks(nb), (int32_t)update, lr,
                     (float)kAdamBeta1, (float)(1.0 - kAdamBeta1), (float)kAdamBeta2, (float)(1.0 - kAdamBeta2),
                     kAdamEps, active);
  return hipGetLastError();
}

hipError_t launch_mlp_grad(const ModelDev& M, const uint16_t* feat, const float* target, int64_t rows, int64_t nb,
                           int sample, int update, uint64_t seed, uint64_t base, hipStream_t s) {
  return grad_impl(M, nullptr, feat, target, rows, nb, sample, update, seed, base, s);
}

hipError_t launch_mlp_reduce(const ModelDev& M, int64_t nb, int update, float lr, hipStream_t s) {
  return reduce_impl(M, nullptr, nb, update, lr, s);
}

hipError_t launch_mlp_grad_guarded(const ModelDev& M, const int32_t* active, const uint16_t* feat,
                                   const float* target, int64_t nb, hipStream_t s) {
  return grad_impl(M, active, feat, target, nb, nb, 0, 1, 0, 0, s);
}

hipError_t launch_mlp_reduce_guarded(const ModelDev& M, const int32_t* active, int64_t nb, float lr, hipStream_t s) {
  return reduce_impl(M, active, nb, 1, lr, s);
}

hipError_t launch_mlp_bf16_copy(const ModelDev& M, hipStream_t s) {
  hipLaunchKernelGGL(k_mlp_bf16_copy, dim3((kNParam + 255) / 256), dim3(256), 0, s, M.w, M.wb);
  return hipGetLastError();
}

}  // namespace chap
