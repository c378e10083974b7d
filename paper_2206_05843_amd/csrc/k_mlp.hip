// Learned rewrite policy: level features, and the network's forward, backward
// and Adam kernels (FP32). The network is 20 -> 64 -> 64 -> 1 with ReLU and a
// sigmoid output; one wave evaluates one sample with lane j holding hidden unit
// j of both layers, so every reduction is a fixed butterfly or a fixed loop
// (deterministic). A lane keeps its unit's weights (and, for the backward pass,
// its column of W2 and its gradient sums) in registers; only a sample's
// activations go through LDS, read back four at a time by all lanes at once.
#include "common.h"

namespace {

constexpr int NIN = 20, HID = 64, NPAR = 5569;
constexpr int OFF_W1 = 0, OFF_B1 = OFF_W1 + HID * NIN, OFF_W2 = OFF_B1 + HID, OFF_B2 = OFF_W2 + HID * HID,
              OFF_W3 = OFF_B2 + HID, OFF_B3 = OFF_W3 + HID;
static_assert(OFF_B3 + 1 == NPAR, "parameter layout");
constexpr int W1S = NIN + 1, W2S = HID + 1;  // padded LDS row strides
constexpr int kWavesPerBlock = 4;
constexpr int kBlocks = 256;  // one workgroup per CU: a wave keeps some 270 registers

struct SParams {
  float w1[HID * W1S];
  float b1[HID];
  float w2[HID * W2S];
  float b2[HID];
  float w3[HID];
  float b3;
};

__device__ void load_params(SParams &sp, const float *__restrict__ P) {
  for (int i = threadIdx.x; i < HID * NIN; i += blockDim.x) sp.w1[(i / NIN) * W1S + i % NIN] = P[OFF_W1 + i];
  for (int i = threadIdx.x; i < HID * HID; i += blockDim.x) sp.w2[(i / HID) * W2S + i % HID] = P[OFF_W2 + i];
  for (int i = threadIdx.x; i < HID; i += blockDim.x) {
    sp.b1[i] = P[OFF_B1 + i];
    sp.b2[i] = P[OFF_B2 + i];
    sp.w3[i] = P[OFF_W3 + i];
  }
  if (threadIdx.x == 0) sp.b3 = P[OFF_B3];
}

__device__ __forceinline__ float wave_sum(float v) {
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}

__device__ __forceinline__ void wsync() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local");
  __builtin_amdgcn_wave_barrier();
}

// One wave's unit of both layers in registers.
struct Unit {
  float w1[NIN], w2[HID], b1, b2, w3, b3;
};

__device__ __forceinline__ Unit load_unit(const SParams &sp, int j) {
  Unit u;
#pragma unroll
  for (int k = 0; k < NIN; ++k) u.w1[k] = sp.w1[j * W1S + k];
#pragma unroll
  for (int i = 0; i < HID; ++i) u.w2[i] = sp.w2[j * W2S + i];
  u.b1 = sp.b1[j], u.b2 = sp.b2[j], u.w3 = sp.w3[j], u.b3 = sp.b3;
  return u;
}

// A sample's normalised features and its 64 activations of one layer, per wave.
struct __align__(16) Acts {
  float f[NIN], h[HID], d[HID];
};

// acc + sum_i w[i] x[i] in order, x read four at a time.
template <int N>
__device__ __forceinline__ float dot_lds(float acc, const float (&w)[N], const float *x) {
#pragma unroll
  for (int i = 0; i < N; i += 4) {
    const float4 v = *reinterpret_cast<const float4 *>(x + i);
    acc += w[i] * v.x;
    acc += w[i + 1] * v.y;
    acc += w[i + 2] * v.z;
    acc += w[i + 3] * v.w;
  }
  return acc;
}

// Forward pass of one sample by one wave (feat: lane j < 20 holds feature j).
// Leaves the normalised features in s.f, h1 in s.h; returns (a1, a2, h2) of
// this lane's unit and z.
struct Fwd {
  float a1, a2, h2, z;
};

__device__ __forceinline__ Fwd forward_one(const Unit &u, float feat, Acts &s) {
  const int j = threadIdx.x & 63;
  if (j < NIN) s.f[j] = feat;
  wsync();
  const float a1 = dot_lds(u.b1, u.w1, s.f);
  s.h[j] = fmaxf(a1, 0.f);
  wsync();
  const float a2 = dot_lds(u.b2, u.w2, s.h);
  const float h2 = fmaxf(a2, 0.f);
  const float z = wave_sum(u.w3 * h2) + u.b3;
  return Fwd{a1, a2, h2, z};
}

// Normalised feature j of sample b (0 for lanes past the features).
__device__ __forceinline__ float feature(const float *__restrict__ feat, const float *__restrict__ norm, int64_t b,
                                         int j) {
  if (j >= NIN) return 0.f;
  float f = feat[b * NIN + j];
  if (norm) f = (f - norm[j]) * norm[NIN + j];
  return f;
}

__global__ __launch_bounds__(64 * kWavesPerBlock) void k_mlp_forward(const float *__restrict__ P,
                                                                       const float *__restrict__ feat,
                                                                       const float *__restrict__ norm, int32_t B,
                                                                       float *prob) {
  __shared__ SParams sp;
  __shared__ Acts acts[kWavesPerBlock];
  load_params(sp, P);
  __syncthreads();
  const int w = threadIdx.x >> 6, j = threadIdx.x & 63;
  const Unit u = load_unit(sp, j);
  const int64_t step = (int64_t)gridDim.x * kWavesPerBlock;
  int64_t b = (int64_t)blockIdx.x * kWavesPerBlock + w;
  float f = b < B ? feature(feat, norm, b, j) : 0.f;
  for (; b < B; b += step) {
    const float cur = f;
    f = b + step < B ? feature(feat, norm, b + step, j) : 0.f;
    const Fwd r = forward_one(u, cur, acts[w]);
    if (j == 0) prob[b] = 1.f / (1.f + expf(-r.z));
    wsync();
  }
}

// Per-workgroup partial gradients of sum_b w_b BCE_b / B, written to
// part[workgroup][*]: every wave sums its samples in registers, then the waves
// are added in order. Bound by the 230 FMAs a sample costs each lane; with one
// wave per SIMD and the waves' sums added in LDS, 4,096 samples take 23 us (44 with
// 64 workgroups whose lanes read every weight from LDS for each sample).
__global__ __launch_bounds__(64 * kWavesPerBlock, 1) void k_mlp_backward(
    const float *__restrict__ P, const float *__restrict__ feat, const float *__restrict__ norm,
    const float *__restrict__ label, const float *__restrict__ weight, int32_t B, float *part, float *part_loss) {
  __shared__ SParams sp;
  __shared__ Acts acts[kWavesPerBlock];
  __shared__ float s_loss;
  load_params(sp, P);
  __syncthreads();
  const int w = threadIdx.x >> 6, j = threadIdx.x & 63;
  const Unit u = load_unit(sp, j);
  float w2c[HID];  // column j of W2
#pragma unroll
  for (int i = 0; i < HID; ++i) w2c[i] = sp.w2[i * W2S + j];
  Acts &s = acts[w];
  float gw1[NIN], gw2[HID];
#pragma unroll
  for (int k = 0; k < NIN; ++k) gw1[k] = 0.f;
#pragma unroll
  for (int i = 0; i < HID; ++i) gw2[i] = 0.f;
  float gb1 = 0.f, gb2 = 0.f, gw3 = 0.f, gb3 = 0.f, loss = 0.f;
  const float invB = 1.f / (float)B;
  const int64_t step = (int64_t)gridDim.x * kWavesPerBlock;
  int64_t b = (int64_t)blockIdx.x * kWavesPerBlock + w;
  float f = b < B ? feature(feat, norm, b, j) : 0.f;
  for (; b < B; b += step) {
    const float cur = f;
    const float y = label[b], wt = weight ? weight[b] : 1.f;
    f = b + step < B ? feature(feat, norm, b + step, j) : 0.f;
    const Fwd r = forward_one(u, cur, s);
    const float p = 1.f / (1.f + expf(-r.z));
    const float dz = wt * (p - y) * invB;
    if (j == 0) {
      loss += wt * (fmaxf(r.z, 0.f) - r.z * y + log1pf(expf(-fabsf(r.z))));
      gb3 += dz;
    }
    gw3 += dz * r.h2;
    const float da2 = r.a2 > 0.f ? dz * u.w3 : 0.f;
    gb2 += da2;
    s.d[j] = da2;
#pragma unroll
    for (int i = 0; i < HID; i += 4) {
      const float4 v = *reinterpret_cast<const float4 *>(s.h + i);
      gw2[i] += da2 * v.x;
      gw2[i + 1] += da2 * v.y;
      gw2[i + 2] += da2 * v.z;
      gw2[i + 3] += da2 * v.w;
    }
    wsync();
    const float dh1 = dot_lds(0.f, w2c, s.d);
    const float da1 = r.a1 > 0.f ? dh1 : 0.f;
    gb1 += da1;
#pragma unroll
    for (int k = 0; k < NIN; k += 4) {
      const float4 v = *reinterpret_cast<const float4 *>(s.f + k);
      gw1[k] += da1 * v.x;
      gw1[k + 1] += da1 * v.y;
      gw1[k + 2] += da1 * v.z;
      gw1[k + 3] += da1 * v.w;
    }
    wsync();
  }
  // the parameters are in registers: their place in LDS takes the sums
  for (int q = 0; q < kWavesPerBlock; ++q) {
    __syncthreads();
    if (w != q) continue;
    auto add = [&](float &to, float v) { to = q == 0 ? v : to + v; };
#pragma unroll
    for (int k = 0; k < NIN; ++k) add(sp.w1[j * W1S + k], gw1[k]);
#pragma unroll
    for (int i = 0; i < HID; ++i) add(sp.w2[j * W2S + i], gw2[i]);
    add(sp.b1[j], gb1);
    add(sp.b2[j], gb2);
    add(sp.w3[j], gw3);
    if (j == 0) {
      add(sp.b3, gb3);
      add(s_loss, loss);
    }
  }
  __syncthreads();
  float *o = part + (int64_t)blockIdx.x * NPAR;
  for (int i = threadIdx.x; i < HID * NIN; i += blockDim.x) o[OFF_W1 + i] = sp.w1[(i / NIN) * W1S + i % NIN];
  for (int i = threadIdx.x; i < HID * HID; i += blockDim.x) o[OFF_W2 + i] = sp.w2[(i / HID) * W2S + i % HID];
  if (threadIdx.x < HID) {
    o[OFF_B1 + threadIdx.x] = sp.b1[threadIdx.x];
    o[OFF_B2 + threadIdx.x] = sp.b2[threadIdx.x];
    o[OFF_W3 + threadIdx.x] = sp.w3[threadIdx.x];
  }
  if (threadIdx.x == 0) {
    o[OFF_B3] = sp.b3;
    part_loss[blockIdx.x] = s_loss * invB;
  }
}

// grad[i] = sum over workgroups of part[q][i]: kRedRows threads of a column sum
// every kRedRows-th part, then their sums are added in order. A workgroup takes
// 32 columns (a 128-byte line a part), so the 5,570 sums of 256 parts are read
// by 175 workgroups at once (4 us; one thread per column read them one by one, 63 us).
constexpr int kRedCols = 32, kRedRows = 16;
__global__ __launch_bounds__(kRedCols * kRedRows) void k_mlp_reduce(const float *__restrict__ part, int32_t nparts,
                                                                     const float *__restrict__ part_loss, float *grad,
                                                                     float *loss) {
  __shared__ float sum[kRedRows][kRedCols];
  const int c = threadIdx.x % kRedCols, r = threadIdx.x / kRedCols;
  const int i = blockIdx.x * kRedCols + c;
  float s = 0.f;
  if (i <= NPAR) {
    const float *from = i < NPAR ? part + i : part_loss;
    const int64_t stride = i < NPAR ? NPAR : 1;
#pragma unroll 8
    for (int q = r; q < nparts; q += kRedRows) s += from[(int64_t)q * stride];
  }
  sum[r][c] = s;
  __syncthreads();
  if (r == 0 && i <= NPAR) {
    for (int q = 1; q < kRedRows; ++q) s += sum[q][c];
    if (i < NPAR)
      grad[i] = s;
    else
      *loss = s;
  }
}

__global__ void k_mlp_adam(float *P, const float *__restrict__ g, float *m, float *v, float lr, float c1, float c2) {
  const float b1 = 0.9f, b2 = 0.999f, eps = 1e-8f;
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < NPAR; i += gridDim.x * blockDim.x) {
    const float gi = g[i];
    const float mi = b1 * m[i] + (1.f - b1) * gi;
    const float vi = b2 * v[i] + (1.f - b2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    P[i] -= lr * (mi / c1) / (sqrtf(vi / c2) + eps);
  }
}

__global__ void k_mlp_mask(const float *__restrict__ prob, int32_t nlev, float thr, uint8_t *mask) {
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < nlev; i += gridDim.x * blockDim.x)
    mask[i] = (i > 0 && prob[i] >= thr) ? 1 : 0;
}

// Tiered actions: a level takes the highest tier whose threshold its
// probability reaches (thresholds ascending) and becomes a source with that
// tier's target budget and fill cap; below the first threshold, and at level
// 0, it is not a source (budget and cap 0: the rewrite's own values).
__global__ void k_mlp_actions(const float *__restrict__ prob, int32_t nlev, MlpTiers t, uint8_t *mask,
                              int32_t *budget, float *cap) {
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < nlev; i += gridDim.x * blockDim.x) {
    int k = -1;
    if (i > 0)
      for (int j = 0; j < t.n; ++j)
        if (prob[i] >= t.thr[j]) k = j;
    mask[i] = k >= 0 ? 1 : 0;
    budget[i] = k >= 0 ? t.budget[k] : 0;
    cap[i] = k >= 0 ? t.cap[k] : 0.0f;
  }
}

// The 20 features of each level (see sptrsv_level_features), from the level
// statistics and the per-row sums of the distance-1 rewrite.
__global__ void k_feat_finalize(int32_t nlev, const int64_t *__restrict__ rows, const int64_t *__restrict__ nnz,
                                const int64_t *__restrict__ cost, double avg, FeatAcc acc, float *feat) {
  for (int64_t l = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; l < nlev; l += (int64_t)gridDim.x * blockDim.x) {
    float *f = feat + l * NIN;
    const int32_t *hist = acc.hist + l * kFeatHist;
    const double R = (double)rows[l];
    f[0] = (float)log1p(R);
    f[1] = (float)log1p((double)nnz[l]);
    f[2] = (float)log1p((double)cost[l]);
    f[3] = (float)(avg > 0.0 ? (double)cost[l] / avg : 0.0);
    f[4] = (float)(R / 32.0);
    f[5] = (float)(R > 0.0 ? (double)nnz[l] / R : 0.0);
    for (int b = 0; b < 6; ++b) f[6 + b] = (float)(R > 0.0 ? (double)hist[b] / R : 0.0);
    f[12] = (float)(nnz[l] > 0 ? (double)acc.sum_lp[l] / (double)nnz[l] : 0.0);
    f[13] = (float)log1p((double)acc.sum_t[l]);
    f[14] = (float)((double)l / (double)nlev);
    f[15] = (float)(l > 0 ? log1p((double)rows[l - 1]) : 0.0);
    f[16] = (float)(R > 0.0 ? (double)hist[6] / R : 0.0);
    f[17] = (float)(R > 0.0 ? (double)hist[7] / R : 0.0);
    f[18] = (float)(R > 0.0 ? log1p((double)acc.sum_span[l] / R) : 0.0);
    f[19] = (float)(R > 0.0 ? (double)hist[8] / R : 0.0);
  }
}

}  // namespace

int mlp_backward_parts() { return kBlocks; }

hipError_t launch_mlp_forward(const float *P, const float *feat, const float *norm, int32_t B, float *prob,
                              hipStream_t s) {
  if (B <= 0) return hipSuccess;
  const int g = grid_for(B, kWavesPerBlock, 2 * kBlocks);
  hipLaunchKernelGGL(k_mlp_forward, dim3(g), dim3(64 * kWavesPerBlock), 0, s, P, feat, norm, B, prob);
  return hipGetLastError();
}

hipError_t launch_mlp_backward(const float *P, const float *feat, const float *norm, const float *label,
                               const float *weight, int32_t B, float *part, float *part_loss, float *grad,
                               float *loss, hipStream_t s) {
  const int g = grid_for(B, kWavesPerBlock, kBlocks);
  hipLaunchKernelGGL(k_mlp_backward, dim3(g), dim3(64 * kWavesPerBlock), 0, s, P, feat, norm, label, weight, B, part,
                     part_loss);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_mlp_reduce, dim3((NPAR + kRedCols) / kRedCols), dim3(kRedCols * kRedRows), 0, s, part, g,
                     part_loss, grad, loss);
  return hipGetLastError();
}

hipError_t launch_mlp_adam(float *P, const float *g, float *m, float *v, float lr, float c1, float c2,
                           hipStream_t s) {
  hipLaunchKernelGGL(k_mlp_adam, dim3((NPAR + 255) / 256), dim3(256), 0, s, P, g, m, v, lr, c1, c2);
  return hipGetLastError();
}

hipError_t launch_mlp_mask(const float *prob, int32_t nlev, float thr, uint8_t *mask, hipStream_t s) {
  if (nlev <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_mlp_mask, dim3((nlev + 255) / 256), dim3(256), 0, s, prob, nlev, thr, mask);
  return hipGetLastError();
}

hipError_t launch_mlp_actions(const float *prob, int32_t nlev, const MlpTiers &t, uint8_t *mask, int32_t *budget,
                              float *cap, hipStream_t s) {
  if (nlev <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_mlp_actions, dim3((nlev + 255) / 256 > 1024 ? 1024 : (nlev + 255) / 256), dim3(256), 0, s,
                     prob, nlev, t, mask, budget, cap);
  return hipGetLastError();
}

hipError_t launch_feat_finalize(int32_t nlev, const int64_t *rows, const int64_t *nnz, const int64_t *cost,
                                double avg, FeatAcc acc, float *feat, hipStream_t s) {
  if (nlev <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_feat_finalize, dim3((nlev + 255) / 256 > 1024 ? 1024 : (nlev + 255) / 256), dim3(256), 0, s,
                     nlev, rows, nnz, cost, avg, acc, feat);
  return hipGetLastError();
}
