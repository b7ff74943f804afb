// Learned cost model on the GPU: forward pass, back-propagation and Adam for the 3-layer
// perceptron f -> 64 -> 64 -> 1 with ReLU (the paper names machine-learning assisted scheduling as future work, Sec. VII),
// trained on op times the runtime records.
//
// Training step on a batch of B samples (row indices into the uploaded sample set):
//   mlp_pass    z1 = W1 xn + b1, h1 = relu(z1), z2 = W2 h1 + b2, h2 = relu(z2), y = W3 h2 + b3,
//               with xn the z-scored features, then dy = 2 (y - t) / B, dz2 = dy W3 * [z2 > 0],
//               dz1 = (W2^T dz2) * [z1 > 0]; h1, h2, y and the deltas are kept per sample.
//   mlp_update  sums every parameter's gradient over the batch in sample order (deterministic),
//               then applies Adam with bias-corrected moments.
// The network is ~9.9 kFLOP per sample forward and every step depends on the one before, so both
// kernels are bound by latency (plain FP32 vector FMAs, not matrix cores): each sum is one chain
// of dependent FMAs in a fixed order, and what can be shortened is the memory latency around it.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <numeric>
#include <random>
#include <string>

#include "mlp.hpp"

namespace psc {

#define MLP_HIP(call)                                                                          \
  do {                                                                                         \
    hipError_t e_ = (call);                                                                    \
    if (e_ != hipSuccess) fail(PSC_ERR_HIP, std::string(#call) + ": " + hipGetErrorString(e_)); \
  } while (0)

namespace {

constexpr int kSPW = 2;          // samples a wavefront of mlp_pass carries at a time
constexpr int kPassBlocks = 512;  // blocks of a full grid (two per CU); larger sets loop
constexpr int kChunk = 256;      // samples of a gradient chunk staged in LDS by mlp_update
constexpr int kAhead = 32;       // samples of a gradient chain read from LDS ahead of their sums

// Forward and (BACK) back-propagation of kSPW samples per wavefront.  Lane j owns hidden unit j of
// both layers: it holds row j of W1 and of W2 and (BACK) column j of W2 in registers, so a layer is
// one chain of FMAs per lane whose other operand is a broadcast LDS read, and a batch of 256 runs
// on 32 blocks.  Every sum keeps one order: z1 over the features, z2 and dz1 over the units, y as
// four chains of 16 units added pairwise.  The outputs are written for mlp_update: H1, H2 after
// ReLU (both are > 0 exactly where their pre-activations are), the deltas, Y and DY.
// Measured at 256 samples: see mlp_update.
template <bool BACK>
__global__ __launch_bounds__(256) void mlp_pass(const float *__restrict__ P, const float *__restrict__ norm,
                                                const float *__restrict__ X, const float *__restrict__ T,
                                                const int32_t *__restrict__ idx, int32_t n, float scale,
                                                float *__restrict__ H1, float *__restrict__ H2,
                                                float *__restrict__ Y, float *__restrict__ DZ1,
                                                float *__restrict__ DZ2, float *__restrict__ DY) {
  __shared__ __attribute__((aligned(16))) float lds[4][kSPW][kMlpH];  // one region per wavefront
  // W2 goes through LDS: its rows, read by lane straight from memory, would touch 64 cache lines
  // per load.  Pitch 68: 16-byte row reads of 16 lanes and column reads cover distinct banks.
  constexpr int kPitch = kMlpH + 4;
  __shared__ __attribute__((aligned(16))) float w2[kMlpH * kPitch];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  static_assert(kMlpW2 % 4 == 0 && kMlpF % 4 == 0 && kMlpW3 % 4 == 0, "16-byte parameter loads");
  const float4 *P4 = reinterpret_cast<const float4 *>(P);
#pragma unroll
  for (int j = 0; j < kMlpH * kMlpH / 4 / 256; ++j) {
    const int u = threadIdx.x + 256 * j;
    *reinterpret_cast<float4 *>(&w2[u / (kMlpH / 4) * kPitch + u % (kMlpH / 4) * 4]) = P4[kMlpW2 / 4 + u];
  }
  float w1[kMlpF], row[kMlpH], col[BACK ? kMlpH : 1];
#pragma unroll
  for (int f = 0; f < kMlpF; f += 4) {
    const float4 v = P4[(kMlpW1 + lane * kMlpF + f) / 4];
    w1[f] = v.x, w1[f + 1] = v.y, w1[f + 2] = v.z, w1[f + 3] = v.w;
  }
  const float b1 = P[kMlpB1 + lane], b2 = P[kMlpB2 + lane], w3 = P[kMlpW3 + lane], b3 = P[kMlpB3];
  // the output layer's chains: lane 4 q + c sums units [16 c, 16 c + 16) of sample q
  const int q = (lane >> 2) % kSPW, c = lane & 3;
  float w3c[kMlpH / 4];
#pragma unroll
  for (int u = 0; u < kMlpH / 4; u += 4) {
    const float4 v = P4[(kMlpW3 + c * (kMlpH / 4) + u) / 4];
    w3c[u] = v.x, w3c[u + 1] = v.y, w3c[u + 2] = v.z, w3c[u + 3] = v.w;
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < kMlpH; i += 4) {
    const float4 v = *reinterpret_cast<const float4 *>(&w2[lane * kPitch + i]);
    row[i] = v.x, row[i + 1] = v.y, row[i + 2] = v.z, row[i + 3] = v.w;
  }
  if constexpr (BACK) {
#pragma unroll
    for (int i = 0; i < kMlpH; ++i) col[i] = w2[i * kPitch + lane];
  }
  float(*buf)[kMlpH] = lds[wv];
  // a wavefront reads only what it wrote itself, and its LDS operations take effect in program
  // order; the fences keep the compiler to that order
  auto order = [] {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  };
  const int64_t step = int64_t(gridDim.x) * 4 * kSPW;
  for (int64_t s0 = (int64_t(blockIdx.x) * 4 + wv) * kSPW; s0 < n; s0 += step) {
    int64_t s[kSPW], r[kSPW];
    float z1[kSPW], z2[kSPW];
#pragma unroll
    for (int k = 0; k < kSPW; ++k) {
      s[k] = s0 + k < n ? s0 + k : s0;  // a missing sample repeats the first and is not stored
      r[k] = idx ? idx[s[k]] : s[k];
      float z = b1;
#pragma unroll
      for (int f = 0; f < kMlpF; ++f) z = fmaf(w1[f], (X[r[k] * kMlpF + f] - norm[f]) * norm[kMlpF + f], z);
      z1[k] = fmaxf(z, 0.0f);
      buf[k][lane] = z1[k];
      z2[k] = b2;
    }
    order();
#pragma unroll
    for (int i = 0; i < kMlpH; i += 4)
#pragma unroll
      for (int k = 0; k < kSPW; ++k) {
        const float4 h = *reinterpret_cast<const float4 *>(&buf[k][i]);
        z2[k] = fmaf(row[i + 3], h.w, fmaf(row[i + 2], h.z, fmaf(row[i + 1], h.y, fmaf(row[i], h.x, z2[k]))));
      }
    order();
#pragma unroll
    for (int k = 0; k < kSPW; ++k) {
      z2[k] = fmaxf(z2[k], 0.0f);
      buf[k][lane] = z2[k];
    }
    order();
    float acc = 0.0f;
#pragma unroll
    for (int u = 0; u < kMlpH / 4; u += 4) {
      const float4 h = *reinterpret_cast<const float4 *>(&buf[q][c * (kMlpH / 4) + u]);
      acc = fmaf(w3c[u + 3], h.w, fmaf(w3c[u + 2], h.z, fmaf(w3c[u + 1], h.y, fmaf(w3c[u], h.x, acc))));
    }
    order();
    float y[kSPW];
#pragma unroll
    for (int k = 0; k < kSPW; ++k) {
      const float r0 = __shfl(acc, 4 * k), r1 = __shfl(acc, 4 * k + 1), r2 = __shfl(acc, 4 * k + 2),
                  r3 = __shfl(acc, 4 * k + 3);
      y[k] = b3 + ((r0 + r1) + (r2 + r3));
    }
    if constexpr (!BACK) {
#pragma unroll
      for (int k = 0; k < kSPW; ++k)
        if (s0 + k < n && lane == k) Y[s0 + k] = y[k];
    } else {
      float dy[kSPW], d1[kSPW];
#pragma unroll
      for (int k = 0; k < kSPW; ++k) {
        dy[k] = scale * (y[k] - T[r[k]]);
        const float d2 = z2[k] > 0.0f ? dy[k] * w3 : 0.0f;
        buf[k][lane] = d2;
        d1[k] = 0.0f;
        if (s0 + k < n) {
          H1[s[k] * kMlpH + lane] = z1[k];
          H2[s[k] * kMlpH + lane] = z2[k];
          DZ2[s[k] * kMlpH + lane] = d2;
          if (lane == k) {
            Y[s0 + k] = y[k];
            DY[s0 + k] = dy[k];
          }
        }
      }
      order();
#pragma unroll
      for (int j = 0; j < kMlpH; j += 4)
#pragma unroll
        for (int k = 0; k < kSPW; ++k) {
          const float4 d = *reinterpret_cast<const float4 *>(&buf[k][j]);
          d1[k] = fmaf(col[j + 3], d.w, fmaf(col[j + 2], d.z, fmaf(col[j + 1], d.y, fmaf(col[j], d.x, d1[k]))));
        }
      order();
#pragma unroll
      for (int k = 0; k < kSPW; ++k)
        if (s0 + k < n) DZ1[s[k] * kMlpH + lane] = z1[k] > 0.0f ? d1[k] : 0.0f;
    }
  }
}

struct UpdateArgs {
  float *P, *M, *V, *G;  // G may be null
  const float *norm, *X;
  const int32_t *idx;
  const float *H1, *H2, *DZ1, *DZ2, *DY;
  int32_t n;
  int32_t update;        // apply Adam
  float lr, beta1, beta2, eps, c1, c2;  // c1 = 1 / (1 - beta1^t), c2 = 1 / (1 - beta2^t)
};

// Blocks of mlp_update: W2 by rows of four, W1 by 256 parameters, b1, b2, W3 with b3.
constexpr int kUpdW1 = kMlpH / 4, kUpdB1 = kUpdW1 + kMlpH * kMlpF / 256, kUpdB2 = kUpdB1 + 1, kUpdW3 = kUpdB2 + 1,
              kUpdBlocks = kUpdW3 + 1;

// One thread per parameter; the batch sum runs in sample order.  A block's operands (256 samples
// of one 64-wide array and of the array or arrays it is multiplied with) are staged in LDS first,
// all their loads in flight together, so the chain of dependent FMAs reads LDS instead of paying a
// cache latency per few samples.  Measured at batches of 256, with mlp_pass: a training step takes
// 14.8 us (5.8 pass, 6.9 update, the launches between); it took 98 us as three kernels that read
// global memory inside the chains (15.6 forward on four blocks, 18.6 back-propagation, 61.3
// update), and 22.7 us with the chunk's loads guarded one by one.
__global__ __launch_bounds__(256) void mlp_update(UpdateArgs a) {
  __shared__ __attribute__((aligned(16))) float big[kChunk * kMlpH];  // one 64-wide array
  __shared__ __attribute__((aligned(16))) float small[kChunk * kMlpF];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, blk = blockIdx.x;
  const float *wide = blk < kUpdW1 ? a.H1 : blk <= kUpdB1 ? a.DZ1 : blk == kUpdB2 ? a.DZ2 : a.H2;
  int p = -1;                          // this thread's parameter
  if (blk < kUpdW1) p = kMlpW2 + (blk * 4 + wv) * kMlpH + lane;
  else if (blk < kUpdB1) p = kMlpW1 + (blk - kUpdW1) * 256 + tid;
  else if (blk == kUpdB1) p = wv == 0 ? kMlpB1 + lane : -1;
  else if (blk == kUpdB2) p = wv == 0 ? kMlpB2 + lane : -1;
  else p = wv == 0 ? kMlpW3 + lane : tid == 64 ? kMlpB3 : -1;
  const int i1 = (p - kMlpW1) / kMlpF, f1 = (p - kMlpW1) % kMlpF;  // W1: unit and feature
  float g = 0.0f;
  for (int32_t s0 = 0; s0 < a.n; s0 += kChunk) {
    const int m = min(kChunk, a.n - s0);
    if (s0) __syncthreads();
    // every load of the chunk is issued before the first LDS write; past the chunk's end they
    // repeat its last element (a guarded load would wait for its own result inside its branch)
    const float4 *src = reinterpret_cast<const float4 *>(wide + int64_t(s0) * kMlpH);
    float4 w[kChunk * kMlpH / 4 / 256];
#pragma unroll
    for (int j = 0; j < kChunk * kMlpH / 4 / 256; ++j) w[j] = src[min(tid + 256 * j, m * (kMlpH / 4) - 1)];
    const int sm = min(tid, m - 1);
    if (blk < kUpdW1) {          // four columns of DZ2, each contiguous over the samples
      const float4 d = *reinterpret_cast<const float4 *>(a.DZ2 + int64_t(s0 + sm) * kMlpH + blk * 4);
      small[tid] = d.x;
      small[kChunk + tid] = d.y;
      small[2 * kChunk + tid] = d.z;
      small[3 * kChunk + tid] = d.w;
    } else if (blk < kUpdB1) {   // the z-scored features, a sample per thread
      const int64_t r = a.idx ? a.idx[s0 + sm] : s0 + sm;
#pragma unroll
      for (int f = 0; f < kMlpF; ++f) small[tid * kMlpF + f] = (a.X[r * kMlpF + f] - a.norm[f]) * a.norm[kMlpF + f];
    } else if (blk == kUpdW3) {
      small[tid] = a.DY[s0 + sm];
    }
#pragma unroll
    for (int j = 0; j < kChunk * kMlpH / 4 / 256; ++j) reinterpret_cast<float4 *>(big)[tid + 256 * j] = w[j];
    __syncthreads();
    if (p < 0) continue;
    // `u` and `v` of sample s, u = 1 for a plain sum
    auto chain = [&](auto u, auto v, auto &&sum) {
      int s = 0;
      for (; s + kAhead <= m; s += kAhead) {
        float x[kAhead], y[kAhead];
#pragma unroll
        for (int e = 0; e < kAhead; ++e) x[e] = u(s + e), y[e] = v(s + e);
#pragma unroll
        for (int e = 0; e < kAhead; ++e) g = sum(x[e], y[e], g);
      }
      for (; s < m; ++s) g = sum(u(s), v(s), g);
    };
    auto fma_ = [](float x, float y, float z) { return fmaf(x, y, z); };
    auto add_ = [](float, float y, float z) { return z + y; };
    auto one = [](int) { return 1.0f; };
    auto wide_lane = [&](int s) { return big[s * kMlpH + lane]; };
    if (blk < kUpdW1) chain([&](int s) { return small[wv * kChunk + s]; }, wide_lane, fma_);
    else if (blk < kUpdB1)
      chain([&](int s) { return big[s * kMlpH + i1]; }, [&](int s) { return small[s * kMlpF + f1]; }, fma_);
    else if (blk < kUpdW3) chain(one, wide_lane, add_);
    else if (wv == 0) chain([&](int s) { return small[s]; }, wide_lane, fma_);
    else chain(one, [&](int s) { return small[s]; }, add_);
  }
  if (p < 0) return;
  if (a.G) a.G[p] = g;
  if (a.update) {
    const float m = a.beta1 * a.M[p] + (1.0f - a.beta1) * g;
    const float v = a.beta2 * a.V[p] + (1.0f - a.beta2) * g * g;
    a.M[p] = m;
    a.V[p] = v;
    a.P[p] -= a.lr * (m * a.c1) / (sqrtf(v * a.c2) + a.eps);
  }
}

void ensure_cap(psc_mlp &m, int64_t n) {
  if (n <= m.cap) return;
  const int64_t c = std::max<int64_t>(n, 2 * m.cap);
  float **fl[] = {&m.x, &m.t, &m.h1, &m.h2, &m.y, &m.dz1, &m.dz2, &m.dy};
  for (float **p : fl)
    if (*p) { MLP_HIP(hipFree(*p)); *p = nullptr; }
  if (m.idx) { MLP_HIP(hipFree(m.idx)); m.idx = nullptr; }
  m.cap = 0;
  MLP_HIP(hipMalloc(&m.x, size_t(c) * kMlpF * 4));
  MLP_HIP(hipMalloc(&m.t, size_t(c) * 4));
  MLP_HIP(hipMalloc(&m.h1, size_t(c) * kMlpH * 4));
  MLP_HIP(hipMalloc(&m.h2, size_t(c) * kMlpH * 4));
  MLP_HIP(hipMalloc(&m.y, size_t(c) * 4));
  MLP_HIP(hipMalloc(&m.dz1, size_t(c) * kMlpH * 4));
  MLP_HIP(hipMalloc(&m.dz2, size_t(c) * kMlpH * 4));
  MLP_HIP(hipMalloc(&m.dy, size_t(c) * 4));
  MLP_HIP(hipMalloc(&m.idx, size_t(c) * 4));
  m.cap = c;
}

unsigned blocks_for(int64_t n) {
  return unsigned(std::min<int64_t>(kPassBlocks, (n + 4 * kSPW - 1) / (4 * kSPW)));
}

void check_n(int64_t n) {
  if (n < 1 || n > (int64_t(1) << 30)) fail(PSC_ERR_ARG, "sample count must be in [1, 2^30]");
}

// Device memory of one forward / backward pass: the samples (x, t), the per-sample activations
// (h1, h2, y) and the back-propagated errors (dz1, dz2, dy).  The model's own buffers (grown on
// demand) or the fixed scratch array of the allocation-free entry point.
struct Work {
  const float *x, *t;
  float *h1, *h2, *y, *dz1, *dz2, *dy;
};

Work work_of(psc_mlp &m) { return Work{m.x, m.t, m.h1, m.h2, m.y, m.dz1, m.dz2, m.dy}; }

void launch_pass(psc_mlp &m, const Work &w, const int32_t *idx, int64_t n, bool back) {
  const float *P = m.params, *norm = m.norm, *X = w.x, *T = w.t;
  int32_t nn = int32_t(n);
  float scale = float(2.0 / double(n));
  float *H1 = w.h1, *H2 = w.h2, *Y = w.y, *DZ1 = w.dz1, *DZ2 = w.dz2, *DY = w.dy;
  void *args[] = {&P, &norm, &X, &T, &idx, &nn, &scale, &H1, &H2, &Y, &DZ1, &DZ2, &DY};
  const void *fn = back ? reinterpret_cast<const void *>(&mlp_pass<true>) : reinterpret_cast<const void *>(&mlp_pass<false>);
  MLP_HIP(hipLaunchKernel(fn, dim3(blocks_for(n)), dim3(256), args, 0, m.stream));
}

// predictions of the first n uploaded samples
void launch_fwd(psc_mlp &m, int64_t n) { launch_pass(m, work_of(m), nullptr, n, false); }

void launch_step(psc_mlp &m, const Work &w, const int32_t *idx, int64_t n, bool update, const MlpTrainOpts &o,
                 float *G) {
  launch_pass(m, w, idx, n, true);
  UpdateArgs a{};
  a.P = m.params;
  a.M = m.m;
  a.V = m.v;
  a.G = G;
  a.norm = m.norm;
  a.X = w.x;
  a.idx = idx;
  a.H1 = w.h1;
  a.H2 = w.h2;
  a.DZ1 = w.dz1;
  a.DZ2 = w.dz2;
  a.DY = w.dy;
  a.n = int32_t(n);
  a.update = update ? 1 : 0;
  if (update) {
    ++m.step;
    a.lr = o.lr;
    a.beta1 = o.beta1;
    a.beta2 = o.beta2;
    a.eps = o.eps;
    a.c1 = float(1.0 / (1.0 - std::pow(double(o.beta1), double(m.step))));
    a.c2 = float(1.0 / (1.0 - std::pow(double(o.beta2), double(m.step))));
  }
  void *uargs[] = {&a};
  MLP_HIP(hipLaunchKernel(reinterpret_cast<const void *>(&mlp_update), dim3(kUpdBlocks), dim3(256), uargs, 0,
                          m.stream));
}

void launch_step(psc_mlp &m, const int32_t *idx, int64_t n, bool update, const MlpTrainOpts &o, float *G) {
  launch_step(m, work_of(m), idx, n, update, o, G);
}

double mse_of(const std::vector<float> &y, const float *t, int64_t n) {
  double acc = 0;
  for (int64_t i = 0; i < n; ++i) {
    const double d = double(y[i]) - double(t[i]);
    acc += d * d;
  }
  return acc / double(n);
}

void upload_x(psc_mlp &m, const float *x, int64_t n) {
  MLP_HIP(hipMemcpyAsync(m.x, x, size_t(n) * kMlpF * 4, hipMemcpyHostToDevice, m.stream));
}

}  // namespace

psc_mlp *mlp_create(int device) {
  int nd = 0;
  MLP_HIP(hipGetDeviceCount(&nd));
  if (device < 0 || device >= nd) fail(PSC_ERR_ARG, "device ordinal out of range");
  MLP_HIP(hipSetDevice(device));
  auto m = std::make_unique<psc_mlp>();
  m->device = device;
  MLP_HIP(hipStreamCreateWithFlags(&m->stream, hipStreamNonBlocking));
  MLP_HIP(hipMalloc(&m->params, kMlpP * 4));
  MLP_HIP(hipMalloc(&m->m, kMlpP * 4));
  MLP_HIP(hipMalloc(&m->v, kMlpP * 4));
  MLP_HIP(hipMalloc(&m->g, kMlpP * 4));
  MLP_HIP(hipMalloc(&m->norm, 2 * kMlpF * 4));
  std::vector<float> z(kMlpP, 0.0f);
  MLP_HIP(hipMemcpy(m->params, z.data(), kMlpP * 4, hipMemcpyHostToDevice));
  MLP_HIP(hipMemcpy(m->m, z.data(), kMlpP * 4, hipMemcpyHostToDevice));
  MLP_HIP(hipMemcpy(m->v, z.data(), kMlpP * 4, hipMemcpyHostToDevice));
  const float mean[kMlpF] = {}, sd[kMlpF] = {1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1};
  mlp_set_norm(*m, mean, sd);
  return m.release();
}

void mlp_set_params(psc_mlp &m, const float *p) {
  std::lock_guard<std::mutex> lk(m.mu);
  MLP_HIP(hipSetDevice(m.device));
  std::vector<float> z(kMlpP, 0.0f);
  MLP_HIP(hipMemcpy(m.params, p, kMlpP * 4, hipMemcpyHostToDevice));
  MLP_HIP(hipMemcpy(m.m, z.data(), kMlpP * 4, hipMemcpyHostToDevice));
  MLP_HIP(hipMemcpy(m.v, z.data(), kMlpP * 4, hipMemcpyHostToDevice));
  m.step = 0;
}

void mlp_get_params(psc_mlp &m, float *p) {
  std::lock_guard<std::mutex> lk(m.mu);
  MLP_HIP(hipSetDevice(m.device));
  MLP_HIP(hipStreamSynchronize(m.stream));
  MLP_HIP(hipMemcpy(p, m.params, kMlpP * 4, hipMemcpyDeviceToHost));
}

void mlp_set_norm(psc_mlp &m, const float *mean, const float *std_) {
  float h[2 * kMlpF];
  for (int f = 0; f < kMlpF; ++f) {
    if (!(std_[f] > 0.0f) || !std::isfinite(std_[f]) || !std::isfinite(mean[f]))
      fail(PSC_ERR_ARG, "feature scales must be finite and positive");
    h[f] = mean[f];
    h[kMlpF + f] = 1.0f / std_[f];
    m.h_mean[f] = mean[f];
    m.h_std[f] = std_[f];
  }
  MLP_HIP(hipSetDevice(m.device));
  MLP_HIP(hipMemcpy(m.norm, h, sizeof(h), hipMemcpyHostToDevice));
}

void mlp_predict(psc_mlp &m, const float *x, int64_t n, float *y) {
  check_n(n);
  std::lock_guard<std::mutex> lk(m.mu);
  MLP_HIP(hipSetDevice(m.device));
  ensure_cap(m, n);
  upload_x(m, x, n);
  launch_fwd(m, n);
  MLP_HIP(hipMemcpyAsync(y, m.y, size_t(n) * 4, hipMemcpyDeviceToHost, m.stream));
  MLP_HIP(hipStreamSynchronize(m.stream));
}

double mlp_grad(psc_mlp &m, const float *x, const float *t, int64_t n, float *grads) {
  check_n(n);
  std::lock_guard<std::mutex> lk(m.mu);
  MLP_HIP(hipSetDevice(m.device));
  ensure_cap(m, n);
  upload_x(m, x, n);
  MLP_HIP(hipMemcpyAsync(m.t, t, size_t(n) * 4, hipMemcpyHostToDevice, m.stream));
  launch_step(m, nullptr, n, false, MlpTrainOpts{}, m.g);
  std::vector<float> y(n);
  MLP_HIP(hipMemcpyAsync(y.data(), m.y, size_t(n) * 4, hipMemcpyDeviceToHost, m.stream));
  if (grads) MLP_HIP(hipMemcpyAsync(grads, m.g, kMlpP * 4, hipMemcpyDeviceToHost, m.stream));
  MLP_HIP(hipStreamSynchronize(m.stream));
  return mse_of(y, t, n);
}

// ---------------------------------------------------------------------------------------------
// Allocation-free gradient (psc_mlp_grad_static): the same kernels as mlp_grad, with every
// buffer of the pass in one fixed device array instead of memory the model allocates.
// ---------------------------------------------------------------------------------------------

namespace {

// Layout of the scratch array, in floats: x (max x F), t, h1, h2, y, dz1, dz2, dy, the gradient
// (kMlpP, padded) and the loss (one double).
constexpr int64_t kSMax = kMlpStaticMax;
constexpr int64_t kOffX = 0;
constexpr int64_t kOffT = kOffX + kSMax * kMlpF;
constexpr int64_t kOffH1 = kOffT + kSMax;
constexpr int64_t kOffH2 = kOffH1 + kSMax * kMlpH;
constexpr int64_t kOffY = kOffH2 + kSMax * kMlpH;
constexpr int64_t kOffDZ1 = kOffY + kSMax;
constexpr int64_t kOffDZ2 = kOffDZ1 + kSMax * kMlpH;
constexpr int64_t kOffDY = kOffDZ2 + kSMax * kMlpH;
constexpr int64_t kOffG = kOffDY + kSMax;
constexpr int64_t kOffLoss = kOffG + ((kMlpP + 63) / 64) * 64;
constexpr int64_t kScratchFloats = kOffLoss + 64;

// One copy per GPU, held until the process ends.  Host code never passes this name to a kernel or
// a copy: it is the host-side stand-in, and the device address comes from hipGetSymbolAddress.
static __device__ __align__(256) float scratch[kScratchFloats];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu[kMaxDevices];   // one call at a time per GPU: every call shares its array
float *g_scratch_ptr[kMaxDevices] = {};

float *scratch_of(int device) {
  if (g_scratch_ptr[device]) return g_scratch_ptr[device];
  void *p = nullptr;
  const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
  if (e != hipSuccess || p == nullptr)
    fail(PSC_ERR_HIP, std::string("hipGetSymbolAddress(scratch): ") + hipGetErrorString(e));
  g_scratch_ptr[device] = static_cast<float *>(p);
  return g_scratch_ptr[device];
}

// Mean squared error of y against t over n samples in float64: 256 threads, thread i sums samples
// i, i + 256, ... in order, then a fixed-order tree over the threads.
__global__ __launch_bounds__(256) void mlp_mse(const float *__restrict__ Y, const float *__restrict__ T, int32_t n,
                                               double *__restrict__ out) {
  __shared__ double part[256];
  double acc = 0.0;
  for (int32_t s = threadIdx.x; s < n; s += 256) {
    const double d = double(Y[s]) - double(T[s]);
    acc = fma(d, d, acc);
  }
  part[threadIdx.x] = acc;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if (int(threadIdx.x) < w) part[threadIdx.x] += part[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) out[0] = part[0] / double(n);
}

}  // namespace

double mlp_grad_static(psc_mlp &m, const float *x, const float *t, int64_t n, float *grads) {
  if (n < 1 || n > kMlpStaticMax)
    fail(PSC_ERR_ARG, "sample count must be in [1, " + std::to_string(kMlpStaticMax) + "] (the fixed scratch size)");
  if (m.device < 0 || m.device >= kMaxDevices) fail(PSC_ERR_ARG, "device ordinal out of range");
  std::lock_guard<std::mutex> lk(m.mu);
  std::lock_guard<std::mutex> sk(g_scratch_mu[m.device]);
  MLP_HIP(hipSetDevice(m.device));
  float *base = scratch_of(m.device);
  float *xs = base + kOffX, *ts = base + kOffT;
  const Work w{xs, ts, base + kOffH1, base + kOffH2, base + kOffY, base + kOffDZ1, base + kOffDZ2, base + kOffDY};
  float *G = base + kOffG;
  double *L = reinterpret_cast<double *>(base + kOffLoss);
  MLP_HIP(hipMemcpyAsync(xs, x, size_t(n) * kMlpF * 4, hipMemcpyHostToDevice, m.stream));
  MLP_HIP(hipMemcpyAsync(ts, t, size_t(n) * 4, hipMemcpyHostToDevice, m.stream));
  // every element the kernels read is written first in this call (x, t above; h, y, deltas by
  // the pass; G and the loss entirely), so nothing left by an earlier call is seen
  launch_step(m, w, nullptr, n, false, MlpTrainOpts{}, G);
  {
    const float *Y = w.y, *T = ts;
    int32_t nn = int32_t(n);
    void *args[] = {&Y, &T, &nn, &L};
    MLP_HIP(hipLaunchKernel(reinterpret_cast<const void *>(&mlp_mse), dim3(1), dim3(256), args, 0, m.stream));
  }
  double loss = 0.0;
  MLP_HIP(hipMemcpyAsync(&loss, L, sizeof(double), hipMemcpyDeviceToHost, m.stream));
  if (grads) MLP_HIP(hipMemcpyAsync(grads, G, kMlpP * 4, hipMemcpyDeviceToHost, m.stream));
  MLP_HIP(hipStreamSynchronize(m.stream));
  return loss;
}

void mlp_train(psc_mlp &m, const float *x, const float *t, int64_t n, const MlpTrainOpts &o, float *epoch_loss) {
  check_n(n);
  if (o.epochs < 1 || o.batch < 1) fail(PSC_ERR_ARG, "epochs and batch must be >= 1");
  if (!(o.lr > 0.0f) || !(o.beta1 >= 0.0f && o.beta1 < 1.0f) || !(o.beta2 >= 0.0f && o.beta2 < 1.0f) ||
      !(o.eps > 0.0f))
    fail(PSC_ERR_ARG, "Adam hyper-parameters out of range");
  std::lock_guard<std::mutex> lk(m.mu);
  MLP_HIP(hipSetDevice(m.device));
  ensure_cap(m, n);
  upload_x(m, x, n);
  MLP_HIP(hipMemcpyAsync(m.t, t, size_t(n) * 4, hipMemcpyHostToDevice, m.stream));
  std::vector<int32_t> order(n);
  std::iota(order.begin(), order.end(), 0);
  std::mt19937_64 gen(o.shuffle_seed);
  std::vector<float> y(n);
  for (int32_t e = 0; e < o.epochs; ++e) {
    if (o.shuffle_seed) std::shuffle(order.begin(), order.end(), gen);
    // the previous epoch's steps must be done with idx before it is overwritten
    MLP_HIP(hipStreamSynchronize(m.stream));
    MLP_HIP(hipMemcpyAsync(m.idx, order.data(), size_t(n) * 4, hipMemcpyHostToDevice, m.stream));
    for (int64_t b0 = 0; b0 < n; b0 += o.batch)
      launch_step(m, m.idx + b0, std::min<int64_t>(o.batch, n - b0), true, o, nullptr);
    if (epoch_loss) {
      launch_fwd(m, n);
      MLP_HIP(hipMemcpyAsync(y.data(), m.y, size_t(n) * 4, hipMemcpyDeviceToHost, m.stream));
      MLP_HIP(hipStreamSynchronize(m.stream));
      epoch_loss[e] = float(mse_of(y, t, n));
    }
  }
  MLP_HIP(hipStreamSynchronize(m.stream));
}

void mlp_get_state(psc_mlp &m, MlpState &st) {
  std::lock_guard<std::mutex> lk(m.mu);
  MLP_HIP(hipSetDevice(m.device));
  MLP_HIP(hipStreamSynchronize(m.stream));
  st.params.resize(kMlpP);
  st.m.resize(kMlpP);
  st.v.resize(kMlpP);
  MLP_HIP(hipMemcpy(st.params.data(), m.params, kMlpP * 4, hipMemcpyDeviceToHost));
  MLP_HIP(hipMemcpy(st.m.data(), m.m, kMlpP * 4, hipMemcpyDeviceToHost));
  MLP_HIP(hipMemcpy(st.v.data(), m.v, kMlpP * 4, hipMemcpyDeviceToHost));
  std::copy(m.h_mean, m.h_mean + kMlpF, st.mean);
  std::copy(m.h_std, m.h_std + kMlpF, st.std_);
  st.step = m.step;
}

void mlp_put_state(psc_mlp &m, const MlpState &st) {
  mlp_set_norm(m, st.mean, st.std_);
  std::lock_guard<std::mutex> lk(m.mu);
  MLP_HIP(hipSetDevice(m.device));
  MLP_HIP(hipStreamSynchronize(m.stream));
  MLP_HIP(hipMemcpy(m.params, st.params.data(), kMlpP * 4, hipMemcpyHostToDevice));
  MLP_HIP(hipMemcpy(m.m, st.m.data(), kMlpP * 4, hipMemcpyHostToDevice));
  MLP_HIP(hipMemcpy(m.v, st.v.data(), kMlpP * 4, hipMemcpyHostToDevice));
  m.step = st.step;
}

namespace {

struct MlpCost final : CostModel {
  psc_mlp &m;
  explicit MlpCost(psc_mlp &m_) : m(m_) {}
  void predict_us(const float *feat, int64_t n, double *us) override {
    if (n <= 0) return;
    std::vector<float> y(n);
    mlp_predict(m, feat, n, y.data());
    for (int64_t i = 0; i < n; ++i) us[i] = std::exp(double(y[i]));
  }
};

}  // namespace

std::unique_ptr<CostModel> mlp_cost_model(const psc_mlp *m) {
  return std::make_unique<MlpCost>(*const_cast<psc_mlp *>(m));
}

}  // namespace psc

psc_mlp::~psc_mlp() {
  if (hipSetDevice(device) != hipSuccess) return;
  if (stream) (void)hipStreamSynchronize(stream);
  float *fl[] = {params, m, v, g, norm, x, t, h1, h2, y, dz1, dz2, dy};
  for (float *p : fl)
    if (p) (void)hipFree(p);
  if (idx) (void)hipFree(idx);
  if (stream) (void)hipStreamDestroy(stream);
}
