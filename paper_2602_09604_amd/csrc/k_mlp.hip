// Fusion cost model: a 3-layer MLP (F -> W -> W -> 1, ReLU) trained on the
// GPU with mean squared error and Adam, all in hand-written kernels.
//
// Parameter layout (row-major): W1 [W x F], b1 [W], W2 [W x W], b2 [W],
// W3 [1 x W], b3 [1].
//
// k_mlp_grad: one workgroup per chunk of 64 samples keeps the inputs and both
// hidden activations in LDS, runs the forward pass, the loss and the whole
// backward pass, and writes its chunk's gradient (sum over its samples of
// dL/dparam) to a partial buffer.  k_mlp_reduce sums the partials in a fixed
// order (deterministic) and, in training, applies the Adam update; k_mlp_adam
// applies it to a gradient that is there.
#include <cmath>
#include <cstring>
#include <random>
#include <vector>

#include "sv_internal.h"

struct sv_mlp {
  int width = 64;
  int nparams = 0;
  hipStream_t stream = nullptr;
  float* params = nullptr;  // device
  float* grad = nullptr;    // device, last loss_grad
  float* m = nullptr;       // Adam moments
  float* v = nullptr;
  float* partial = nullptr;  // [max_blocks][nparams + 1]
  int max_blocks = 0;
  float* loss_dev = nullptr;
  float* host_pinned = nullptr;  // nparams + 1
  int step = 0;
};

namespace sv {

namespace {

constexpr int F = SV_COST_FEATURES;
constexpr int CH = 64;  // samples per workgroup

int num_params(int w) { return w * F + w + w * w + w + w + 1; }

// Two workgroups of 16 waves per chunk: both run the forward pass, the first
// takes the gradients of layers 2 and 3 and the loss, the second those of
// layer 1.  7200 samples are 113 chunks for 256 CUs, so the time is that of
// one chunk's vector FMAs and the latency of its phases.  The weights sit in LDS beside the
// activations; rows are padded to 44 and 68 floats (16-byte reads of 64 rows
// fall on distinct banks), and a thread computes four outputs of a phase and
// reads what they share once.  Every output is the same chain of FMAs in the
// same order whatever the split, so the gradients do not depend on it.  7200
// samples: 40 us with one workgroup of 4 waves and the weights read from
// memory, 22.5 with one of 16, 18.8 so.
template <int W>
__global__ __launch_bounds__(1024) void k_mlp_grad(const float* __restrict__ P, const float* __restrict__ X,
                                                   const float* __restrict__ T, int B, float* __restrict__ partial,
                                                   int stride) {
  static_assert(W == 64 && F == 40 && CH == 64, "the thread maps below are for this network");
  constexpr int S1 = 44, S2 = 68;
  __shared__ __align__(16) float xs[CH][F];
  __shared__ __align__(16) float h1[CH][S2];
  __shared__ __align__(16) float w2[W][S2];
  __shared__ __align__(16) float h2[CH][S2];  // first W1, rows of S1
  __shared__ float dy[CH], err[CH];
  float(*w1)[S1] = reinterpret_cast<float(*)[S1]>(&h2[0][0]);
  const float* W1 = P;
  const float* b1 = W1 + W * F;
  const float* W2 = b1 + W;
  const float* b2 = W2 + W * W;
  const float* W3 = b2 + W;
  const float* b3 = W3 + W;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int s0 = blockIdx.x * CH;
  const int ns = min(CH, B - s0);
  float* out = partial + (size_t)blockIdx.x * stride;
  for (int i = tid; i < CH * F; i += 1024) xs[i / F][i % F] = i / F < ns ? X[(size_t)s0 * F + i] : 0.f;
  for (int i = tid; i < W * F; i += 1024) w1[i / F][i % F] = W1[i];
  for (int i = tid; i < W * W; i += 1024) w2[i / W][i % W] = W2[i];
  __syncthreads();
  // forward: a thread owns unit `lane` of samples wave + 16 t
  float a[4];
#pragma unroll
  for (int t = 0; t < 4; ++t) a[t] = b1[lane];
#pragma unroll
  for (int f = 0; f < F; f += 4) {
    const float4 w = *reinterpret_cast<const float4*>(&w1[lane][f]);
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const float4 x = *reinterpret_cast<const float4*>(&xs[wave + 16 * t][f]);
      a[t] = fmaf(w.w, x.w, fmaf(w.z, x.z, fmaf(w.y, x.y, fmaf(w.x, x.x, a[t]))));
    }
  }
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    h1[wave + 16 * t][lane] = a[t] > 0.f ? a[t] : 0.f;
    a[t] = b2[lane];
  }
  __syncthreads();  // also: w1 is done with, h2 may take its place
#pragma unroll 4
  for (int q = 0; q < W; q += 4) {
    const float4 w = *reinterpret_cast<const float4*>(&w2[lane][q]);
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const float4 x = *reinterpret_cast<const float4*>(&h1[wave + 16 * t][q]);
      a[t] = fmaf(w.w, x.w, fmaf(w.z, x.z, fmaf(w.y, x.y, fmaf(w.x, x.x, a[t]))));
    }
  }
#pragma unroll
  for (int t = 0; t < 4; ++t) h2[wave + 16 * t][lane] = a[t] > 0.f ? a[t] : 0.f;
  __syncthreads();
  // output and dL/dy = 2 (y - t) / B
  if (tid < CH) {
    float d = 0.f;
    if (tid < ns) {
      float y = b3[0];
#pragma unroll 4
      for (int q = 0; q < W; q += 4) {
        const float4 h = *reinterpret_cast<const float4*>(&h2[tid][q]);
        y = fmaf(W3[q + 3], h.w, fmaf(W3[q + 2], h.z, fmaf(W3[q + 1], h.y, fmaf(W3[q], h.x, y))));
      }
      d = y - T[s0 + tid];
    }
    err[tid] = d;
    dy[tid] = d * (2.f / (float)B);
  }
  __syncthreads();
  float* gW1 = out;
  float* gb1 = gW1 + W * F;
  float* gW2 = gb1 + W;
  float* gb2 = gW2 + W * W;
  float* gW3 = gb2 + W;
  float* gb3 = gW3 + W;
  // dh2 = dy * W3 where the unit was active, into registers; beside it, in
  // waves of their own, the layer 3 gradients and the loss
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    const int s = wave + 16 * t;
    a[t] = h2[s][lane] > 0.f ? dy[s] * W3[lane] : 0.f;
  }
  const bool first = blockIdx.y == 0;  // which of the chunk's two workgroups
  if (first && wave == 0) {
    float g = 0.f;
#pragma unroll 16
    for (int s = 0; s < CH; ++s) g = fmaf(dy[s], h2[s][lane], g);
    gW3[lane] = g;
  } else if (first && wave == 1 && lane == 0) {
    float g = 0.f;
#pragma unroll 16
    for (int s = 0; s < CH; ++s) g += dy[s];
    gb3[0] = g;
  } else if (first && wave == 2 && lane == 0) {
    float l = 0.f;
    for (int s = 0; s < ns; ++s) l += err[s] * err[s];
    out[stride - 1] = l;  // sum of squared errors of the chunk
  }
  __syncthreads();
#pragma unroll
  for (int t = 0; t < 4; ++t) h2[wave + 16 * t][lane] = a[t];
  __syncthreads();
  // layer 2 gradients: gW2[i][j] = sum_s dh2[s][i] h1[s][j], 2 x 2 outputs per thread
  if (first) {
    const int r = 2 * (tid >> 5), c = 2 * (tid & 31);
    float g00 = 0.f, g01 = 0.f, g10 = 0.f, g11 = 0.f;
#pragma unroll 8
    for (int s = 0; s < CH; ++s) {
      const float2 u = *reinterpret_cast<const float2*>(&h2[s][r]);
      const float2 v = *reinterpret_cast<const float2*>(&h1[s][c]);
      g00 = fmaf(u.x, v.x, g00);
      g01 = fmaf(u.x, v.y, g01);
      g10 = fmaf(u.y, v.x, g10);
      g11 = fmaf(u.y, v.y, g11);
    }
    gW2[r * W + c] = g00;
    gW2[r * W + c + 1] = g01;
    gW2[(r + 1) * W + c] = g10;
    gW2[(r + 1) * W + c + 1] = g11;
  }
  if (first) {
    if (wave == 3) {
      float g = 0.f;
#pragma unroll 16
      for (int s = 0; s < CH; ++s) g += h2[s][lane];
      gb2[lane] = g;
    }
    return;
  }
  // dh1 = (dh2 W2) where the unit was active; computed into registers first
  // because the mask reads h1 in place
#pragma unroll
  for (int t = 0; t < 4; ++t) a[t] = 0.f;
#pragma unroll 4
  for (int q = 0; q < W; q += 4) {
    const float w[4] = {w2[q][lane], w2[q + 1][lane], w2[q + 2][lane], w2[q + 3][lane]};
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const float4 x = *reinterpret_cast<const float4*>(&h2[wave + 16 * t][q]);
      a[t] = fmaf(x.w, w[3], fmaf(x.z, w[2], fmaf(x.y, w[1], fmaf(x.x, w[0], a[t]))));
    }
  }
#pragma unroll
  for (int t = 0; t < 4; ++t) a[t] = h1[wave + 16 * t][lane] > 0.f ? a[t] : 0.f;
  __syncthreads();
#pragma unroll
  for (int t = 0; t < 4; ++t) h1[wave + 16 * t][lane] = a[t];
  __syncthreads();
  // layer 1 gradients: gW1[i][f] = sum_s dh1[s][i] x[s][f], 2 x 2 outputs per thread
  if (tid < (W / 2) * (F / 2)) {
    const int r = 2 * (tid / (F / 2)), c = 2 * (tid % (F / 2));
    float g00 = 0.f, g01 = 0.f, g10 = 0.f, g11 = 0.f;
#pragma unroll 8
    for (int s = 0; s < CH; ++s) {
      const float2 u = *reinterpret_cast<const float2*>(&h1[s][r]);
      const float2 v = *reinterpret_cast<const float2*>(&xs[s][c]);
      g00 = fmaf(u.x, v.x, g00);
      g01 = fmaf(u.x, v.y, g01);
      g10 = fmaf(u.y, v.x, g10);
      g11 = fmaf(u.y, v.y, g11);
    }
    gW1[r * F + c] = g00;
    gW1[r * F + c + 1] = g01;
    gW1[(r + 1) * F + c] = g10;
    gW1[(r + 1) * F + c + 1] = g11;
  } else if (tid >= 1024 - W) {
    const int r = tid - (1024 - W);
    float g = 0.f;
#pragma unroll 16
    for (int s = 0; s < CH; ++s) g += h1[s][r];
    gb1[r] = g;
  }
}

struct AdamArgs {
  float* p;
  float* m;
  float* v;
  float lr, b1, b2, eps, c1, c2;
};

__device__ __forceinline__ void adam_update(const AdamArgs& a, int i, float gi) {
  const float mi = a.b1 * a.m[i] + (1.f - a.b1) * gi;
  const float vi = a.b2 * a.v[i] + (1.f - a.b2) * gi * gi;
  a.m[i] = mi;
  a.v[i] = vi;
  a.p[i] -= a.lr * (mi / a.c1) / (sqrtf(vi / a.c2) + a.eps);
}

// Sum the per-chunk partials in chunk order: grad[i] = sum_b partial[b][i];
// with ADAM the parameter's update follows at once.  One wave per workgroup
// (108 of them) and 16 loads in flight: 5.0 us at 113 chunks, against 27.5
// (+ 4.8 for the update) with one workgroup per 256 parameters.
template <bool ADAM>
__global__ __launch_bounds__(64) void k_mlp_reduce(const float* __restrict__ partial, int blocks, int stride,
                                                   float* __restrict__ grad, float* __restrict__ loss, int B,
                                                   const AdamArgs adam) {
  const int i = blockIdx.x * 64 + threadIdx.x;
  if (i >= stride) return;
  const float* p = partial + i;
  float a = 0.f;
  int b = 0;
  for (; b + 16 <= blocks; b += 16) {
    float v[16];
#pragma unroll
    for (int u = 0; u < 16; ++u) v[u] = p[(size_t)(b + u) * stride];
#pragma unroll
    for (int u = 0; u < 16; ++u) a += v[u];
  }
  for (; b < blocks; ++b) a += p[(size_t)b * stride];
  if (i == stride - 1) {
    *loss = a / (float)B;
    return;
  }
  grad[i] = a;
  if (ADAM) adam_update(adam, i, a);
}

__global__ __launch_bounds__(256) void k_mlp_adam(const float* __restrict__ g, int n, const AdamArgs a) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i < n) adam_update(a, i, g[i]);
}

template <int W>
__global__ __launch_bounds__(256) void k_mlp_forward(const float* __restrict__ P, const float* __restrict__ X, int B,
                                                     float* __restrict__ Y) {
  __shared__ float h1[4][W];
  __shared__ float h2[4][W];
  const float* W1 = P;
  const float* b1 = W1 + W * F;
  const float* W2 = b1 + W;
  const float* b2 = W2 + W * W;
  const float* W3 = b2 + W;
  const float* b3 = W3 + W;
  const int w = threadIdx.x / 64, j = threadIdx.x % 64;  // one wave per sample
  const int s = blockIdx.x * 4 + w;
  const bool ok = s < B;
  if (j < W) {
    float a = b1[j];
    if (ok)
      for (int f = 0; f < F; ++f) a = fmaf(W1[j * F + f], X[(size_t)s * F + f], a);
    h1[w][j] = a > 0.f ? a : 0.f;
  }
  __syncthreads();
  if (j < W) {
    float a = b2[j];
    for (int q = 0; q < W; ++q) a = fmaf(W2[j * W + q], h1[w][q], a);
    h2[w][j] = a > 0.f ? a : 0.f;
  }
  __syncthreads();
  if (j == 0 && ok) {
    float y = b3[0];
    for (int q = 0; q < W; ++q) y = fmaf(W3[q], h2[w][q], y);
    Y[s] = y;
  }
}

uint64_t splitmix64(uint64_t& x) {
  uint64_t z = (x += 0x9E3779B97F4A7C15ull);
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}

}  // namespace

void cost_model_set(const std::vector<float>& params, int width);

}  // namespace sv

using namespace sv;

#define MLP_GUARD_BEGIN try {
#define MLP_GUARD_END                                                                    \
  }                                                                                      \
  catch (const DeviceError& e) {                                                         \
    return fail(SV_EDEVICE, std::string(e.what) + ": " + hipGetErrorString(e.err));      \
  }                                                                                      \
  catch (const std::bad_alloc&) {                                                        \
    return fail(SV_ENOMEM, "host allocation failed");                                    \
  }                                                                                      \
  catch (...) {                                                                          \
    return fail(SV_EINVAL, "unknown failure");                                           \
  }

extern "C" {

int sv_mlp_create(int width, uint64_t seed, void* hip_stream, sv_mlp** out) {
  if (!out) return fail(SV_EINVAL, "out is NULL");
  *out = nullptr;
  if (width != 64) return fail(SV_EINVAL, "width must be 64 (the kernels are built for it)");
  sv_mlp* m = new sv_mlp();
  MLP_GUARD_BEGIN
  m->width = width;
  m->nparams = num_params(width);
  m->stream = (hipStream_t)hip_stream;
  const size_t pb = sizeof(float) * m->nparams;
  SV_HIP(hipMalloc(&m->params, pb));
  SV_HIP(hipMalloc(&m->grad, pb));
  SV_HIP(hipMalloc(&m->m, pb));
  SV_HIP(hipMalloc(&m->v, pb));
  SV_HIP(hipMalloc(&m->loss_dev, sizeof(float)));
  SV_HIP(hipHostMalloc(&m->host_pinned, pb + sizeof(float), hipHostMallocDefault));
  // He-uniform weights from a SplitMix64 stream, zero biases
  std::vector<float> p(m->nparams, 0.f);
  uint64_t st = seed;
  auto fill = [&](size_t off, int count, int fan_in) {
    const double lim = std::sqrt(6.0 / fan_in);
    for (int i = 0; i < count; ++i) {
      const double u = (double)(splitmix64(st) >> 11) * (1.0 / 9007199254740992.0);
      p[off + i] = (float)((2.0 * u - 1.0) * lim);
    }
  };
  const int W = width;
  fill(0, W * F, F);
  fill((size_t)W * F + W, W * W, W);
  fill((size_t)W * F + W + W * W + W, W, W);
  SV_HIP(hipMemcpy(m->params, p.data(), pb, hipMemcpyHostToDevice));
  std::vector<float> z(m->nparams, 0.f);
  SV_HIP(hipMemcpy(m->m, z.data(), pb, hipMemcpyHostToDevice));
  SV_HIP(hipMemcpy(m->v, z.data(), pb, hipMemcpyHostToDevice));
  SV_HIP(hipMemcpy(m->grad, z.data(), pb, hipMemcpyHostToDevice));
  *out = m;
  return SV_OK;
  }
  catch (const DeviceError& e) {
    sv_mlp_free(m);
    return fail(SV_EDEVICE, std::string(e.what) + ": " + hipGetErrorString(e.err));
  }
  catch (...) {
    sv_mlp_free(m);
    return fail(SV_ENOMEM, "host allocation failed");
  }
}

int sv_mlp_free(sv_mlp* m) {
  if (!m) return SV_OK;
  (void)hipStreamSynchronize(m->stream);
  if (m->params) (void)hipFree(m->params);
  if (m->grad) (void)hipFree(m->grad);
  if (m->m) (void)hipFree(m->m);
  if (m->v) (void)hipFree(m->v);
  if (m->partial) (void)hipFree(m->partial);
  if (m->loss_dev) (void)hipFree(m->loss_dev);
  if (m->host_pinned) (void)hipHostFree(m->host_pinned);
  delete m;
  return SV_OK;
}

int sv_mlp_num_params(const sv_mlp* m, size_t* count) {
  if (!m || !count) return fail(SV_EINVAL, "NULL argument");
  *count = (size_t)m->nparams;
  return SV_OK;
}

int sv_mlp_get_params(sv_mlp* m, float* host_params) {
  if (!m || !host_params) return fail(SV_EINVAL, "NULL argument");
  MLP_GUARD_BEGIN
  SV_HIP(hipMemcpyAsync(m->host_pinned, m->params, sizeof(float) * m->nparams, hipMemcpyDeviceToHost, m->stream));
  SV_HIP(hipStreamSynchronize(m->stream));
  std::memcpy(host_params, m->host_pinned, sizeof(float) * m->nparams);
  return SV_OK;
  MLP_GUARD_END
}

int sv_mlp_set_params(sv_mlp* m, const float* host_params) {
  if (!m || !host_params) return fail(SV_EINVAL, "NULL argument");
  MLP_GUARD_BEGIN
  std::memcpy(m->host_pinned, host_params, sizeof(float) * m->nparams);
  SV_HIP(hipMemcpyAsync(m->params, m->host_pinned, sizeof(float) * m->nparams, hipMemcpyHostToDevice, m->stream));
  SV_HIP(hipStreamSynchronize(m->stream));
  m->step = 0;
  return SV_OK;
  MLP_GUARD_END
}

int sv_mlp_forward(sv_mlp* m, const float* x_dev, int batch, float* y_dev) {
  if (!m || !x_dev || !y_dev || batch < 1) return fail(SV_EINVAL, "bad arguments");
  MLP_GUARD_BEGIN
  hipLaunchKernelGGL(k_mlp_forward<64>, dim3((batch + 3) / 4), dim3(256), 0, m->stream, m->params, x_dev, batch,
                     y_dev);
  SV_HIP(hipGetLastError());
  SV_HIP(hipStreamSynchronize(m->stream));
  return SV_OK;
  MLP_GUARD_END
}

// Room for the partials of a batch of `batch` samples.  Without it the network
// is as it was, and calls with smaller batches go on.
static void mlp_reserve(sv_mlp* m, int batch) {
  const int blocks = (batch + CH - 1) / CH;
  if (blocks <= m->max_blocks) return;
  SV_HIP(hipStreamSynchronize(m->stream));
  float* old = m->partial;
  m->partial = nullptr;
  m->max_blocks = 0;
  if (old) SV_HIP(hipFree(old));
  const hipError_t e = hipMalloc(&m->partial, sizeof(float) * (size_t)(m->nparams + 1) * blocks);
  if (e != hipSuccess) {
    (void)hipGetLastError();  // reported here, not by the next launch
    m->partial = nullptr;
    throw DeviceError{e, "hipMalloc of the gradient partials"};
  }
  m->max_blocks = blocks;
}

// `adam`: also update the parameters with this gradient
static void mlp_loss_grad_async(sv_mlp* m, const float* x_dev, const float* y_dev, int batch,
                                const AdamArgs* adam = nullptr) {
  const int blocks = (batch + CH - 1) / CH;
  const int stride = m->nparams + 1;
  mlp_reserve(m, batch);
  hipLaunchKernelGGL(k_mlp_grad<64>, dim3(blocks, 2), dim3(1024), 0, m->stream, m->params, x_dev, y_dev, batch,
                     m->partial, stride);
  SV_HIP(hipGetLastError());
  auto* reduce = adam ? k_mlp_reduce<true> : k_mlp_reduce<false>;
  hipLaunchKernelGGL(reduce, dim3((stride + 63) / 64), dim3(64), 0, m->stream, m->partial, blocks, stride, m->grad,
                     m->loss_dev, batch, adam ? *adam : AdamArgs{});
  SV_HIP(hipGetLastError());
}

int sv_mlp_loss_grad(sv_mlp* m, const float* x_dev, const float* y_dev, int batch, float* loss_host,
                     float* grad_host) {
  if (!m || !x_dev || !y_dev || batch < 1) return fail(SV_EINVAL, "bad arguments");
  MLP_GUARD_BEGIN
  mlp_loss_grad_async(m, x_dev, y_dev, batch);
  SV_HIP(hipMemcpyAsync(m->host_pinned, m->grad, sizeof(float) * m->nparams, hipMemcpyDeviceToHost, m->stream));
  SV_HIP(hipMemcpyAsync(m->host_pinned + m->nparams, m->loss_dev, sizeof(float), hipMemcpyDeviceToHost, m->stream));
  SV_HIP(hipStreamSynchronize(m->stream));
  if (loss_host) *loss_host = m->host_pinned[m->nparams];
  if (grad_host) std::memcpy(grad_host, m->host_pinned, sizeof(float) * m->nparams);
  return SV_OK;
  MLP_GUARD_END
}

// The next step's update: bias corrections of its number.
static AdamArgs mlp_adam_next(sv_mlp* m, float lr, float b1, float b2, float eps) {
  m->step += 1;
  const float c1 = 1.f - std::pow(b1, (float)m->step);
  const float c2 = 1.f - std::pow(b2, (float)m->step);
  return AdamArgs{m->params, m->m, m->v, lr, b1, b2, eps, c1, c2};
}

int sv_mlp_adam_step(sv_mlp* m, float lr, float beta1, float beta2, float eps) {
  if (!m || !(lr > 0) || !(beta1 >= 0 && beta1 < 1) || !(beta2 >= 0 && beta2 < 1) || !(eps > 0))
    return fail(SV_EINVAL, "bad Adam arguments");
  MLP_GUARD_BEGIN
  hipLaunchKernelGGL(k_mlp_adam, dim3((m->nparams + 255) / 256), dim3(256), 0, m->stream, m->grad, m->nparams,
                     mlp_adam_next(m, lr, beta1, beta2, eps));
  SV_HIP(hipGetLastError());
  SV_HIP(hipStreamSynchronize(m->stream));
  return SV_OK;
  MLP_GUARD_END
}

int sv_mlp_train(sv_mlp* m, const float* x_dev, const float* y_dev, int n, int epochs, float lr, float* final_loss) {
  if (!m || !x_dev || !y_dev || n < 1 || epochs < 1 || !(lr > 0)) return fail(SV_EINVAL, "bad arguments");
  MLP_GUARD_BEGIN
  mlp_reserve(m, n);  // before the first step is counted
  for (int e = 0; e < epochs; ++e) {
    const AdamArgs adam = mlp_adam_next(m, lr, 0.9f, 0.999f, 1e-8f);
    mlp_loss_grad_async(m, x_dev, y_dev, n, &adam);
  }
  mlp_loss_grad_async(m, x_dev, y_dev, n);  // loss at the final parameters
  SV_HIP(hipMemcpyAsync(m->host_pinned + m->nparams, m->loss_dev, sizeof(float), hipMemcpyDeviceToHost, m->stream));
  SV_HIP(hipStreamSynchronize(m->stream));
  if (final_loss) *final_loss = m->host_pinned[m->nparams];
  return SV_OK;
  MLP_GUARD_END
}

int sv_cost_model_install(sv_mlp* m) {
  return host_guard([&]() -> int {
    if (!m) return fail(SV_EINVAL, "NULL model");
    std::vector<float> p(m->nparams);
    if (int rc = sv_mlp_get_params(m, p.data())) return rc;
    cost_model_set(p, m->width);
    return SV_OK;
  });
}

}  // extern "C"
