// Cost-model MLP: forward, backward and Adam kernels (FP32); the host
// forward for the planner is in sv_mlp_host.cpp.  Sizes are tiny (5k
// parameters, batches of a few thousand rows), so a step is bound by latency:
// launches, and the chain of each sum.  A network of at most 64 inputs and 64
// hidden units runs a wave per row with the weights in LDS (one launch
// forward, one for the row part of the backward pass); the sums over the batch
// take a wave's lane per column and 16 slices of the rows, combined in a
// fixed order so every run gives the same bits.
#include <cmath>
#include <vector>

#include "sv_internal.h"
#include "sv_mlp.h"
#include "sv_mlp_layout.h"

namespace sv {
namespace {

constexpr int kT = 256;

using Off = MlpOffsets;
inline Off offsets(int nin, int hid) { return mlp_offsets(nin, hid); }

// z[r][u] = sum_i in[r][i] W[i][u] + b[u]; relu_in: apply relu to `in` on read
__global__ __launch_bounds__(kT) void k_dense(const float *__restrict__ in, int nin, bool relu_in,
                                              const float *__restrict__ W, const float *__restrict__ b, int hid,
                                              int batch, float *__restrict__ z) {
  const int64_t idx = int64_t(blockIdx.x) * kT + threadIdx.x;
  if (idx >= int64_t(batch) * hid) return;
  const int r = int(idx / hid), u = int(idx % hid);
  float acc = b[u];
  for (int i = 0; i < nin; ++i) {
    float x = in[int64_t(r) * nin + i];
    if (relu_in) x = x > 0.f ? x : 0.f;
    acc = fmaf(x, W[i * hid + u], acc);
  }
  z[idx] = acc;
}

__global__ __launch_bounds__(kT) void k_out(const float *__restrict__ z2, int hid, const float *__restrict__ w3,
                                            const float *__restrict__ b3, int batch, float *__restrict__ y) {
  const int r = blockIdx.x * kT + threadIdx.x;
  if (r >= batch) return;
  float acc = b3[0];
  for (int u = 0; u < hid; ++u) {
    const float h = z2[int64_t(r) * hid + u];
    acc = fmaf(h > 0.f ? h : 0.f, w3[u], acc);
  }
  y[r] = acc;
}

// Forward of up to 64 inputs and 64 hidden units: lane u of a wave is hidden
// unit u of the wave's row; sums run in input order, as in k_dense.
constexpr int kRowWaves = 4, kRowsPerWave = 4, kMaxUnits = 64;
__global__ __launch_bounds__(64 * kRowWaves) void k_forward_rows(const float *__restrict__ X, int nin, int hid,
                                                                 const float *__restrict__ params, Off o, int batch,
                                                                 float *__restrict__ z1, float *__restrict__ z2,
                                                                 float *__restrict__ y) {
  __shared__ float w1[kMaxUnits * kMaxUnits], w2[kMaxUnits * kMaxUnits];
  __shared__ float row[kRowWaves][kMaxUnits];
  for (int i = threadIdx.x; i < nin * hid; i += 64 * kRowWaves) w1[i] = params[o.w1 + i];
  for (int i = threadIdx.x; i < hid * hid; i += 64 * kRowWaves) w2[i] = params[o.w2 + i];
  const int u = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const bool on = u < hid;
  const float b1 = on ? params[o.b1 + u] : 0.f, b2 = on ? params[o.b2 + u] : 0.f;
  const float w3 = on ? params[o.w3 + u] : 0.f, b3 = params[o.b3];
  const int uu = on ? u : 0;
  __syncthreads();
  for (int j = 0; j < kRowsPerWave; ++j) {
    const int r = (int(blockIdx.x) * kRowsPerWave + j) * kRowWaves + wave;
    const bool live = r < batch;
    if (live && u < nin) row[wave][u] = X[int64_t(r) * nin + u];
    __syncthreads();
    float a = b1;
#pragma unroll 4
    for (int i = 0; i < nin; ++i) a = fmaf(row[wave][i], w1[i * hid + uu], a);
    __syncthreads();
    row[wave][u] = a > 0.f ? a : 0.f;
    if (live && on) z1[int64_t(r) * hid + u] = a;
    __syncthreads();
    float c = b2;
#pragma unroll 8
    for (int i = 0; i < hid; ++i) c = fmaf(row[wave][i], w2[i * hid + uu], c);
    if (live && on) z2[int64_t(r) * hid + u] = c;
    float s = (on && c > 0.f) ? c * w3 : 0.f;
#pragma unroll
    for (int m = 32; m > 0; m >>= 1) s += __shfl_xor(s, m);
    if (live && u == 0) y[r] = s + b3;
    __syncthreads();
  }
}

// Row part of the backward pass, likewise: dz2 = dy w3 [z2 > 0], then
// dz1[a] = sum_u dz2[u] W2[a][u] [z1 > 0] with W2's rows a word apart in LDS.
__global__ __launch_bounds__(64 * kRowWaves) void k_backward_rows(const float *__restrict__ y,
                                                                  const float *__restrict__ t, int hid,
                                                                  const float *__restrict__ params, Off o, int batch,
                                                                  const float *__restrict__ z1,
                                                                  const float *__restrict__ z2,
                                                                  float *__restrict__ dz1, float *__restrict__ dz2) {
  __shared__ float w2[kMaxUnits * (kMaxUnits + 1)];
  __shared__ float row[kRowWaves][kMaxUnits];
  for (int i = threadIdx.x; i < hid * hid; i += 64 * kRowWaves)
    w2[(i / hid) * (kMaxUnits + 1) + i % hid] = params[o.w2 + i];
  const int u = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const bool on = u < hid;
  const float w3 = on ? params[o.w3 + u] : 0.f;
  const int uu = on ? u : 0;
  __syncthreads();
  for (int j = 0; j < kRowsPerWave; ++j) {
    const int r = (int(blockIdx.x) * kRowsPerWave + j) * kRowWaves + wave;
    const bool live = r < batch && on;
    const int64_t at = int64_t(r) * hid + u;
    const float dy = live ? (y[r] - t[r]) / float(batch) : 0.f;
    const float d2 = live && z2[at] > 0.f ? dy * w3 : 0.f;
    if (live) dz2[at] = d2;
    row[wave][u] = d2;
    __syncthreads();
    float a = 0.f;
#pragma unroll 8
    for (int i = 0; i < hid; ++i) a = fmaf(row[wave][i], w2[uu * (kMaxUnits + 1) + i], a);
    if (live) dz1[at] = z1[at] > 0.f ? a : 0.f;
    __syncthreads();
  }
}

// Sums over the batch: workgroup x is one gradient row (W2's rows and b2, W1's
// rows and b1, W3, then b3 and the loss), workgroup y 64 of its columns.  A lane
// takes a column, a wave one of 16 slices of the rows; the slices meet in LDS
// in order.  One thread per output over the whole batch (1712 rows) took 414
// us for each layer and 475 for the output; all of them
// take 23 us.
constexpr int kSlices = 16;
__global__ __launch_bounds__(64 * kSlices) void k_grads(const float *__restrict__ X, int nin, int hid,
                                                        const float *__restrict__ z1, const float *__restrict__ z2,
                                                        const float *__restrict__ dz1,
                                                        const float *__restrict__ dz2, const float *__restrict__ y,
                                                        const float *__restrict__ t, Off o, int batch,
                                                        float *__restrict__ grads, float *__restrict__ loss) {
  __shared__ float red[2][kSlices][64];
  const int lane = threadIdx.x & 63, slice = threadIdx.x >> 6;
  const int u = int(blockIdx.y) * 64 + lane;
  int g = blockIdx.x;
  const bool last = g == hid + nin + 3;
  float s = 0.f, q = 0.f;
  float *out = nullptr;
  if (g <= hid + nin + 1) {  // a row of a weight matrix, or its bias
    const bool second = g <= hid;
    const int i = second ? g : g - (hid + 1), ni = second ? hid : nin;
    const float *in = second ? z1 : X, *d = second ? dz2 : dz1;
    out = grads + (i < ni ? (second ? o.w2 : o.w1) + int64_t(i) * hid : int64_t(second ? o.b2 : o.b1));
    // eight rows at a time, all their loads before the first sum
    const bool bias = i == ni;
    const float *xp = in + (bias ? 0 : i), *dp = d + (u < hid ? u : 0);
    for (int r0 = slice; r0 < batch; r0 += 8 * kSlices) {
      float x[8], e[8];
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        const int r = r0 + k * kSlices, rc = r < batch ? r : r0;
        x[k] = xp[int64_t(rc) * ni];
        e[k] = dp[int64_t(rc) * hid];
        if (r >= batch) x[k] = e[k] = 0.f;
      }
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        const float h = second && !(x[k] > 0.f) ? 0.f : x[k];
        s = fmaf(bias ? 1.f : h, e[k], s);
      }
    }
  } else if (!last) {  // W3
    out = grads + o.w3;
    const float *zp = z2 + (u < hid ? u : 0);
    for (int r0 = slice; r0 < batch; r0 += 8 * kSlices) {
      float h[8], e[8];
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        const int r = r0 + k * kSlices, rc = r < batch ? r : r0;
        h[k] = zp[int64_t(rc) * hid];
        e[k] = (y[rc] - t[rc]) / float(batch);
        if (r >= batch) h[k] = e[k] = 0.f;
      }
#pragma unroll
      for (int k = 0; k < 8; ++k) s = fmaf(h[k] > 0.f ? h[k] : 0.f, e[k], s);
    }
  } else if (blockIdx.y == 0) {  // b3 and the loss: the rows over all threads
    for (int r = threadIdx.x; r < batch; r += 64 * kSlices) {
      const float e = y[r] - t[r];
      s += e / float(batch);
      q = fmaf(e, e, q);
    }
  }
  red[0][slice][lane] = s;
  red[1][slice][lane] = q;
  __syncthreads();
  if (slice) return;
  for (int k = 1; k < kSlices; ++k) {
    s += red[0][k][lane];
    q += red[1][k][lane];
  }
  if (last) {
#pragma unroll
    for (int m = 32; m > 0; m >>= 1) {
      s += __shfl_xor(s, m);
      q += __shfl_xor(q, m);
    }
    if (lane == 0 && blockIdx.y == 0) {
      grads[o.b3] = s;
      *loss = 0.5f * q / float(batch);
    }
  } else if (u < hid) {
    out[u] = s;
  }
}

// dz2[r][u] = (y - t)/B * w3[u] * [z2 > 0]
__global__ __launch_bounds__(kT) void k_dz2(const float *__restrict__ y, const float *__restrict__ t,
                                            const float *__restrict__ z2, const float *__restrict__ w3, int hid,
                                            int batch, float *__restrict__ dz2) {
  const int64_t idx = int64_t(blockIdx.x) * kT + threadIdx.x;
  if (idx >= int64_t(batch) * hid) return;
  const int r = int(idx / hid), u = int(idx % hid);
  const float dy = (y[r] - t[r]) / float(batch);
  dz2[idx] = z2[idx] > 0.f ? dy * w3[u] : 0.f;
}

// dz1[r][a] = sum_u dz2[r][u] W2[a][u] * [z1 > 0]
__global__ __launch_bounds__(kT) void k_dz1(const float *__restrict__ dz2, const float *__restrict__ W2,
                                            const float *__restrict__ z1, int hid, int batch,
                                            float *__restrict__ dz1) {
  const int64_t idx = int64_t(blockIdx.x) * kT + threadIdx.x;
  if (idx >= int64_t(batch) * hid) return;
  const int r = int(idx / hid), a = int(idx % hid);
  float acc = 0.f;
  for (int u = 0; u < hid; ++u) acc = fmaf(dz2[int64_t(r) * hid + u], W2[a * hid + u], acc);
  dz1[idx] = z1[idx] > 0.f ? acc : 0.f;
}

__global__ __launch_bounds__(kT) void k_adam(float *__restrict__ p, const float *__restrict__ g,
                                             float *__restrict__ m, float *__restrict__ v, int count, float lr,
                                             float b1, float b2, float eps, float c1, float c2) {
  const int i = blockIdx.x * kT + threadIdx.x;
  if (i >= count) return;
  const float gi = g[i];
  const float mi = b1 * m[i] + (1.f - b1) * gi;
  const float vi = b2 * v[i] + (1.f - b2) * gi * gi;
  m[i] = mi;
  v[i] = vi;
  const float mhat = mi / c1, vhat = vi / c2;
  p[i] -= lr * mhat / (sqrtf(vhat) + eps);
}

unsigned blocks(int64_t n) { return unsigned((n + kT - 1) / kT); }

// Networks that fit the row kernels, and their launch.
bool rows_fit(int nin, int hid) { return nin <= kMaxUnits && hid <= kMaxUnits; }
unsigned row_blocks(int batch) { return unsigned((int64_t(batch) + kRowWaves * kRowsPerWave - 1) / (kRowWaves * kRowsPerWave)); }

}  // namespace
}  // namespace sv

using namespace sv;

extern "C" {

int sv_mlp_forward(const float *params, int nin, int hid, const float *X, int batch, float *y, float *cache,
                   void *stream) {
  return guard([&]() -> int {
    if (!params || !X || !y || nin < 1 || hid < 1 || batch < 1 || !cache) {
      set_error("bad mlp forward argument (cache is required)");
      return SV_ERR_ARG;
    }
    hipStream_t st = static_cast<hipStream_t>(stream);
    const Off o = offsets(nin, hid);
    float *z1 = cache, *z2 = cache + int64_t(hid) * batch;
    if (rows_fit(nin, hid)) {
      hipLaunchKernelGGL(k_forward_rows, dim3(row_blocks(batch)), dim3(64 * kRowWaves), 0, st, X, nin, hid, params, o,
                         batch, z1, z2, y);
      SV_HIP_CHECK(hipGetLastError());
      return SV_OK;
    }
    hipLaunchKernelGGL(k_dense, dim3(blocks(int64_t(batch) * hid)), dim3(kT), 0, st, X, nin, false, params + o.w1,
                       params + o.b1, hid, batch, z1);
    hipLaunchKernelGGL(k_dense, dim3(blocks(int64_t(batch) * hid)), dim3(kT), 0, st, z1, hid, true, params + o.w2,
                       params + o.b2, hid, batch, z2);
    hipLaunchKernelGGL(k_out, dim3(blocks(batch)), dim3(kT), 0, st, z2, hid, params + o.w3, params + o.b3, batch, y);
    SV_HIP_CHECK(hipGetLastError());
    return SV_OK;
  });
}

int sv_mlp_backward(const float *params, int nin, int hid, const float *X, const float *target, int batch,
                    const float *y, const float *cache, float *grads, float *loss, void *stream) {
  return guard([&]() -> int {
    if (!params || !X || !target || !y || !cache || !grads || !loss || nin < 1 || hid < 1 || batch < 1) {
      set_error("bad mlp backward argument");
      return SV_ERR_ARG;
    }
    hipStream_t st = static_cast<hipStream_t>(stream);
    const Off o = offsets(nin, hid);
    const float *z1 = cache, *z2 = cache + int64_t(hid) * batch;
    float *dz2 = const_cast<float *>(cache) + 2 * int64_t(hid) * batch;
    float *dz1 = const_cast<float *>(cache) + 3 * int64_t(hid) * batch;
    if (rows_fit(nin, hid)) {
      hipLaunchKernelGGL(k_backward_rows, dim3(row_blocks(batch)), dim3(64 * kRowWaves), 0, st, y, target, hid, params,
                         o, batch, z1, z2, dz1, dz2);
    } else {
      hipLaunchKernelGGL(k_dz2, dim3(blocks(int64_t(batch) * hid)), dim3(kT), 0, st, y, target, z2, params + o.w3, hid,
                         batch, dz2);
      hipLaunchKernelGGL(k_dz1, dim3(blocks(int64_t(batch) * hid)), dim3(kT), 0, st, dz2, params + o.w2, z1, hid, batch,
                         dz1);
    }
    hipLaunchKernelGGL(k_grads, dim3(unsigned(hid + nin + 4), unsigned((hid + 63) / 64)), dim3(64 * kSlices), 0, st, X,
                       nin, hid, z1, z2, dz1, dz2, y, target, o, batch, grads, loss);
    SV_HIP_CHECK(hipGetLastError());
    return SV_OK;
  });
}

int sv_mlp_adam(float *params, const float *grads, float *m, float *v, int count, int t, float lr, float beta1,
                float beta2, float eps, void *stream) {
  return guard([&]() -> int {
    if (!params || !grads || !m || !v || count < 1 || t < 1) {
      set_error("bad adam argument");
      return SV_ERR_ARG;
    }
    const float c1 = 1.f - std::pow(beta1, float(t)), c2 = 1.f - std::pow(beta2, float(t));
    hipLaunchKernelGGL(k_adam, dim3(blocks(count)), dim3(kT), 0, static_cast<hipStream_t>(stream), params, grads, m,
                       v, count, lr, beta1, beta2, eps, c1, c2);
    SV_HIP_CHECK(hipGetLastError());
    return SV_OK;
  });
}

}  // extern "C"
