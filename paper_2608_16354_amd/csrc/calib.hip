// Tangent-mode (forward-mode) kernels of the fp32 network, for the anchor calibration
// of the run tables (Sec. 3.1 after Eq. 4; Eq. 5-7).  The joint run response of Eq. 7
// moves an output perturbation through the frozen sampler tail with Jacobian-vector
// products of the whole network; the projections are linear, so their tangents are
// the same GEMMs without the bias, and only the nonlinear pieces need kernels here:
//   * LayerNorm with modulation: y = (x - mu) r, r = (var + eps)^-1/2,
//     dy = r (dxc - y mean(y dxc)), dxc = dx - mean(dx); a = y (1 + s) + sh, da = dy (1 + s);
//   * softmax attention per head, s = q.k c, ds = (dq.k + q.dk) c (c = 1/sqrt(d_h)):
//     o = sum_j P_j v_j, do = sum_j P_j (ds_j - sum_i P_i ds_i) v_j + P_j dv_j (attention_f32.hip);
//   * GELU-tanh: g = z/2 (1 + tanh u), u = sqrt(2/pi)(z + 0.044715 z^3),
//     dg = (1/2 (1 + tanh u) + z/2 (1 - tanh^2 u) sqrt(2/pi)(1 + 3 0.044715 z^2)) dz.
// Plus a fixed-order sum-of-squares reduction (the L2 norms of Eq. 5 and Eq. 7) and small
// elementwise kernels.  Many tangents at one point share the primal activations, and one
// launch serves all of them: at the small model's sizes (272 tokens) these calls are bound
// by their launches, not by their work.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>

#include "internal.h"

namespace dc {

namespace {

constexpr int kWave = 64;

__device__ inline double wave_sum(double v) {
#pragma unroll
  for (int o = kWave / 2; o > 0; o >>= 1) v += __shfl_xor(v, o, kWave);
  return v;
}

// one wave per row and tangent (blockIdx.y); the row statistics in double.  Every tangent's
// wave recomputes its primal row's statistics; the first also writes a.
__global__ void __launch_bounds__(256) k_ln_mod_jvp(const float* __restrict__ x, int rows, int d,
                                                    const float* __restrict__ shift,
                                                    const float* __restrict__ scale,
                                                    float* __restrict__ a, float eps) {
  const int lane = threadIdx.x & 63, row = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (row >= rows) return;
  const size_t base = size_t(row) * d, tan = size_t(blockIdx.y + 1) * rows * d + base;
  const float* xr = x + base;
  const float* dr = x + tan;
  double s = 0.0, sd = 0.0;
  for (int c = lane; c < d; c += kWave) {
    s += xr[c];
    sd += dr[c];
  }
  const double mu = wave_sum(s) / d, mud = wave_sum(sd) / d;
  double q = 0.0, xd = 0.0;
  for (int c = lane; c < d; c += kWave) {
    const double xc = xr[c] - mu;
    q += xc * xc;
    xd += xc * (dr[c] - mud);
  }
  const double r = 1.0 / sqrt(wave_sum(q) / d + double(eps));
  const double m_ydxc = wave_sum(xd) * r / d;
  for (int c = lane; c < d; c += kWave) {
    const double y = (xr[c] - mu) * r;
    const double dy = r * ((dr[c] - mud) - y * m_ydxc);
    const double f = 1.0 + double(scale[c]);
    if (blockIdx.y == 0) a[base + c] = float(y * f + double(shift[c]));
    a[tan + c] = float(dy * f);
  }
}

// z <- GELU_tanh(z), its n tangents dz <- GELU_tanh'(z) dz
__global__ void k_gelu_jvp(float* __restrict__ z, int n, size_t count) {
  const float c = 0.7978845608028654f;
  for (size_t i = size_t(blockIdx.x) * blockDim.x + threadIdx.x; i < count; i += size_t(gridDim.x) * blockDim.x) {
    const float v = z[i];
    const float t = tanhf(c * (v + 0.044715f * v * v * v));
    const float dg = 0.5f * (1.0f + t) + 0.5f * v * (1.0f - t * t) * c * (1.0f + 3.0f * 0.044715f * v * v);
    z[i] = 0.5f * v * (1.0f + t);
    for (int k = 1; k <= n; ++k) z[size_t(k) * count + i] *= dg;
  }
}

// patches[k, m, c p^2 + a p + b] = dx[k, c, t, p i + a, p j + b] for video tokens m = (t Hp + i) Wp + j,
// zero for the text tokens
__global__ void __launch_bounds__(256) k_patchify_tangents(const float* __restrict__ dx,
                                                           float* __restrict__ patches, int T, int Hl,
                                                           int Wl, int p, int Hp, int Wp, int N, int Nv,
                                                           size_t lat) {
  const int q = threadIdx.x & 63, m = blockIdx.x * 4 + (threadIdx.x >> 6), k = blockIdx.y;
  if (m >= N) return;
  float v = 0.f;
  if (m < Nv) {
    const int c = q / (p * p), a = (q / p) % p, b = q % p;
    const int t = m / (Hp * Wp), i = (m / Wp) % Hp, j = m % Wp;
    v = dx[size_t(k) * lat + ((size_t(c) * T + t) * Hl + (p * i + a)) * Wl + (p * j + b)];
  }
  patches[(size_t(k) * N + m) * 64 + q] = v;
}

struct Ptrs { const float* p[kMaxTangents + 1]; };

// out[k] = x + r[k]
__global__ void k_add_each(const float4* __restrict__ x, Ptrs r, size_t n4, float4* __restrict__ out,
                           size_t stride4) {
  const float4* rk = reinterpret_cast<const float4*>(r.p[blockIdx.y]);
  float4* ok = out + blockIdx.y * stride4;
  for (size_t i = size_t(blockIdx.x) * blockDim.x + threadIdx.x; i < n4; i += size_t(gridDim.x) * blockDim.x) {
    const float4 a = x[i], b = rk[i];
    ok[i] = make_float4(a.x + b.x, a.y + b.y, a.z + b.z, a.w + b.w);
  }
}

// out = alpha x + beta y
__global__ void k_lincomb(float* __restrict__ out, const float* __restrict__ x, float alpha,
                          const float* __restrict__ y, float beta, size_t n) {
  for (size_t i = size_t(blockIdx.x) * blockDim.x + threadIdx.x; i < n; i += size_t(gridDim.x) * blockDim.x)
    out[i] = alpha * x[i] + beta * y[i];
}

// out = alpha (x - y): the difference first, which is exact where x and y are close
__global__ void k_scaled_diff(float* __restrict__ out, const float* __restrict__ x,
                              const float* __restrict__ y, float alpha, size_t n) {
  for (size_t i = size_t(blockIdx.x) * blockDim.x + threadIdx.x; i < n; i += size_t(gridDim.x) * blockDim.x)
    out[i] = alpha * (x[i] - y[i]);
}

// fixed-order partial sums of pair blockIdx.y: part[b] = (sum (a - b)^2, sum a^2) over block b's
// strided elements; k_sumsq_final adds the kSqBlocks partials in a fixed order
constexpr int kSqBlocks = 256;
constexpr int kSqPairs = kMaxTangents;
struct SqPtrs { const float* a[kSqPairs]; const float* b[kSqPairs]; };

__global__ void __launch_bounds__(256) k_sumsq(SqPtrs ptr, size_t n, double* __restrict__ part) {
  __shared__ double red[4][2];
  const float* a = ptr.a[blockIdx.y];
  const float* b = ptr.b[blockIdx.y];
  double s1 = 0.0, s2 = 0.0;
  for (size_t i = size_t(blockIdx.x) * 256 + threadIdx.x; i < n; i += size_t(kSqBlocks) * 256) {
    const double av = a[i];
    const double dv = b ? av - double(b[i]) : av;
    s1 += dv * dv;
    s2 += av * av;
  }
  s1 = wave_sum(s1);
  s2 = wave_sum(s2);
  if ((threadIdx.x & 63) == 0) {
    red[threadIdx.x >> 6][0] = s1;
    red[threadIdx.x >> 6][1] = s2;
  }
  __syncthreads();
  if (threadIdx.x < 2)
    part[2 * (size_t(blockIdx.y) * kSqBlocks + blockIdx.x) + threadIdx.x] =
        ((red[0][threadIdx.x] + red[1][threadIdx.x]) + red[2][threadIdx.x]) + red[3][threadIdx.x];
}

__global__ void __launch_bounds__(128) k_sumsq_final(const double* __restrict__ part, double* __restrict__ out) {
  // wave q adds quantity q: four partials per lane, then the lanes, in a fixed order
  const int lane = threadIdx.x & 63, q = threadIdx.x >> 6;
  const double* p = part + 2 * size_t(blockIdx.x) * kSqBlocks + q;
  double s = 0.0;
  for (int i = lane; i < kSqBlocks; i += kWave) s += p[2 * i];
  s = wave_sum(s);
  if (lane == 0) out[2 * blockIdx.x + q] = s;
}

inline unsigned grid_of(size_t n, unsigned cap) {
  const size_t g = (n + 255) / 256;
  return unsigned(g < 1 ? 1 : (g > cap ? cap : g));
}

}  // namespace

Status ln_mod_jvp(const float* x, int n, int rows, int d, const float* shift, const float* scale, float* a,
                  float eps, hipStream_t s) {
  if (rows <= 0 || n <= 0) return Status::ok();
  hipLaunchKernelGGL(k_ln_mod_jvp, dim3((rows + 3) / 4, n), dim3(256), 0, s, x, rows, d, shift, scale, a, eps);
  DC_HIP(hipGetLastError());
  return Status::ok();
}

Status gelu_jvp(float* z, int n, size_t count, hipStream_t s) {
  hipLaunchKernelGGL(k_gelu_jvp, dim3(grid_of(count, 4096)), dim3(256), 0, s, z, n, count);
  DC_HIP(hipGetLastError());
  return Status::ok();
}

Status patchify_tangents(const float* dx, float* patches, const Geo& g, int n, hipStream_t s) {
  hipLaunchKernelGGL(k_patchify_tangents, dim3((g.N + 3) / 4, n), dim3(256), 0, s, dx, patches, g.T, g.Hl,
                     g.Wl, g.p, g.Hp, g.Wp, g.N, g.Nv, size_t(g.C) * g.T * g.Hl * g.Wl);
  DC_HIP(hipGetLastError());
  return Status::ok();
}

Status add_each(const float* x, const float* const* r, int n, size_t count, float* out, size_t stride,
                hipStream_t s) {
  if (n < 1 || n > kMaxTangents + 1) return Status::arg("add_each: bad count");
  Ptrs p{};
  for (int i = 0; i < n; ++i) p.p[i] = r[i];
  hipLaunchKernelGGL(k_add_each, dim3(grid_of(count / 4, 2048), n), dim3(256), 0, s,
                     reinterpret_cast<const float4*>(x), p, count / 4, reinterpret_cast<float4*>(out), stride / 4);
  DC_HIP(hipGetLastError());
  return Status::ok();
}

Status lincomb(float* out, const float* x, float alpha, const float* y, float beta, size_t n,
               hipStream_t s) {
  hipLaunchKernelGGL(k_lincomb, dim3(grid_of(n, 4096)), dim3(256), 0, s, out, x, alpha, y, beta, n);
  DC_HIP(hipGetLastError());
  return Status::ok();
}

Status scaled_diff(float* out, const float* x, const float* y, float alpha, size_t n, hipStream_t s) {
  hipLaunchKernelGGL(k_scaled_diff, dim3(grid_of(n, 4096)), dim3(256), 0, s, out, x, y, alpha, n);
  DC_HIP(hipGetLastError());
  return Status::ok();
}

size_t sumsq_scratch_doubles() { return size_t(2) * kSqBlocks * kSqPairs; }

Status sumsq(const float* const* a, const float* const* b, int count, size_t n, double* scratch, double* out2,
             hipStream_t s) {
  for (int i0 = 0; i0 < count; i0 += kSqPairs) {
    const int c = std::min(kSqPairs, count - i0);
    SqPtrs p{};
    for (int i = 0; i < c; ++i) {
      p.a[i] = a[i0 + i];
      p.b[i] = b ? b[i0 + i] : nullptr;
    }
    hipLaunchKernelGGL(k_sumsq, dim3(kSqBlocks, c), dim3(256), 0, s, p, n, scratch);
    DC_HIP(hipGetLastError());
    hipLaunchKernelGGL(k_sumsq_final, dim3(c), dim3(128), 0, s, scratch, out2 + 2 * i0);
    DC_HIP(hipGetLastError());
  }
  return Status::ok();
}

}  // namespace dc
