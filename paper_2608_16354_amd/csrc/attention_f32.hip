// fp32 attention of the fp32 model and its tangent for the anchor calibration, on
// v_mfma_f32_16x16x4_f32 (fp32 operands, fp32 accumulation).
//
// softmax(Q K^T / sqrt(d_h)) V per head over qkv [M, 3d] (Q | K | V, head-major columns),
// head_dim 64, with an online softmax.  The tangent form takes n tangents dqkv stacked below
// qkv and returns for each, with ds = (dq.k + q.dk) / sqrt(d_h) and P the softmax,
//   do = sum_j P_j (ds_j - sum_i P_i ds_i) v_j + P_j dv_j
// stacked below o.
//
// These calls are short (272 tokens x 4 heads in the small model), so what bounds them is
// the length of the serial chain over the keys and how few wavefronts there are: a
// workgroup takes QB blocks of 16 queries of one head, its KS waves share out the keys in
// chunks of 32 and merge their partial sums through LDS at the end.  Against the earlier
// one-thread-per-query kernels (20 workgroups of one wave): 272 tokens x 4 heads
// 697 -> 8.1 us, the tangent 826 -> 16 us; 2,400 tokens x 12 heads run at 97 TFLOP/s.
//
// Operands go global -> registers; no layout needs LDS or a transposed V:
//  - S^T = K Q^T: lane (c = lane % 16, g = lane / 16) reads 16 bytes of key c and of query c
//    at dimensions 16 j + 4 g; step s of the four k-steps takes element s of both, so the
//    k slot of lane group g is dimension 16 j + 4 g + s on either side.
//  - a lane then holds the scores of query c for keys 4 g + i, which is the B operand of
//    O^T += V^T P^T for k slot g = key 4 g + s in step s;
//  - the V^T operand of accumulator b is row c <-> dimension 4 c + b, so one 16-byte read
//    of V[key 4 g + s][4 c ..] feeds all four accumulators, and the four accumulators of a
//    lane hold four consecutive dimensions of the output.
#include <hip/hip_runtime.h>

#include <cmath>

#include "internal.h"

namespace dc {

namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kDh = 64;
constexpr int kOs = kDh + 4;       // row stride (floats) of a wave's partial output in LDS

__device__ inline f32x4 ld4(const float* p) { return *reinterpret_cast<const f32x4*>(p); }
__device__ inline f32x4 mma(float a, float b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}
__device__ inline float over_groups_max(float v) {      // over the four lanes of a query
  v = fmaxf(v, __shfl_xor(v, 16, 64));
  return fmaxf(v, __shfl_xor(v, 32, 64));
}
__device__ inline float over_groups_sum(float v) {
  v += __shfl_xor(v, 16, 64);
  return v + __shfl_xor(v, 32, 64);
}

// c2 = log2(e) / sqrt(d_h): exponentials are 2^(c2 (s - m)); rs = 1 / sqrt(d_h).
template <int QB, int KS, bool kTan>
__global__ void __launch_bounds__(KS * 64) k_attn_f32(const float* __restrict__ qkv, int M, int d,
                                                      float c2, float rs, int nqb, int items,
                                                      int per_xcd, float* __restrict__ out) {
  constexpr int NT = kTan ? 2 : 1;                  // accumulated tensors: O (and the tangent's sums)
  __shared__ float s_m[KS][QB * 16], s_l[KS][QB * 16], s_c[KS][QB * 16];
  __shared__ __attribute__((aligned(16))) float s_o[NT][KS][QB * 16 * kOs];
  // each XCD (workgroups are dealt round-robin) sweeps the query blocks of one head at a time
  const int w = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
  if (w >= items) return;
  const int head = w / nqb, q0 = (w - head * nqb) * 16 * QB;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int c = lane & 15, g = lane >> 4;
  const int ld = 3 * d;
  const float* Qb = qkv + head * kDh;
  const float* Kb = Qb + d;
  const float* Vb = Qb + 2 * d;
  // tangent blockIdx.y: from a primal element to its tangent
  const size_t tan = kTan ? size_t(blockIdx.y + 1) * M * ld : 0;

  f32x4 qf[QB][4], dqf[kTan ? QB : 1][4];
#pragma unroll
  for (int b = 0; b < QB; ++b) {
    const float* r = Qb + size_t(min(q0 + 16 * b + c, M - 1)) * ld + 4 * g;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      qf[b][j] = ld4(r + 16 * j);
      if constexpr (kTan) dqf[b][j] = ld4(r + tan + 16 * j);
    }
  }
  const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
  f32x4 o[NT][QB][4];
  float m[QB], l[QB], cs[QB];                       // l, cs: this lane's keys only
#pragma unroll
  for (int b = 0; b < QB; ++b) {
    m[b] = -INFINITY;
    l[b] = cs[b] = 0.f;
#pragma unroll
    for (int n = 0; n < NT; ++n)
#pragma unroll
      for (int i = 0; i < 4; ++i) o[n][b][i] = zero;
  }

  for (int k0 = 32 * wave; k0 < M; k0 += 32 * KS) {
    f32x4 kf[2][4], vf[2][4], dkf[kTan ? 2 : 1][4], dvf[kTan ? 2 : 1][4];
#pragma unroll
    for (int h = 0; h < 2; ++h) {                   // 16-key halves; rows past M re-read the last one
      const float* kr = Kb + size_t(min(k0 + 16 * h + c, M - 1)) * ld + 4 * g;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        kf[h][j] = ld4(kr + 16 * j);
        if constexpr (kTan) dkf[h][j] = ld4(kr + tan + 16 * j);
      }
    }
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        const float* vr = Vb + size_t(min(k0 + 16 * h + 4 * g + s, M - 1)) * ld + 4 * c;
        vf[h][s] = ld4(vr);
        if constexpr (kTan) dvf[h][s] = ld4(vr + tan);
      }
    f32x4 sc[QB][2], ds[kTan ? QB : 1][2];
#pragma unroll
    for (int b = 0; b < QB; ++b)
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        sc[b][h] = zero;
        if constexpr (kTan) ds[b][h] = zero;
      }
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int b = 0; b < QB; ++b)
#pragma unroll
          for (int h = 0; h < 2; ++h) {
            sc[b][h] = mma(kf[h][j][s], qf[b][j][s], sc[b][h]);
            if constexpr (kTan) {
              ds[b][h] = mma(kf[h][j][s], dqf[b][j][s], ds[b][h]);
              ds[b][h] = mma(dkf[h][j][s], qf[b][j][s], ds[b][h]);
            }
          }
    if (k0 + 32 > M) {
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (k0 + 16 * h + 4 * g + i >= M)
#pragma unroll
            for (int b = 0; b < QB; ++b) sc[b][h][i] = -INFINITY;
    }
#pragma unroll
    for (int b = 0; b < QB; ++b) {
      float mx = sc[b][0][0];
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int i = 0; i < 4; ++i) mx = fmaxf(mx, sc[b][h][i]);
      const float mn = fmaxf(m[b], over_groups_max(mx));   // finite: a chunk holds a key below M
      const float al = __builtin_amdgcn_exp2f((m[b] - mn) * c2);
      m[b] = mn;
      l[b] *= al;
      if constexpr (kTan) cs[b] *= al;
#pragma unroll
      for (int n = 0; n < NT; ++n)
#pragma unroll
        for (int i = 0; i < 4; ++i) o[n][b][i] *= al;
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const float p = __builtin_amdgcn_exp2f((sc[b][h][i] - mn) * c2);
          sc[b][h][i] = p;
          l[b] += p;
          if constexpr (kTan) {
            const float pd = p * (ds[b][h][i] * rs);
            ds[b][h][i] = pd;
            cs[b] += pd;
          }
        }
    }
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int b = 0; b < QB; ++b) {
            o[0][b][i] = mma(vf[h][s][i], sc[b][h][s], o[0][b][i]);
            if constexpr (kTan) {
              o[1][b][i] = mma(vf[h][s][i], ds[b][h][s], o[1][b][i]);
              o[1][b][i] = mma(dvf[h][s][i], sc[b][h][s], o[1][b][i]);
            }
          }
  }

  // merge: every wave scales its sums to the common maximum, then threads add the KS partials
  // (a wave without keys has m = -inf and scales by 0)
#pragma unroll
  for (int b = 0; b < QB; ++b)
    if (g == 0) s_m[wave][16 * b + c] = m[b];
  __syncthreads();
#pragma unroll
  for (int b = 0; b < QB; ++b) {
    const int q = 16 * b + c;
    float mx = s_m[0][q];
#pragma unroll
    for (int v = 1; v < KS; ++v) mx = fmaxf(mx, s_m[v][q]);
    const float al = __builtin_amdgcn_exp2f((m[b] - mx) * c2);
    const float lw = over_groups_sum(l[b]) * al;
    float cw = 0.f;
    if constexpr (kTan) cw = over_groups_sum(cs[b]) * al;
    if (g == 0) {
      s_l[wave][q] = lw;
      s_c[wave][q] = cw;
    }
#pragma unroll
    for (int n = 0; n < NT; ++n)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const f32x4 v = {o[n][b][0][i] * al, o[n][b][1][i] * al, o[n][b][2][i] * al, o[n][b][3][i] * al};
        *reinterpret_cast<f32x4*>(&s_o[n][wave][q * kOs + 16 * g + 4 * i]) = v;
      }
  }
  __syncthreads();
  for (int e = tid; e < QB * 16 * 16; e += KS * 64) {
    const int q = e >> 4, c4 = (e & 15) * 4;
    if (q0 + q >= M) continue;
    float lt = 0.f, ct = 0.f;
    f32x4 a = zero, t = zero;
#pragma unroll
    for (int v = 0; v < KS; ++v) {
      lt += s_l[v][q];
      a += *reinterpret_cast<const f32x4*>(&s_o[0][v][q * kOs + c4]);
      if constexpr (kTan) {
        ct += s_c[v][q];
        t += *reinterpret_cast<const f32x4*>(&s_o[NT - 1][v][q * kOs + c4]);
      }
    }
    const float inv = 1.0f / lt;
    const size_t dst = size_t(q0 + q) * d + head * kDh + c4;
    if (!kTan || blockIdx.y == 0) *reinterpret_cast<f32x4*>(out + dst) = a * inv;
    if constexpr (kTan)
      *reinterpret_cast<f32x4*>(out + size_t(blockIdx.y + 1) * M * d + dst) = (t - a * (ct * inv)) * inv;
  }
}

template <int QB, int KS, bool kTan>
Status launch(const float* qkv, int n, const Geo& g, int M, float* o, hipStream_t s) {
  const int nqb = (M + 16 * QB - 1) / (16 * QB), items = nqb * g.H, per_xcd = (items + 7) / 8;
  const double rs = 1.0 / std::sqrt(double(g.Dh));
  hipLaunchKernelGGL((k_attn_f32<QB, KS, kTan>), dim3(8 * per_xcd, n), dim3(KS * 64), 0, s, qkv, M, g.d,
                     float(1.4426950408889634 * rs), float(rs), nqb, items, per_xcd, o);
  DC_HIP(hipGetLastError());
  return Status::ok();
}

}  // namespace

// Which split.  A compute unit works through its workgroups at a rate that hardly depends on
// how many it holds, so the time follows the rounds ceil(workgroups / compute units); a round
// of 32 queries takes 1.65 to 1.8 rounds of 16.  Measured on 256 compute units: 8 heads x 1,000
// tokens 25.6 us in two rounds of 16 queries, 24.3 in one of 32; 8 x 2,400 121.7 us in five
// of 16, 138.3 in three of 32; 12 x 2,400 188.5 in eight, 182.5 in four.  While 16 queries
// need one round only, eight waves share the keys (4 x 1,000: 15.2 us, four waves 16.4);
// beyond, four (8 x 2,400: 121.7, eight 140.6).  The tangent is fastest with 16 queries and
// four waves throughout.
Status attention_f32(const float* qkv, float* out, const Geo& g, int M, hipStream_t s) {
  if (g.Dh != kDh) return Status::shape("fp32 attention supports head_dim 64");
  if (M <= 0) return Status::ok();
  const int64_t cus = compute_units();
  if (cus <= 0) return Status::make(DC_ERR_HIP, "fp32 attention: no device");
  const int64_t r16 = (int64_t(g.H) * ((M + 15) / 16) + cus - 1) / cus;
  const int64_t r32 = (int64_t(g.H) * ((M + 31) / 32) + cus - 1) / cus;
  if (9 * r32 < 5 * r16) return launch<2, 4, false>(qkv, 1, g, M, out, s);
  if (r16 > 1) return launch<1, 4, false>(qkv, 1, g, M, out, s);
  return launch<1, 8, false>(qkv, 1, g, M, out, s);
}

Status attention_jvp_f32(const float* qkv, int n, const Geo& g, int M, float* o, hipStream_t s) {
  if (g.Dh != kDh) return Status::shape("calibration attention tangent supports head_dim 64");
  if (M <= 0 || n <= 0) return Status::ok();
  return launch<1, 4, true>(qkv, n, g, M, o, s);
}

}  // namespace dc
