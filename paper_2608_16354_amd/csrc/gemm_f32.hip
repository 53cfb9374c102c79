// fp32 GEMMs with fused epilogues, C = A W^T, on v_mfma_f32_16x16x4_f32 (fp32 operands and
// accumulation): the fp32 model, the timestep MLP and modulation of every model, and the
// tangent passes of the calibration (those also with bf16 weights, widened exactly on load).
//
// Two kernels:
//  - k_gemm_f32: operands global -> registers.  Lane (c = lane % 16, g = lane / 16) reads 16
//    bytes of row c at k = 16 j + 4 g, and step s of the four MFMA k-steps takes element s on
//    both sides (the same k permutation for A and W).  SK waves split the K chunks of one
//    tile and add their partial sums through LDS in a fixed order.  For the calls too small
//    to fill the chip (272 rows x 256 columns), which are bound by launch and by the serial
//    chain over K, and for 50 rows against 88 MB of modulation weights.
//  - k_gemm_f32_lds: 64 x 64 tiles through LDS, for everything larger.
// Against the SIMT kernel this replaced (64 x 64 tile, LDS, no K split), us on MI355X:
//   272 x 256, K 256: 20.5 -> 3.7;  K 1024: 71 -> 7.5;  2400 x 768, K 3072: 101.7 (111 TFLOP/s);
//   50 x 11520, K 1920: 220 -> 33.5 called back to back (88 MB of weights: 2.6 TB/s); 40 once a
//   sample, with the weights in memory only (2.2 TB/s).
#include <hip/hip_runtime.h>

#include "internal.h"

namespace dc {

namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));

__device__ inline float gelu_tanh(float z) {
  const float y = 0.7978845608028654f * (z + 0.044715f * z * z * z);
  return z / (1.0f + __expf(-2.0f * y));
}
__device__ inline float silu(float z) { return z / (1.0f + expf(-z)); }

// Epilogues: load(m, n) fetches what the result is added to (all of a lane's loads go out
// before its first store), store(m, n, acc, loaded) writes one element.
// With bias_rows, rows from there on (the tangents stacked below a primal activation) get no bias.
struct EpiBiasAct {
  const float* bias; float* out; int ldo; int act;
  __device__ float load(int, int) const { return 0.f; }
  __device__ void store(int m, int n, float v, float) const {
    v += bias[n];
    out[size_t(m) * ldo + n] = act ? silu(v) : v;
  }
};
struct EpiBiasRows {
  const float* bias; float* out; int ldo; int bias_rows;
  __device__ float load(int, int) const { return 0.f; }
  __device__ void store(int m, int n, float v, float) const {
    out[size_t(m) * ldo + n] = m < bias_rows ? v + bias[n] : v;
  }
};
struct EpiBiasAndSilu {
  const float* bias; float* out; float* silu_out; int ldo;
  __device__ float load(int, int) const { return 0.f; }
  __device__ void store(int m, int n, float v, float) const {
    v += bias[n];
    out[size_t(m) * ldo + n] = v;
    silu_out[size_t(m) * ldo + n] = silu(v);
  }
};
struct EpiGelu {
  const float* bias; float* out; int ldo;
  __device__ float load(int, int) const { return 0.f; }
  __device__ void store(int m, int n, float v, float) const { out[size_t(m) * ldo + n] = gelu_tanh(v + bias[n]); }
};
struct EpiGateResidual {
  const float* bias; const float* gate; float* h; int ldh;
  __device__ float load(int m, int n) const { return h[size_t(m) * ldh + n]; }
  __device__ void store(int m, int n, float v, float old) const {
    h[size_t(m) * ldh + n] = old + gate[n] * (v + bias[n]);
  }
};
struct EpiGateResidualRows {
  const float* bias; const float* gate; float* h; int ldh; int bias_rows;
  __device__ float load(int m, int n) const { return h[size_t(m) * ldh + n]; }
  __device__ void store(int m, int n, float v, float old) const {
    h[size_t(m) * ldh + n] = old + gate[n] * (m < bias_rows ? v + bias[n] : v);
  }
};
// token m, patch-vector index n -> latent element; x += dsigma * (acc + b)
struct EpiHeadEuler {
  const float* bias; float* x; float dsigma; int T, Hl, Wl, p, Hp, Wp;
  __device__ size_t at(int m, int n) const {
    const int pp = p * p;
    const int c = n / pp, a = (n / p) % p, b = n % p;
    const int t = m / (Hp * Wp), i = (m / Wp) % Hp, j = m % Wp;
    return ((size_t(c) * T + t) * Hl + (p * i + a)) * Wl + (p * j + b);
  }
  __device__ float load(int m, int n) const { return x[at(m, n)]; }
  __device__ void store(int m, int n, float v, float old) const { x[at(m, n)] = old + dsigma * (v + bias[n]); }
};
// the same for tangents: row m = token m % N of tangent m / N, tokens from Nv on (text) have no
// output, no bias; x: one latent of `lat` elements per tangent
struct EpiHeadTangents {
  EpiHeadEuler e; int N, Nv; size_t lat;
  __device__ float load(int m, int n) const { return e.x[size_t(m / N) * lat + e.at(min(m % N, Nv - 1), n)]; }
  __device__ void store(int m, int n, float v, float old) const {
    if (m % N < Nv) e.x[size_t(m / N) * lat + e.at(m % N, n)] = old + e.dsigma * v;
  }
};

// four consecutive weights as fp32
__device__ inline f32x4 ld4(const float* p) { return *reinterpret_cast<const f32x4*>(p); }
__device__ inline f32x4 ld4(const uint16_t* p) {
  const uint2 u = *reinterpret_cast<const uint2*>(p);
  const f32x4 r = {__uint_as_float(u.x << 16), __uint_as_float(u.x & 0xFFFF0000u),
                   __uint_as_float(u.y << 16), __uint_as_float(u.y & 0xFFFF0000u)};
  return r;
}

// A tile of TM x TN blocks of 16 x 16; SK waves split its K chunks (of 16 KC).  Rows and
// columns past M and N re-read the last.
template <int TM, int TN, int SK, int KC, class Epi, class WT>
__global__ void __launch_bounds__(SK * 64) k_gemm_f32(const float* __restrict__ A, int lda,
                                                      const WT* __restrict__ W, int ldw, int M, int N,
                                                      int K, int tiles_n, int tiles, int per_xcd, Epi epi) {
  constexpr int BM = 16 * TM, BN = 16 * TN;
  const int t = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);   // an XCD runs neighbouring tiles
  if (t >= tiles) return;
  const int m0 = t / tiles_n * BM, n0 = t % tiles_n * BN;
  const int tid = threadIdx.x, lane = tid & 63;
  const int sk = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int c = lane & 15, g = lane >> 4;

  const float* ap[TM];
  const WT* wp[TN];
#pragma unroll
  for (int a = 0; a < TM; ++a) ap[a] = A + size_t(min(m0 + 16 * a + c, M - 1)) * lda + 4 * g;
#pragma unroll
  for (int b = 0; b < TN; ++b) wp[b] = W + size_t(min(n0 + 16 * b + c, N - 1)) * ldw + 4 * g;
  f32x4 acc[TM][TN];
#pragma unroll
  for (int a = 0; a < TM; ++a)
#pragma unroll
    for (int b = 0; b < TN; ++b) acc[a][b] = f32x4{0.f, 0.f, 0.f, 0.f};

  struct Frag { f32x4 a[TM][KC], w[TN][KC]; };
  auto load = [&](Frag& f, int k) {
#pragma unroll
    for (int j = 0; j < KC; ++j) {
#pragma unroll
      for (int a = 0; a < TM; ++a) f.a[a][j] = ld4(ap[a] + k + 16 * j);
#pragma unroll
      for (int b = 0; b < TN; ++b) f.w[b][j] = ld4(wp[b] + k + 16 * j);
    }
  };
  auto mul = [&](const Frag& f) {
#pragma unroll
    for (int j = 0; j < KC; ++j)
#pragma unroll
      for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int a = 0; a < TM; ++a)
#pragma unroll
          for (int b = 0; b < TN; ++b)
            acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x4f32(f.a[a][j][s], f.w[b][j][s], acc[a][b], 0, 0, 0);
  };
  constexpr int KS = 16 * KC, STEP = KS * SK;
  const int kl = K - KS;                          // last chunk: loads past it re-read it, unused
  if (KS * sk < K) {
    Frag f0, f1;
    load(f0, KS * sk);
    for (int k = KS * sk; k < K; k += 2 * STEP) {
      load(f1, min(k + STEP, kl));
      mul(f0);
      if (k + STEP >= K) break;
      load(f0, min(k + 2 * STEP, kl));
      mul(f1);
    }
  }

  // accumulator register i of lane (c, g): row 4 g + i, column c of its block; the wave
  // partials of an element are added in wave order
  constexpr int E = (BM * BN + SK * 64 - 1) / (SK * 64);
  __shared__ float part[SK][BM * BN];
#pragma unroll
  for (int a = 0; a < TM; ++a)
#pragma unroll
    for (int b = 0; b < TN; ++b)
#pragma unroll
      for (int i = 0; i < 4; ++i) part[sk][(16 * a + 4 * g + i) * BN + 16 * b + c] = acc[a][b][i];
  float old[E];
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const int q = min(tid + e * SK * 64, BM * BN - 1);
    old[e] = epi.load(min(m0 + q / BN, M - 1), min(n0 + q % BN, N - 1));
  }
  __syncthreads();
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const int q = tid + e * SK * 64, m = m0 + q / BN, n = n0 + q % BN;
    if (q >= BM * BN) continue;
    float v = part[0][q];
#pragma unroll
    for (int w = 1; w < SK; ++w) v += part[w][q];
    if (m < M && n < N) epi.store(m, n, v, old[e]);
  }
}

// The larger shapes go through LDS: a 16-row fragment load of the kernel above touches 16 half
// cache lines, about 64 cycles of the address unit whatever the tile (2400 x 2304, K 768: 135 us
// at best), whereas LDS-DMA moves 8 rows x 128 bytes per instruction and every fragment is
// shared by the waves beside it (78 us).  k-steps of 32, two stages (three: 80 us, four: 87);
// 64 x 64 tile (128 x 64: 85 us, 128 x 128: 102 us, fewer tiles per compute unit); 16-byte
// pieces of a 128-byte row XOR-swizzled by row / 2 (conflict-free b128 reads).
__device__ inline void dma16(const void* base, uint32_t off, const void* dst) {
  const uint32_t lds = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(dst));
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1"
               :: "v"(off), "s"(base), "s"(lds) : "memory", "m0");
}
__device__ inline int swz(int row) { return (row >> 1) & 7; }

template <class Epi>
__global__ void __launch_bounds__(256) k_gemm_f32_lds(const float* __restrict__ A, int lda,
                                                      const float* __restrict__ W, int ldw, int M, int N,
                                                      int K, int tiles_n, int tiles, int per_xcd, Epi epi) {
  constexpr int TM = 2, TN = 2, WM = 2, NW = 4;          // 2 x 2 waves of 32 x 32
  constexpr int BM = 64, BN = 64;
  constexpr int AI = BM / 8 / NW, BI = BN / 8 / NW;      // DMA instructions per wave and k-step
  __shared__ uint4 lds[2][(BM + BN) * 8];
  const int t = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
  if (t >= tiles) return;
  const int m0 = t / tiles_n * BM, n0 = t % tiles_n * BN;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int c = lane & 15, g = lane >> 4;
  const int wm = wave % WM, wn = wave / WM;
  uint32_t offA[AI], offB[BI];                           // byte offsets; operands stay below 2^30 elements
#pragma unroll
  for (int i = 0; i < AI; ++i) {
    const int r = (wave * AI + i) * 8 + (lane >> 3), pc = (lane & 7) ^ swz(r);
    offA[i] = 4u * uint32_t(min(m0 + r, M - 1) * lda + 4 * pc);
  }
#pragma unroll
  for (int i = 0; i < BI; ++i) {
    const int r = (wave * BI + i) * 8 + (lane >> 3), pc = (lane & 7) ^ swz(r);
    offB[i] = 4u * uint32_t(min(n0 + r, N - 1) * ldw + 4 * pc);
  }
  auto fill = [&](int st, int kt) {
#pragma unroll
    for (int i = 0; i < AI; ++i) dma16(A + kt * 32, offA[i], &lds[st][(wave * AI + i) * 64]);
#pragma unroll
    for (int i = 0; i < BI; ++i) dma16(W + kt * 32, offB[i], &lds[st][BM * 8 + (wave * BI + i) * 64]);
  };
  f32x4 acc[TM][TN];
#pragma unroll
  for (int a = 0; a < TM; ++a)
#pragma unroll
    for (int b = 0; b < TN; ++b) acc[a][b] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int KT = K / 32;
  fill(0, 0);
  for (int kt = 0; kt < KT; ++kt) {
    // k-step kt has landed everywhere, and every wave is done with the other stage
    const int st = kt & 1;
    __builtin_amdgcn_s_waitcnt(0x0F70);                  // vmcnt(0)
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    if (kt + 1 < KT) fill(st ^ 1, kt + 1);
    const uint4* sa = lds[st];
    const uint4* sb = sa + BM * 8;
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      f32x4 fa[TM], fb[TN];
#pragma unroll
      for (int a = 0; a < TM; ++a) {
        const int r = 16 * (wm * TM + a) + c;
        fa[a] = __builtin_bit_cast(f32x4, sa[r * 8 + ((4 * j + g) ^ swz(r))]);
      }
#pragma unroll
      for (int b = 0; b < TN; ++b) {
        const int r = 16 * (wn * TN + b) + c;
        fb[b] = __builtin_bit_cast(f32x4, sb[r * 8 + ((4 * j + g) ^ swz(r))]);
      }
#pragma unroll
      for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int a = 0; a < TM; ++a)
#pragma unroll
          for (int b = 0; b < TN; ++b)
            acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x4f32(fa[a][s], fb[b][s], acc[a][b], 0, 0, 0);
    }
  }
  const int mw = m0 + wm * 16 * TM, nw = n0 + wn * 16 * TN;
  float old[TM][TN][4];
#pragma unroll
  for (int a = 0; a < TM; ++a)
#pragma unroll
    for (int b = 0; b < TN; ++b)
#pragma unroll
      for (int i = 0; i < 4; ++i)
        old[a][b][i] = epi.load(min(mw + 16 * a + 4 * g + i, M - 1), min(nw + 16 * b + c, N - 1));
#pragma unroll
  for (int a = 0; a < TM; ++a)
#pragma unroll
    for (int b = 0; b < TN; ++b)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int m = mw + 16 * a + 4 * g + i, n = nw + 16 * b + c;
        if (m < M && n < N) epi.store(m, n, acc[a][b][i], old[a][b][i]);
      }
}

template <class Epi>
Status launch_lds(const float* A, int lda, const float* W, int ldw, int M, int N, int K, const Epi& epi,
                  hipStream_t s) {
  const int tn = (N + 63) / 64, tiles = tn * ((M + 63) / 64), per = (tiles + 7) / 8;
  hipLaunchKernelGGL((k_gemm_f32_lds<Epi>), dim3(8 * per), dim3(256), 0, s, A, lda, W, ldw, M, N, K, tn,
                     tiles, per, epi);
  DC_HIP(hipGetLastError());
  return Status::ok();
}

template <int TM, int TN, int SK, int KC, class Epi, class WT>
Status launch(const float* A, int lda, const WT* W, int ldw, int M, int N, int K, const Epi& epi,
              hipStream_t s) {
  constexpr int BM = 16 * TM, BN = 16 * TN;
  const int tn = (N + BN - 1) / BN, tiles = tn * ((M + BM - 1) / BM), per = (tiles + 7) / 8;
  hipLaunchKernelGGL((k_gemm_f32<TM, TN, SK, KC, Epi, WT>), dim3(8 * per), dim3(SK * 64), 0, s, A, lda, W,
                     ldw, M, N, K, tn, tiles, per, epi);
  DC_HIP(hipGetLastError());
  return Status::ok();
}

// Which tile (256 compute units, us; the direct kernel's tiles are 32 x 16 and 32 x 32 with four
// waves on K, 64 x 48 with eight):
//  - through LDS from about 3/4 of a round of 64 x 64 tiles: 640 x 1536, K 512 (240 tiles) 14.2,
//    32 x 32 18.6; 1000 x 512, K 2048 (128 tiles) 42.3, 32 x 32 34.3;
//  - 64 x 48 for 33 to 128 rows and many columns: every weight read once or twice and three
//    products per load of A (50 x 11520, K 1920, back to back: 33.5, 32 x 16 62, LDS 40; 50 x 1920
//    (40 tiles): 33.4, 32 x 16 12.9);
//  - 32 x 16 while its tiles fit one round (272 x 256, K 1024: 7.5, 32 x 32 10.0), else 32 x 32
//    (544 x 256, K 1024: 10.1, 32 x 16 12.7).
// bf16 weights (calibration only) take the direct tiles.
template <class Epi, class WT>
Status gemm(const float* A, int lda, const WT* W, int ldw, int M, int N, int K, const Epi& epi,
            hipStream_t s) {
  if (M <= 0 || N <= 0) return Status::ok();
  if (K % 64 || lda % 4 || ldw % 4) return Status::shape("f32 GEMM needs K % 64 == 0, aligned rows");
  const int64_t cus = compute_units();
  if (cus <= 0) return Status::make(DC_ERR_HIP, "f32 GEMM: no device");
  auto tiles = [&](int bm, int bn) { return int64_t((M + bm - 1) / bm) * ((N + bn - 1) / bn); };
  if (M > 32 && M <= 128 && 2 * tiles(64, 48) >= cus) return launch<4, 3, 8, 1>(A, lda, W, ldw, M, N, K, epi, s);
  if constexpr (sizeof(WT) == 4) {
    // its byte offsets are 32 bits wide
    const bool fits = int64_t(M) * lda < (1 << 30) && int64_t(N) * ldw < (1 << 30);
    if (fits && 4 * tiles(64, 64) >= 3 * cus) return launch_lds(A, lda, W, ldw, M, N, K, epi, s);
  }
  if (tiles(32, 16) <= cus) return launch<2, 1, 4, 4>(A, lda, W, ldw, M, N, K, epi, s);
  return launch<2, 2, 4, 2>(A, lda, W, ldw, M, N, K, epi, s);
}

}  // namespace

Status gemm_f32_bias_act(const float* A, int lda, const float* W, int ldw, const float* bias,
                         float* out, int ldo, int M, int N, int K, Act act, hipStream_t s) {
  return gemm(A, lda, W, ldw, M, N, K, EpiBiasAct{bias, out, ldo, act == Act::kSilu ? 1 : 0}, s);
}

Status gemm_f32_bias_and_silu(const float* A, int lda, const float* W, int ldw, const float* bias,
                              float* out, float* silu_out, int ldo, int M, int N, int K, hipStream_t s) {
  return gemm(A, lda, W, ldw, M, N, K, EpiBiasAndSilu{bias, out, silu_out, ldo}, s);
}

Status gemm_f32_gate_residual(const float* A, int lda, const float* W, int ldw, const float* bias,
                              const float* gate, float* h, int ldh, int M, int N, int K,
                              hipStream_t s) {
  return gemm(A, lda, W, ldw, M, N, K, EpiGateResidual{bias, gate, h, ldh}, s);
}

Status gemm_f32_rows(const float* A, int lda, const void* W, bool w_bf16, int ldw, const float* bias,
                     int bias_rows, float* out, int ldo, int M, int N, int K, hipStream_t s) {
  const EpiBiasRows e{bias, out, ldo, bias_rows};
  if (w_bf16) return gemm(A, lda, static_cast<const uint16_t*>(W), ldw, M, N, K, e, s);
  return gemm(A, lda, static_cast<const float*>(W), ldw, M, N, K, e, s);
}

Status gemm_f32_gate_residual_rows(const float* A, int lda, const void* W, bool w_bf16, int ldw,
                                   const float* bias, int bias_rows, const float* gate, float* h, int ldh,
                                   int M, int N, int K, hipStream_t s) {
  const EpiGateResidualRows e{bias, gate, h, ldh, bias_rows};
  if (w_bf16) return gemm(A, lda, static_cast<const uint16_t*>(W), ldw, M, N, K, e, s);
  return gemm(A, lda, static_cast<const float*>(W), ldw, M, N, K, e, s);
}

Status gemm_f32_head_tangents(const float* A, const void* W, bool w_bf16, float* x, float dsigma,
                              const Geo& g, int n, hipStream_t s) {
  if (g.Nv <= 0) return Status::ok();           // no latent to move (its rows are all text)
  const EpiHeadTangents e{{nullptr, x, dsigma, g.T, g.Hl, g.Wl, g.p, g.Hp, g.Wp}, g.N, g.Nv,
                          size_t(g.C) * g.T * g.Hl * g.Wl};
  if (w_bf16) return gemm(A, g.d, static_cast<const uint16_t*>(W), g.d, n * g.N, g.P, g.d, e, s);
  return gemm(A, g.d, static_cast<const float*>(W), g.d, n * g.N, g.P, g.d, e, s);
}

Status gemm_f32_gelu(const float* A, int lda, const float* W, int ldw, const float* bias, float* out,
                     int ldo, int M, int N, int K, hipStream_t s) {
  return gemm(A, lda, W, ldw, M, N, K, EpiGelu{bias, out, ldo}, s);
}

Status gemm_f32_head(const float* A, int lda, const float* W, const float* bias, float* x,
                     float dsigma, const Geo& g, int M, hipStream_t s) {
  return gemm(A, lda, W, g.d, M, g.P, g.d, EpiHeadEuler{bias, x, dsigma, g.T, g.Hl, g.Wl, g.p, g.Hp, g.Wp}, s);
}

}  // namespace dc
