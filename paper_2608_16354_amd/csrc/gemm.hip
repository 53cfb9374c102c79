// bf16 GEMMs of the denoising step: C = A W^T with fused epilogues.
//
// bf16 block GEMMs (QKV, out-projection, MLP up / down): v_mfma_f32_32x32x16_bf16, tiles
// fed global -> LDS by LDS-DMA, XOR-swizzled 128-byte rows, k-steps of 64, one barrier per
// k-step, XCD-aware tile order; epilogues take one accumulator column at a time.  Six tile
// shapes, chosen per call by a cost model (block_gemm): long sequences take 384 x 192 or 320 x 256
// (fewest operand lines per FLOP, the L1 miss queue being the limit there), short ones the
// smaller tiles that spread over all compute units.
// (fp32 GEMMs: gemm_f32.hip; bf16 patch embedding: patch_embed.hip.)
#include <hip/hip_runtime.h>

#include <cmath>

#include "internal.h"

namespace dc {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4n __attribute__((ext_vector_type(4)));

// 16-byte streaming stores for the block GEMM epilogues: every CU finishes its tile at
// about the same time, and the output (not reused by the GEMM) then does not displace
// the operand lines the next tiles read from L2 (-1 to -4 % per GEMM on MI355X)
__device__ inline void store_nt(void* p, uint4 v) {
  __builtin_nontemporal_store(__builtin_bit_cast(u32x4, v), reinterpret_cast<u32x4*>(p));
}
__device__ inline void store_nt(float* p, float4 v) {
  __builtin_nontemporal_store(__builtin_bit_cast(f32x4n, v), reinterpret_cast<f32x4n*>(p));
}
typedef float f32x16 __attribute__((ext_vector_type(16)));

__device__ inline uint16_t to_bf16(float f) {
  return __builtin_bit_cast(uint16_t, static_cast<__bf16>(f));
}
__device__ inline float from_bf16(uint16_t u) { return __uint_as_float(uint32_t(u) << 16); }
inline bool al16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; }

// LDS chunk swizzle for 128-byte tile rows.  gfx950's LDS serves 256 bytes per
// cycle (64 banks), so two consecutive 128-byte rows share a bank cycle: keying
// the XOR on row / 2 makes the 16 rows read by 16 consecutive lanes hit 16
// distinct 16-byte bank groups.
__device__ inline int swz(int row) { return (row >> 1) & 7; }

// GELU with the tanh approximation, written as z * sigmoid(2y), y = sqrt(2/pi)(z + 0.044715 z^3)
// (0.5 (1 + tanh y) = 1 / (1 + exp(-2y))).
__device__ inline float gelu_tanh(float z) {
  const float y = 0.7978845608028654f * (z + 0.044715f * z * z * z);
  return z / (1.0f + __expf(-2.0f * y));
}
// the same with v_rcp_f32 (1 ulp) in place of the IEEE division, for bf16 outputs
__device__ inline float gelu_tanh_fast(float z) {
  const float y = 0.7978845608028654f * (z + 0.044715f * z * z * z);
  return z * __builtin_amdgcn_rcpf(1.0f + __expf(-2.0f * y));
}

// ---------------------------------------------------------------------------
// epilogues
// ---------------------------------------------------------------------------
// The MFMA GEMM hands its epilogue either one accumulator column at a time: col(mb,
// n, M, v) gets v[i] = C[mb + 8 (i / 4) + i % 4][n] for i < 16 (mb a multiple of 4),
// or, when the epilogue declares kRowVec = V > 0, V consecutive columns of NP rows:
// rows<NP>(m0, dm, n, M, v) gets v[k][j] = C[m0 + k dm][n + j] (n a multiple of V), so
// it can issue all of its loads before any store; the GEMM transposes
// each 32 x 32 accumulator tile through LDS for that, so the stores are 16 bytes
// per lane instead of one element.  isrow(n) says whether the 32-column tile that
// starts at n goes the row way (otherwise col).
// Q (columns < d) leaves pre-multiplied by qscale = log2(e)/sqrt(d_h): the bf16
// attention kernel takes its scores in log2 units.
struct EpiQKVBf16 {
  const float* bias; uint16_t* qk; uint16_t* vt; int d; int ldv; float qscale;
  static constexpr int kRowVec = 8;
  __device__ bool isrow(int n) const { return n < 2 * d; }    // Q and K rows; V^T by column
  bool rows_aligned() const { return al16(qk) && al16(bias) && d % 4 == 0; }
  template <int NP>
  __device__ void rows(int m0, int dm, int n, int M, const float (&v)[NP][8]) const {
    const float4 b0 = *reinterpret_cast<const float4*>(bias + n);
    const float4 b1 = *reinterpret_cast<const float4*>(bias + n + 4);
    const float sc = n < d ? qscale : 1.0f;
#pragma unroll
    for (int k = 0; k < NP; ++k) {
      uint4 pk;
      pk.x = uint32_t(to_bf16((v[k][0] + b0.x) * sc)) | (uint32_t(to_bf16((v[k][1] + b0.y) * sc)) << 16);
      pk.y = uint32_t(to_bf16((v[k][2] + b0.z) * sc)) | (uint32_t(to_bf16((v[k][3] + b0.w) * sc)) << 16);
      pk.z = uint32_t(to_bf16((v[k][4] + b1.x) * sc)) | (uint32_t(to_bf16((v[k][5] + b1.y) * sc)) << 16);
      pk.w = uint32_t(to_bf16((v[k][6] + b1.z) * sc)) | (uint32_t(to_bf16((v[k][7] + b1.w) * sc)) << 16);
      if (m0 + k * dm < M) store_nt(qk + size_t(m0 + k * dm) * 2 * d + n, pk);
    }
  }
  __device__ void col(int mb, int n, int M, const f32x16& v) const {
    const float b = bias[n];
    if (n < 2 * d) {
      const float sc = n < d ? qscale : 1.0f;
      uint16_t* __restrict__ q = qk + size_t(mb) * 2 * d + n;
      if (mb + 28 <= M) {                     // all 16 rows present: no per-row guards
#pragma unroll
        for (int i = 0; i < 16; ++i) q[size_t(8 * (i >> 2) + (i & 3)) * 2 * d] = to_bf16((v[i] + b) * sc);
      } else {
#pragma unroll
        for (int i = 0; i < 16; ++i)
          if (mb + 8 * (i >> 2) + (i & 3) < M) q[size_t(8 * (i >> 2) + (i & 3)) * 2 * d] = to_bf16((v[i] + b) * sc);
      }
    } else {
      // V^T row n - 2d: four consecutive tokens per 8-byte store (ldv and mb are multiples of 4).
      // The padding tokens [M, ldv) get zeros: the attention's last value tile reads them
      // (and multiplies them by zero probabilities, which NaN garbage would turn into NaN).
      // The last row tile always reaches ldv (tile heights are multiples of 64).
      uint16_t* __restrict__ r = vt + size_t(n - 2 * d) * ldv + mb;
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        uint2 pk;
        pk.x = uint32_t(to_bf16(v[4 * g] + b)) | (uint32_t(to_bf16(v[4 * g + 1] + b)) << 16);
        pk.y = uint32_t(to_bf16(v[4 * g + 2] + b)) | (uint32_t(to_bf16(v[4 * g + 3] + b)) << 16);
        if (mb + 8 * g + 3 < M) {
          *reinterpret_cast<uint2*>(r + 8 * g) = pk;
        } else {
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            const int m = mb + 8 * g + j;
            if (m < M) r[8 * g + j] = to_bf16(v[4 * g + j] + b);
            else if (m < ldv) r[8 * g + j] = 0;
          }
        }
      }
    }
  }
};
struct EpiGateResidual {
  const float* bias; const float* gate; float* h; int ldh;
  static constexpr int kRowVec = 4;
  __device__ bool isrow(int) const { return true; }
  bool rows_aligned() const { return al16(h) && al16(bias) && al16(gate) && ldh % 4 == 0; }
  // rows m0 + k * dm (k < NP), columns n .. n + 3: all loads of h, then all stores
  template <int NP>
  __device__ void rows(int m0, int dm, int n, int M, const float (&v)[NP][4]) const {
    const float4 g = *reinterpret_cast<const float4*>(gate + n);
    const float4 b = *reinterpret_cast<const float4*>(bias + n);
    float4 o[NP];
#pragma unroll
    for (int k = 0; k < NP; ++k)
      o[k] = *reinterpret_cast<const float4*>(h + size_t(min(m0 + k * dm, M - 1)) * ldh + n);
#pragma unroll
    for (int k = 0; k < NP; ++k) {
      o[k].x += g.x * (v[k][0] + b.x);
      o[k].y += g.y * (v[k][1] + b.y);
      o[k].z += g.z * (v[k][2] + b.z);
      o[k].w += g.w * (v[k][3] + b.w);
      if (m0 + k * dm < M) store_nt(h + size_t(m0 + k * dm) * ldh + n, o[k]);
    }
  }
  __device__ void col(int mb, int n, int M, const f32x16& v) const {
    const float g = gate[n], b = bias[n];
    float* __restrict__ p = h + size_t(mb) * ldh + n;
    if (mb + 28 <= M) {                       // all 16 rows present: batched loads, no guards
      float old[16];
#pragma unroll
      for (int i = 0; i < 16; ++i) old[i] = p[size_t(8 * (i >> 2) + (i & 3)) * ldh];
#pragma unroll
      for (int i = 0; i < 16; ++i) p[size_t(8 * (i >> 2) + (i & 3)) * ldh] = old[i] + g * (v[i] + b);
      return;
    }
    float old[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const int r = min(mb + 8 * (i >> 2) + (i & 3), M - 1) - mb;   // clamped: in bounds
      old[i] = p[size_t(r) * ldh];
    }
#pragma unroll
    for (int i = 0; i < 16; ++i)
      if (mb + 8 * (i >> 2) + (i & 3) < M) p[size_t(8 * (i >> 2) + (i & 3)) * ldh] = old[i] + g * (v[i] + b);
  }
};
struct EpiGeluBf16 {
  const float* bias; uint16_t* out; int ldo;
  static constexpr int kRowVec = 8;
  __device__ bool isrow(int) const { return true; }
  bool rows_aligned() const { return al16(out) && al16(bias) && ldo % 8 == 0; }
  template <int NP>
  __device__ void rows(int m0, int dm, int n, int M, const float (&v)[NP][8]) const {
    const float4 b0 = *reinterpret_cast<const float4*>(bias + n);
    const float4 b1 = *reinterpret_cast<const float4*>(bias + n + 4);
    const float bb[8] = {b0.x, b0.y, b0.z, b0.w, b1.x, b1.y, b1.z, b1.w};
#pragma unroll
    for (int k = 0; k < NP; ++k) {
      uint32_t w[4];
#pragma unroll
      for (int j = 0; j < 4; ++j)
        w[j] = uint32_t(to_bf16(gelu_tanh_fast(v[k][2 * j] + bb[2 * j]))) |
               (uint32_t(to_bf16(gelu_tanh_fast(v[k][2 * j + 1] + bb[2 * j + 1]))) << 16);
      if (m0 + k * dm < M) store_nt(out + size_t(m0 + k * dm) * ldo + n, make_uint4(w[0], w[1], w[2], w[3]));
    }
  }
  __device__ void col(int mb, int n, int M, const f32x16& v) const {
    const float b = bias[n];
    uint16_t* __restrict__ o = out + size_t(mb) * ldo + n;
    if (mb + 28 <= M) {
#pragma unroll
      for (int i = 0; i < 16; ++i) o[size_t(8 * (i >> 2) + (i & 3)) * ldo] = to_bf16(gelu_tanh(v[i] + b));
    } else {
#pragma unroll
      for (int i = 0; i < 16; ++i)
        if (mb + 8 * (i >> 2) + (i & 3) < M) o[size_t(8 * (i >> 2) + (i & 3)) * ldo] = to_bf16(gelu_tanh(v[i] + b));
    }
  }
};

// ---------------------------------------------------------------------------
// bf16 MFMA GEMM, LDS-DMA pipeline.  WM x WN waves, block tile BM x BN x 64.  Tiles go global -> LDS with global_load_lds_dwordx4 (lane i
// of an instruction lands at LDS base + 16 i, so the XOR swizzle is applied to the
// global address each lane fetches): no staging registers and no LDS write
// instructions.  ST stages, one barrier per k-step: the loads for step k + ST - 1 are
// issued among the MFMAs of the first DS 16-wide k-slices of step k (the block
// GEMMs use DS = 2, so with two stages the last refill has half a step to land).  Rows past M or N
// are clamped to the last row (their results are never stored).  Workgroups are
// renumbered so that each XCD (assigned round-robin by workgroup id) processes a
// contiguous range of tiles.
// ---------------------------------------------------------------------------
typedef __attribute__((address_space(3))) void lds_void;
// 16 bytes per lane global -> LDS (global_load_lds_dwordx4): lane i reads
// base + off (wave-uniform 64-bit base in SGPRs, per-lane 32-bit byte offset) and
// its bytes land at the wave-uniform LDS address dst + 16 i.  Issued as inline
// assembly so that the compiler neither makes LDS reads of the other stage wait
// for it nor reorders it; the kernel waits for its own fills (vmcnt) before each
// barrier.
__device__ inline void dma16(const void* base, uint32_t off, const void* dst) {
  const uint32_t lds = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(dst));
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1"
               :: "v"(off), "s"(base), "s"(lds) : "memory", "m0");
}

// s_waitcnt vmcnt(N) with the other counters left alone (gfx9 encoding: vmcnt bits
// [3:0] and [15:14], expcnt [6:4], lgkmcnt [11:8])
template <int N>
__device__ inline void wait_vmcnt() {
  static_assert(N >= 0 && N < 64, "vmcnt range");
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | 0x0F70);
}
constexpr int kEpiStride = 40;   // floats per row of the epilogue's per-wave LDS transpose buffer

// Epilogue of the bf16 block GEMMs.  Row-vector epilogues: each 32 x 32
// accumulator tile goes through a per-wave LDS buffer (rows of 40 floats: the two
// row groups a ds_write_b32 covers land 32 banks apart) and comes back as V
// consecutive columns of one row per lane.  The caller has finished every read of
// the LDS stages (the barrier here orders the reuse).
template <int BM, int BN, int WM, int WN, class Epi, int TM, int TN>
__device__ inline void gemm_epilogue(f32x16 (&acc)[TM][TN], uint4* lds, int m0, int n0, int M,
                                     int N, int wave, int lane, int rows_ok, const Epi& epi) {
  constexpr int WTM = BM / WM, WTN = BN / WN;
  constexpr int RV = Epi::kRowVec > 0 ? Epi::kRowVec : 4;
  constexpr int kS = kEpiStride;
  const int wm = wave % WM, wn = wave / WM;
  const int r32 = lane & 31, hi = lane >> 5;
  if constexpr (Epi::kRowVec > 0) {
    __builtin_amdgcn_s_barrier();              // every wave is done with the last stage
    asm volatile("" ::: "memory");
  }
  float* const st = reinterpret_cast<float*>(lds) + wave * 32 * kS;
#pragma unroll
  for (int b = 0; b < TN; ++b) {
    const int nb = n0 + wn * WTN + b * 32;     // first column of the tile
    if (nb >= N) continue;
    if (Epi::kRowVec > 0 && rows_ok && nb + 32 <= N && epi.isrow(nb)) {
#pragma unroll
      for (int a = 0; a < TM; ++a) {
        const int mb = m0 + wm * WTM + a * 32;
#pragma unroll
        for (int i = 0; i < 16; ++i) st[(8 * (i >> 2) + 4 * hi + (i & 3)) * kS + r32] = acc[a][b][i];
        constexpr int LPR = 32 / RV, RPI = 64 / LPR, NP = 32 / RPI;   // lanes per row, rows per pass
        const int r0 = lane / LPR, c = (lane % LPR) * RV;
        float v[NP][RV];
#pragma unroll
        for (int k = 0; k < NP; ++k)
#pragma unroll
          for (int q = 0; q < RV; q += 4) {
            const float4 t = *reinterpret_cast<const float4*>(st + (k * RPI + r0) * kS + c + q);
            v[k][q] = t.x; v[k][q + 1] = t.y; v[k][q + 2] = t.z; v[k][q + 3] = t.w;
          }
        epi.template rows<NP>(mb + r0, RPI, nb + c, M, v);
      }
    } else {
#pragma unroll
      for (int a = 0; a < TM; ++a)
        if (nb + r32 < N) epi.col(m0 + wm * WTM + a * 32 + 4 * hi, nb + r32, M, acc[a][b]);
    }
  }
}

template <int BM, int BN, int WM, int WN, int DS, int ST, class Epi>
__global__ void __launch_bounds__(WM * WN * 64) k_gemm_dma(const uint16_t* __restrict__ A, int lda,
                                                  const uint16_t* __restrict__ W, int ldw, int M,
                                                  int N, int K, int tiles_n, int tiles, int per_xcd,
                                                  int rows_ok, Epi epi) {
  constexpr int BK = 64;
  constexpr int NW = WM * WN;
  constexpr int WTM = BM / WM, WTN = BN / WN;
  constexpr int TM = WTM / 32, TN = WTN / 32;
  constexpr int AI = BM * 8 / 64 / NW, BI = BN * 8 / 64 / NW;   // DMA instructions per wave
  static_assert(TM >= 1 && TN >= 1 && AI * NW * 64 == BM * 8 && BI * NW * 64 == BN * 8,
                "tile shape");
  // one array, so every stage address is a constant offset from one base
  constexpr int STAGE = (BM + BN) * 8;
  __shared__ uint4 lds[ST * STAGE];

  const int t = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
  if (t >= tiles) return;
  // groups of four row tiles: consecutive tiles (the ones an XCD runs together)
  // walk down a group before moving right, so their A and W k-slices share L2
  const int tiles_m = (M + BM - 1) / BM;
  const int grp = t / (4 * tiles_n), gbase = grp * 4;
  const int gsz = min(4, tiles_m - gbase);
  const int tin = t - grp * 4 * tiles_n;
  const int m0 = (gbase + tin % gsz) * BM, n0 = (tin / gsz) * BN;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // uniform: DMA addresses in SGPRs
  const int wm = wave % WM, wn = wave / WM;

  // per-lane global byte offsets of this wave's DMA instructions (k-step 0); the
  // operands stay below 2^31 elements, so the byte offsets fit 32 bits
  uint32_t offA[AI], offB[BI];
#pragma unroll
  for (int i = 0; i < AI; ++i) {
    const int slot = (wave * AI + i) * 64 + lane;
    const int r = slot >> 3, c = (slot & 7) ^ swz(slot >> 3);
    offA[i] = 2u * uint32_t(min(m0 + r, M - 1) * lda + 8 * c);
  }
#pragma unroll
  for (int i = 0; i < BI; ++i) {
    const int slot = (wave * BI + i) * 64 + lane;
    const int r = slot >> 3, c = (slot & 7) ^ swz(slot >> 3);
    offB[i] = 2u * uint32_t(min(n0 + r, N - 1) * ldw + 8 * c);
  }
  f32x16 acc[TM][TN];
#pragma unroll
  for (int a = 0; a < TM; ++a)
#pragma unroll
    for (int b = 0; b < TN; ++b)
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[a][b][i] = 0.f;

  const int KT = K / BK;                         // even: the launcher requires K % 128 == 0

  const int r32 = lane & 31, hi = lane >> 5;
  // one DMA instruction (j < AI + BI) of the refill of stage `to` with k-step kt;
  // compute() spreads the refill over its first DS k-slices
  auto dma_one = [&](uint4* to, int kt, int j) {
    const int k0 = kt * BK;
    if (j < AI) dma16(A + k0, offA[j], to + (wave * AI + j) * 64);
    else dma16(W + k0, offB[j - AI], to + BM * 8 + (wave * BI + (j - AI)) * 64);
  };
  auto compute = [&](const uint4* sa, uint4* to, int kt) {
    const uint4* sb = sa + BM * 8;
#pragma unroll
    for (int kk = 0; kk < BK / 16; ++kk) {
      if (kt >= 0) {
        // the refill goes out over the first DS k-slices, DPS instructions per slice
        constexpr int DPS = (AI + BI + DS - 1) / DS;
#pragma unroll
        for (int j = kk * DPS; j < (kk + 1) * DPS; ++j)
          if (j < AI + BI && kk < DS) dma_one(to, kt, j);
      }
      const int ch = kk * 2 + hi;
      bf16x8 af[TM], bf[TN];
#pragma unroll
      for (int a = 0; a < TM; ++a) {
        const int r = wm * WTM + a * 32 + r32;
        af[a] = __builtin_bit_cast(bf16x8, sa[r * 8 + (ch ^ swz(r))]);
      }
#pragma unroll
      for (int b = 0; b < TN; ++b) {
        const int r = wn * WTN + b * 32 + r32;
        bf[b] = __builtin_bit_cast(bf16x8, sb[r * 8 + (ch ^ swz(r))]);
      }
#pragma unroll
      for (int a = 0; a < TM; ++a)
#pragma unroll
        for (int b = 0; b < TN; ++b)
          acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[a], bf[b], acc[a][b], 0, 0, 0);
    }
  };

#pragma unroll
  for (int i = 0; i < ST - 1; ++i)
    if (i < KT)
#pragma unroll
      for (int j = 0; j < AI + BI; ++j) dma_one(lds + i * STAGE, i, j);
  for (int kt0 = 0; kt0 < KT; kt0 += ST) {
#pragma unroll
    for (int i = 0; i < ST; ++i) {
      const int kt = kt0 + i;
      if (kt >= KT) break;
      // before the barrier: this wave's part of k-step kt has landed (the ST - 2 steps after
      // it may still be in flight)
      if (ST > 2 && kt + ST - 2 < KT) wait_vmcnt<(ST - 2) * (AI + BI)>();
      else wait_vmcnt<0>();
      __builtin_amdgcn_s_barrier();
      asm volatile("" ::: "memory");
      compute(lds + i * STAGE, lds + (i + ST - 1) % ST * STAGE, kt + ST - 1 < KT ? kt + ST - 1 : -1);
    }
  }

  static_assert(Epi::kRowVec == 0 || sizeof(lds) >= NW * 32 * kEpiStride * sizeof(float), "epilogue LDS");
  gemm_epilogue<BM, BN, WM, WN>(acc, lds, m0, n0, M, N, wave, lane, rows_ok, epi);
}

// 128 x 128 tile for the middle sizes (8 waves of 64 x 32).  A tile this small has little
// MFMA work per k-step (512 cycles), so the LDS latency after each barrier shows: here the
// fragments of the next k-slice, across the barrier too, are read while this slice
// multiplies.  For that a k-step has to have landed one barrier before it is multiplied,
// hence four stages of 32 KB.  120 k-steps on 195 tiles: 53.8 us, 60.0 with k_gemm_dma (the
// fill of 32 KB per k-step and compute unit is the rest: about 38 of 64 bytes per cycle).
template <class Epi>
__global__ void __launch_bounds__(512) k_gemm_pipe(const uint16_t* __restrict__ A, int lda,
                                                   const uint16_t* __restrict__ W, int ldw, int M,
                                                   int N, int K, int tiles_n, int tiles, int per_xcd,
                                                   int rows_ok, Epi epi) {
  constexpr int BM = 128, BN = 128, WM = 2, WN = 4, ST = 4, BK = 64, NW = WM * WN;
  constexpr int WTM = BM / WM, WTN = BN / WN, TM = WTM / 32, TN = WTN / 32;
  constexpr int AI = BM * 8 / 64 / NW, BI = BN * 8 / 64 / NW;     // DMA instructions per wave
  static_assert(AI + BI == 4, "one DMA instruction per k-slice");
  constexpr int STAGE = (BM + BN) * 8;
  __shared__ uint4 lds[ST * STAGE];
  const int t = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
  if (t >= tiles) return;
  const int tiles_m = (M + BM - 1) / BM;
  const int grp = t / (4 * tiles_n), gbase = grp * 4;
  const int gsz = min(4, tiles_m - gbase);
  const int tin = t - grp * 4 * tiles_n;
  const int m0 = (gbase + tin % gsz) * BM, n0 = (tin / gsz) * BN;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave % WM, wn = wave / WM;
  const int r32 = lane & 31, hi = lane >> 5;
  uint32_t off[AI + BI];                         // byte offsets, as in k_gemm_dma: A, then W
#pragma unroll
  for (int i = 0; i < AI; ++i) {
    const int slot = (wave * AI + i) * 64 + lane, r = slot >> 3, c = (slot & 7) ^ swz(r);
    off[i] = 2u * uint32_t(min(m0 + r, M - 1) * lda + 8 * c);
  }
#pragma unroll
  for (int i = 0; i < BI; ++i) {
    const int slot = (wave * BI + i) * 64 + lane, r = slot >> 3, c = (slot & 7) ^ swz(r);
    off[AI + i] = 2u * uint32_t(min(n0 + r, N - 1) * ldw + 8 * c);
  }
  auto dma_one = [&](int st, int kt, int j) {
    uint4* to = lds + st * STAGE;
    if (j < AI) dma16(A + kt * BK, off[j], to + (wave * AI + j) * 64);
    else dma16(W + kt * BK, off[j], to + BM * 8 + (wave * BI + (j - AI)) * 64);
  };
  struct Frag { bf16x8 a[TM], b[TN]; };
  auto read = [&](Frag& f, const uint4* s, int kk) {
    const int ch = 2 * kk + hi;
#pragma unroll
    for (int a = 0; a < TM; ++a) {
      const int r = wm * WTM + a * 32 + r32;
      f.a[a] = __builtin_bit_cast(bf16x8, s[r * 8 + (ch ^ swz(r))]);
    }
#pragma unroll
    for (int b = 0; b < TN; ++b) {
      const int r = wn * WTN + b * 32 + r32;
      f.b[b] = __builtin_bit_cast(bf16x8, s[BM * 8 + r * 8 + (ch ^ swz(r))]);
    }
  };
  f32x16 acc[TM][TN];
#pragma unroll
  for (int a = 0; a < TM; ++a)
#pragma unroll
    for (int b = 0; b < TN; ++b)
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[a][b][i] = 0.f;

  const int KT = K / BK;
#pragma unroll
  for (int i = 0; i < ST - 1; ++i)
    if (i < KT)
#pragma unroll
      for (int j = 0; j < AI + BI; ++j) dma_one(i, i, j);
  if (KT >= ST - 1) wait_vmcnt<(ST - 2) * (AI + BI)>();          // k-step 0 has landed
  else wait_vmcnt<0>();
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
  Frag f[2];
  read(f[0], lds, 0);
  for (int kt0 = 0; kt0 < KT; kt0 += ST) {
#pragma unroll
    for (int i = 0; i < ST; ++i) {
      const int kt = kt0 + i;
      if (kt >= KT) break;
      // k-step kt + 1 has landed in every wave's view, and every wave's reads of k-step
      // kt - 1 have returned: its stage takes k-step kt + ST - 1
      if (kt + ST - 2 < KT) __builtin_amdgcn_s_waitcnt(0x0070 | (AI + BI));   // vmcnt(4) lgkmcnt(0)
      else __builtin_amdgcn_s_waitcnt(0x0070);
      __builtin_amdgcn_s_barrier();
      asm volatile("" ::: "memory");
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) {
        if (kk < 3) read(f[(kk + 1) & 1], lds + i * STAGE, kk + 1);
        else read(f[0], lds + (i + 1) % ST * STAGE, 0);          // past the last k-step: unused
        if (kt + ST - 1 < KT) dma_one((i + ST - 1) % ST, kt + ST - 1, kk);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int a = 0; a < TM; ++a)
#pragma unroll
          for (int b = 0; b < TN; ++b)
            acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f[kk & 1].a[a], f[kk & 1].b[b], acc[a][b], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  }
  __builtin_amdgcn_s_waitcnt(0x0070);            // the reads ahead are done: the epilogue reuses LDS
  static_assert(sizeof(lds) >= NW * 32 * kEpiStride * sizeof(float), "epilogue LDS");
  gemm_epilogue<BM, BN, WM, WN>(acc, lds, m0, n0, M, N, wave, lane, rows_ok, epi);
}

inline Status check_gemm(int lda, int ldw, int M, int N, int K) {
  if (K % 128 || lda % 8 || ldw % 8) return Status::shape("bf16 GEMM needs K % 128 == 0 and 16-byte rows");
  if (int64_t(M) * lda > INT32_MAX || int64_t(N) * ldw > INT32_MAX)
    return Status::shape("bf16 GEMM operand exceeds 2^31 elements");
  return Status::ok();
}

template <int BM, int BN, int WM, int WN, int DS, int ST, class Epi>
Status launch_dma(const uint16_t* A, int lda, const uint16_t* W, int ldw, int M, int N, int K,
                  const Epi& epi, hipStream_t s) {
  const int tn = (N + BN - 1) / BN, tm = (M + BM - 1) / BM;
  const int tiles = tn * tm;
  const int per = (tiles + 7) / 8;
  // row-vector epilogue stores need 16-byte aligned rows; otherwise every tile goes by column
  const int rows_ok = epi.rows_aligned() ? 1 : 0;
  hipLaunchKernelGGL((k_gemm_dma<BM, BN, WM, WN, DS, ST, Epi>), dim3(8 * per), dim3(WM * WN * 64), 0, s, A, lda,
                     W, ldw, M, N, K, tn, tiles, per, rows_ok, epi);
  DC_HIP(hipGetLastError());
  return Status::ok();
}

template <class Epi>
Status launch_pipe(const uint16_t* A, int lda, const uint16_t* W, int ldw, int M, int N, int K,
                   const Epi& epi, hipStream_t s) {
  const int tn = (N + 127) / 128, tiles = tn * ((M + 127) / 128), per = (tiles + 7) / 8;
  hipLaunchKernelGGL((k_gemm_pipe<Epi>), dim3(8 * per), dim3(512), 0, s, A, lda, W, ldw, M, N, K, tn, tiles,
                     per, epi.rows_aligned() ? 1 : 0, epi);
  DC_HIP(hipGetLastError());
  return Status::ok();
}

// Cost of a block GEMM in us with tile i: rounds of one workgroup per compute unit, each
// `fixed` (launch, first fill, epilogue) plus K / 64 k-steps of `alone` (a nearly empty chip) to
// `full` (every compute unit fetching operands).  The 64 x 64 tile runs up to three
// workgroups per compute unit, a k-step taking c[n - 1] with n of them.  Fitted to timings of
// all six tiles on 80 shapes (M 300 to 17,776; d 512, 1,152, 1,920, 3,072; QKV, out, up, down)
// on MI355X: the tile it picks is 0.04 % slower than the best one on average, 6 % at worst.
// Examples (us, the earlier fixed choice of 384 x 192 / 320 x 256 -> now): out 1,556 x 1,920 52 -> 18,
// down 162 -> 54; down 3,704 x 1,152 102 -> 57; up 300 x 7,680 54 -> 17; 17,776 tokens unchanged.
struct TileCost { int bm, bn; float alone, full, fixed; };
constexpr TileCost kTiles[] = {{384, 192, 1.168f, 1.706f, 11.2f}, {320, 256, 1.295f, 1.792f, 12.9f},
                               {256, 192, 0.849f, 1.204f, 7.6f},  {256, 128, 0.666f, 0.982f, 5.0f},
                               {128, 128, 0.341f, 0.471f, 3.9f},  {64, 64, 0.f, 0.f, 2.1f}};
constexpr float kSmallStep[3] = {0.302f, 0.401f, 0.496f};

}  // namespace

int block_gemm_tile(int M, int N, int K, int cus) {
  const float steps = float(K / 64);
  int best = 0;
  float least = 0.f;
  for (int i = 0; i < 6; ++i) {
    const TileCost& c = kTiles[i];
    const int64_t tiles = int64_t((M + c.bm - 1) / c.bm) * ((N + c.bn - 1) / c.bn);
    float t;
    if (i == 5) {
      const int64_t rounds = tiles / (3 * cus), rest = tiles % (3 * cus);
      t = float(rounds) * (steps * kSmallStep[2] + c.fixed);
      if (rest) t += steps * kSmallStep[(rest - 1) / cus] + c.fixed;
    } else {
      const int64_t rounds = tiles / cus, rest = tiles % cus;
      t = float(rounds) * (steps * c.full + c.fixed);
      if (rest) t += steps * (c.alone + (c.full - c.alone) * float(rest) / float(cus)) + c.fixed;
    }
    if (i == 0 || t < least) {
      best = i;
      least = t;
    }
  }
  return best;
}

namespace {

template <class Epi>
Status block_gemm(const uint16_t* A, int lda, const uint16_t* W, int ldw, int M, int N, int K,
                  const Epi& epi, hipStream_t s) {
  if (M <= 0) return Status::ok();
  DC_TRY(check_gemm(lda, ldw, M, N, K));
  const int cus = compute_units();
  if (cus <= 0) return Status::make(DC_ERR_HIP, "bf16 GEMM: no device");
  switch (block_gemm_tile(M, N, K, cus)) {
    case 0: return launch_dma<384, 192, 4, 2, 2, 2>(A, lda, W, ldw, M, N, K, epi, s);
    case 1: return launch_dma<320, 256, 2, 4, 2, 2>(A, lda, W, ldw, M, N, K, epi, s);
    case 2: return launch_dma<256, 192, 4, 2, 2, 2>(A, lda, W, ldw, M, N, K, epi, s);
    case 3: return launch_dma<256, 128, 4, 2, 2, 3>(A, lda, W, ldw, M, N, K, epi, s);
    case 4: return launch_pipe(A, lda, W, ldw, M, N, K, epi, s);
    default: return launch_dma<64, 64, 2, 2, 2, 3>(A, lda, W, ldw, M, N, K, epi, s);
  }
}

}  // namespace

// ---------------------------------------------------------------------------
// entry points
// ---------------------------------------------------------------------------
Status gemm_bf16_qkv(const uint16_t* A, const uint16_t* W, const float* bias, uint16_t* qk,
                     uint16_t* vt, int ldv, const Geo& g, int M, hipStream_t s) {
  return block_gemm(A, g.d, W, g.d, M, 3 * g.d, g.d,
                    EpiQKVBf16{bias, qk, vt, g.d, ldv, float(1.4426950408889634 / std::sqrt(double(g.Dh)))}, s);
}

Status gemm_bf16_gate_residual(const uint16_t* A, int lda, const uint16_t* W, const float* bias,
                               const float* gate, float* h, int ldh, int M, int N, int K,
                               hipStream_t s) {
  return block_gemm(A, lda, W, K, M, N, K, EpiGateResidual{bias, gate, h, ldh}, s);
}

Status gemm_bf16_gelu(const uint16_t* A, int lda, const uint16_t* W, const float* bias,
                      uint16_t* out, int ldo, int M, int N, int K, hipStream_t s) {
  return block_gemm(A, lda, W, K, M, N, K, EpiGeluBf16{bias, out, ldo}, s);
}

}  // namespace dc
