// Joint video + text self-attention, softmax(Q K^T / sqrt(d_h)) V per head, with
// an online softmax (flash-style: the N x N score matrix never leaves registers).
//
// Three bf16 kernels (the fp32 model's attention is in attention_f32.hip): k_attn16 (head_dim 64,
// many items), k_attn_keys (short sequences) and k_attn_bf16 (head_dim 64 between those, and
// head_dim 72); which one is chosen at attention_bf16, the first two have comments of their own.
//
// k_attn_bf16 (gfx950 MFMA 32x32x16).  A workgroup is 4 waves x 32 query rows of one
// head; key/value tiles of 64 tokens stream through a 3-stage LDS ring.  The QKV
// GEMM stores Q pre-multiplied by log2(e)/sqrt(d_h), so scores arrive in log2
// units and P = 2^(s - m).  Each wave
// computes the transposed scores S^T = K Q^T, so in the accumulator layout every
// lane holds scores of a single query row (lane % 32): the row max needs one
// cross-lane exchange (lanes l and l^32) and the rescale of the output is a
// per-lane multiply.  The output is accumulated transposed as well,
// O^T += V^T P^T, which needs V^T in LDS (the QKV GEMM writes V transposed).
// The K rows feeding the S^T tiles are permuted (bits 2 and 3 of the row index
// swapped) so that the eight scores a lane holds for each 16-token slice of P are
// eight consecutive tokens: P goes from the score registers straight into the
// B operand of the P V product, and V^T is read with one 16-byte LDS load.
// Per-score VALU work is kept to the exponential, half a bf16 conversion and one
// fp32 add for the row sum: the subtraction of the running maximum m rides on
// the MFMA as one extra rank-1 step (a column of ones times -m).  The row sum is
// a plain v_add chain rather than v_dot2 on the bf16 pairs: on gfx950 the dot
// instructions do not issue alongside running MFMAs, adds do.  m is set from
// the first tile's maximum and raised only when a tile's P would grow past 2^64
// (the tile's row sum is the test), so the common path takes no tile maximum;
// P and the fp32 sums stay far inside the fp32 range either way.
#include <hip/hip_runtime.h>

#include <cmath>
#include <type_traits>

#include "internal.h"

namespace dc {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

__device__ inline uint16_t to_bf16(float f) {
  return __builtin_bit_cast(uint16_t, static_cast<__bf16>(f));
}

// LDS chunk swizzle for 128-byte tile rows.  gfx950's LDS serves 256 bytes per
// cycle (64 banks): two consecutive rows share a bank cycle, so the XOR key is
// row / 2, which gives the 16 rows that 16 consecutive lanes read (in any order,
// including the permuted K order) 16 distinct 16-byte bank groups.
__device__ inline int swz_k(int row) { return (row >> 1) & 7; }
__device__ inline int swz_v(int row) { return (row >> 1) & 7; }
__device__ inline int perm_kv(int m) { return (m & ~12) | ((m & 4) << 1) | ((m & 8) >> 1); }


typedef __attribute__((address_space(3))) void lds_void;

// 16 bytes per lane global -> LDS (global_load_lds_dwordx4): lane i reads
// base + off (a wave-uniform 64-bit base, a per-lane 32-bit byte offset) and its
// bytes land at the wave-uniform LDS address dst + 16 i.  Issued as inline
// assembly: the compiler cannot tell the stage being filled from the stage being
// read and would otherwise wait for every outstanding fill before each LDS read.
// The kernel waits for its own fills explicitly (vmcnt) before the barrier that
// publishes a stage.
__device__ inline void dma16(const void* base, uint32_t off, const void* dst) {
  const uint32_t lds = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(dst));
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1"
               :: "v"(off), "s"(base), "s"(lds) : "memory", "m0");
}

template <int D>
struct AttnShape {
  static constexpr int DK = (D + 15) / 16 * 16;   // contraction width of Q K^T (zero padded)
  static constexpr int KC = DK / 8;               // 16-byte chunks per K row in LDS
  static constexpr int DC8 = D / 8;               // chunks holding real data
  static constexpr int DV = (D + 31) / 32 * 32;   // rows of the O^T accumulator
  static constexpr int TV = DV / 32;
  static constexpr int BKV = 64;                  // tokens per K/V tile
  static constexpr int KSLOTS = BKV * KC;         // 16-byte LDS slots of a K tile
  static constexpr int VSLOTS = DV * 8;           // of a V^T tile (64 tokens = 8 chunks per row)
  static constexpr int KI = (KSLOTS + 255) / 256; // DMA instructions per wave (4 waves x 64 lanes)
  static constexpr int VI = (VSLOTS + 255) / 256;
};

// K/V^T tiles go global -> LDS into a ring of three stages (separate arrays),
// prefetched two tiles ahead; one barrier per tile.
// Lane i of a DMA instruction lands at the instruction's LDS base + 16 i, so each
// lane fetches the global chunk that belongs at its slot: the swizzle and the
// K-padding are applied on the global side.  Rows past the data (K rows past M,
// padding chunks, V^T rows past D) fetch real, finite data whose products are
// either multiplied by zero (padded Q columns, masked P) or never stored.
template <int D>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(D == 64 ? 3 : 2)))
k_attn_bf16(const uint16_t* __restrict__ qk,
                                                   const uint16_t* __restrict__ vt, int ldv,
                                                   uint16_t* __restrict__ out, int M, int d,
                                                   int nqb, int items, int per_xcd, int full,
                                                   float* __restrict__ part) {
  using S = AttnShape<D>;
  constexpr int DK = S::DK, KC = S::KC, DC8 = S::DC8, TV = S::TV, BKV = S::BKV;
  constexpr int KI = S::KI, VI = S::VI;
  // one array, so every stage address is a constant offset from one base
  constexpr int STAGE = (KI + VI) * 256;
  __shared__ uint4 lds[3 * STAGE];
  uint4* const sK0 = lds;
  uint4* const sV0 = lds + KI * 256;
  uint4* const sK1 = lds + STAGE;
  uint4* const sV1 = lds + STAGE + KI * 256;
  uint4* const sK2 = lds + 2 * STAGE;
  uint4* const sV2 = lds + 2 * STAGE + KI * 256;

  // Work item w = head * nqb + query block.  Workgroups are dealt to the XCDs
  // round-robin, so workgroup b runs item (b % 8) * per_xcd + b / 8: each XCD
  // sweeps a contiguous range of items, i.e. the query blocks of one head at a
  // time, and that head's K and V stay in its L2.
  //
  // Tail split: XCD x owns items [x per_xcd, (x + 1) per_xcd).  Its first `full`
  // work units are whole items; every later item is split into two units, one per
  // half of the key tiles, so the last (partial) round of resident workgroups runs
  // half as long.  A split unit leaves its unnormalised output, running maximum and
  // row sum in `part` (record si = x (per_xcd - full) + index among the XCD's split
  // items); k_attn_combine merges the two halves.
  const int xcd = blockIdx.x & 7, u = blockIdx.x >> 3;
  const int ibeg = xcd * per_xcd, iend = min(items, ibeg + per_xcd);
  const int nfull = min(full, iend - ibeg);
  int w, half = -1;
  if (u < nfull) {
    w = ibeg + u;
  } else {
    w = ibeg + nfull + ((u - nfull) >> 1);
    half = (u - nfull) & 1;
  }
  if (w >= iend) return;
  const int ntile = (M + BKV - 1) / BKV;
  const int tb = half == 1 ? ntile / 2 : 0;              // key tiles [tb, te)
  const int te = half == 0 ? ntile / 2 : ntile;
  const int head = w / nqb;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // uniform: DMA addresses in SGPRs
  const int g = lane >> 5, r32 = lane & 31;
  const int q0 = (w - head * nqb) * 128 + wave * 32;
  const int ldq = 2 * d;
  const uint16_t* Qb = qk + head * D;
  const uint16_t* Kb = qk + d + head * D;
  const uint16_t* Vb = vt + size_t(head) * D * ldv;
  const uint4 zero4 = make_uint4(0, 0, 0, 0);

  // query fragments (B operand of S^T): lane holds Q[q0 + r32][16 kk + 8 g .. + 8]
  bf16x8 qf[DK / 16];
#pragma unroll
  for (int kk = 0; kk < DK / 16; ++kk) {
    const int col = 16 * kk + 8 * g;
    const int q = q0 + r32;
    uint4 v = zero4;
    if (q < M && col < D) v = *reinterpret_cast<const uint4*>(Qb + size_t(q) * ldq + col);
    qf[kk] = __builtin_bit_cast(bf16x8, v);
  }
  // the query fragments have landed before the first LDS-DMA is issued, so no
  // later wait on them can also hold up the tile pipeline
  __builtin_amdgcn_s_waitcnt(0x0F70);

  // per-lane source byte offsets of this wave's DMA instructions for tile 0; tile t
  // adds a uniform t * 64 rows (K) or t * 64 columns (V^T).  K rows run up to
  // 64 + 12 past the tile start: the qk buffer has ldv + 64 rows, and rows past M
  // only feed scores that the last tile masks (by assignment, so any bits are safe).
  uint32_t offK[KI], offV[VI];
#pragma unroll
  for (int i = 0; i < KI; ++i) {
    const int slot = (wave * KI + i) * 64 + lane;
    const int r = slot / KC, pc = slot % KC;
    const int c = (KC == 8) ? (pc ^ swz_k(r)) : pc;
    const int cc = c < DC8 ? c : 0;                    // padding chunk: any real chunk
    offK[i] = 2u * uint32_t(r * ldq + 8 * cc);
  }
#pragma unroll
  for (int i = 0; i < VI; ++i) {
    const int slot = (wave * VI + i) * 64 + lane;
    const int r = slot >> 3, c = (slot & 7) ^ swz_v(slot >> 3);
    offV[i] = 2u * uint32_t(min(r, D - 1) * ldv + 8 * c);
  }
  auto issue = [&](uint4* sk, uint4* sv, int t) {
    const uint16_t* kt = Kb + size_t(t) * BKV * ldq;
    const uint16_t* vtt = Vb + t * BKV;
#pragma unroll
    for (int i = 0; i < KI; ++i) dma16(kt, offK[i], sk + (wave * KI + i) * 64);
#pragma unroll
    for (int i = 0; i < VI; ++i) dma16(vtt, offV[i], sv + (wave * VI + i) * 64);
  };

  f32x16 o[TV];
#pragma unroll
  for (int t = 0; t < TV; ++t)
#pragma unroll
    for (int i = 0; i < 16; ++i) o[t][i] = 0.f;
  // Scores arrive in log2 units (Q pre-scaled by log2(e)/sqrt(d_h)).  One extra
  // rank-1 MFMA step (k = 8) adds -m to every score: A is a column of ones (the
  // first k slot of the lanes with g = 0), B holds -m of the lane's query in its
  // first k slot.  m is kept exactly representable in bf16.
  typedef short s16x4 __attribute__((ext_vector_type(4)));
  const s16x4 kaug = {short(g == 0 ? 0x3F80 : 0), 0, 0, 0};
  s16x4 qaug = {0, 0, 0, 0};
  float mrow = 0.f, lsum = 0.f;

  auto compute = [&](const uint4* sk, const uint4* sv, int t) {
    // S^T for two 32-token sub-tiles; sub-tile st, register i holds token
    // 32 st + 16 (i / 8) + 8 g + (i % 8) of the tile, query q0 + r32.
    f32x16 s[2];
#pragma unroll
    for (int st = 0; st < 2; ++st) {
      f32x16 z;
#pragma unroll
      for (int i = 0; i < 16; ++i) z[i] = 0.f;
      s[st] = __builtin_amdgcn_mfma_f32_32x32x8bf16_1k(kaug, qaug, z, 0, 0, 0);
      const int row = 32 * st + perm_kv(r32);
#pragma unroll
      for (int kk = 0; kk < DK / 16; ++kk) {
        const int ch = 2 * kk + g;
        const int pc = (KC == 8) ? (ch ^ swz_k(row)) : ch;
        const bf16x8 kf = __builtin_bit_cast(bf16x8, sk[row * KC + pc]);
        s[st] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf, qf[kk], s[st], 0, 0, 0);
      }
    }
    if ((t + 1) * BKV > M) {
#pragma unroll
      for (int st = 0; st < 2; ++st)
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          const int kv = t * BKV + 32 * st + 16 * (i >> 3) + 8 * g + (i & 7);
          if (kv >= M) s[st][i] = -INFINITY;
        }
    }
    // raise m to the tile maximum (first tile; later only when P would grow past 2^64)
    auto raise = [&](bool first) {
      float mx = s[0][0];
#pragma unroll
      for (int st = 0; st < 2; ++st)
#pragma unroll
        for (int i = 0; i < 16; ++i) mx = fmaxf(mx, s[st][i]);
      mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
      const float mnew = __uint_as_float(uint32_t(to_bf16(mrow + (first ? mx : fmaxf(mx, 0.f)))) << 16);
      const float up = mnew - mrow;
      // (up < 0 only on the first tile, where O and l are zero and 2^-up may overflow)
      const float alpha = __builtin_amdgcn_exp2f(fminf(-up, 0.f));
      mrow = mnew;
      qaug[0] = short(to_bf16(-mnew));
      lsum *= alpha;
#pragma unroll
      for (int tv = 0; tv < TV; ++tv)
#pragma unroll
        for (int i = 0; i < 16; ++i) o[tv][i] *= alpha;
#pragma unroll
      for (int st = 0; st < 2; ++st)
#pragma unroll
        for (int i = 0; i < 16; ++i) s[st][i] -= up;
    };
    if (t == tb) raise(true);
    bf16x8 pf[4];
    float ts = 0.f;
    auto exps = [&]() {
      // two add chains over the fp32 exponentials (the MFMA consumes them rounded to bf16)
      float t2[2];
#pragma unroll
      for (int c = 0; c < 4; ++c)
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const float p = __builtin_amdgcn_exp2f(s[c >> 1][8 * (c & 1) + e]);
          t2[e & 1] = (c == 0 && e < 2) ? p : t2[e & 1] + p;
          pf[c][e] = static_cast<__bf16>(p);
        }
      ts = t2[0] + t2[1];
    };
    exps();
    // P stays far inside fp32 range while m lags the running maximum by less than
    // about 58 (log2 units); only then is m raised (rare), so no tile maximum is
    // taken on the common path
    if (t > tb && __builtin_amdgcn_ballot_w64(!(ts < 0x1p64f)) != 0) {
      raise(false);
      exps();
    }
    lsum += ts;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const int ch = 2 * c + g;
#pragma unroll
      for (int tv = 0; tv < TV; ++tv) {
        const int row = 32 * tv + r32;
        const bf16x8 vf = __builtin_bit_cast(bf16x8, sv[row * 8 + (ch ^ swz_v(row))]);
        o[tv] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf, pf[c], o[tv], 0, 0, 0);
      }
    }
  };

  // vmcnt(n) with the other counters left alone
  constexpr int kPerTile = KI + VI;
  issue(sK0, sV0, tb);
  if (tb + 1 < te) issue(sK1, sV1, tb + 1);
  auto step = [&](uint4* sk, uint4* sv, uint4* nk, uint4* nv, int t) {
    if (t + 1 < te) __builtin_amdgcn_s_waitcnt(0x0F70 | kPerTile);    // tile t landed (t+1 may fly)
    else __builtin_amdgcn_s_waitcnt(0x0F70);
    __builtin_amdgcn_s_barrier();          // everyone's tile t landed; tile t-1's stage is free
    if (t + 2 < te) issue(nk, nv, t + 2);
    compute(sk, sv, t);
  };
  for (int t = tb; t < te; t += 3) {
    step(sK0, sV0, sK2, sV2, t);
    if (t + 1 >= te) break;
    step(sK1, sV1, sK0, sV0, t + 1);
    if (t + 2 >= te) break;
    step(sK2, sV2, sK1, sV1, t + 2);
  }

  lsum += __shfl_xor(lsum, 32, 64);
  if (half >= 0) {
    // split unit: unnormalised O, m and l of the wave's 32 queries; record layout
    // [half][128 queries][D + 4] floats (O, m, l, two unused: 16-byte aligned rows)
    const int si = xcd * (per_xcd - full) + (w - ibeg - nfull);
    float* rec = part + (size_t(si) * 2 + half) * 128 * (D + 4) + size_t(wave * 32 + r32) * (D + 4);
#pragma unroll
    for (int tv = 0; tv < TV; ++tv)
#pragma unroll
      for (int i4 = 0; i4 < 4; ++i4) {
        const int dh = 32 * tv + 8 * i4 + 4 * g;
        if (dh < D)
          *reinterpret_cast<float4*>(rec + dh) =
              make_float4(o[tv][4 * i4 + 0], o[tv][4 * i4 + 1], o[tv][4 * i4 + 2], o[tv][4 * i4 + 3]);
      }
    if (g == 0) {
      rec[D] = mrow;
      rec[D + 1] = lsum;
    }
    return;
  }
  const float inv = 1.0f / lsum;
  const int q = q0 + r32;
  if (q < M) {
    uint16_t* orow = out + size_t(q) * d + head * D;
#pragma unroll
    for (int tv = 0; tv < TV; ++tv)
#pragma unroll
      for (int i4 = 0; i4 < 4; ++i4) {
        const int dh = 32 * tv + 8 * i4 + 4 * g;
        if (dh < D) {
          ushort4 u;
          u.x = to_bf16(o[tv][4 * i4 + 0] * inv);
          u.y = to_bf16(o[tv][4 * i4 + 1] * inv);
          u.z = to_bf16(o[tv][4 * i4 + 2] * inv);
          u.w = to_bf16(o[tv][4 * i4 + 3] * inv);
          *reinterpret_cast<ushort4*>(orow + dh) = u;
        }
      }
  }
}

// Merge the two key halves of every split item: O = (O0 2^(m0-m) + O1 2^(m1-m)) /
// (l0 2^(m0-m) + l1 2^(m1-m)) with m = max(m0, m1).  One workgroup per split item,
// two threads per query (half of the head dimension each).
template <int D>
__global__ void __launch_bounds__(256) k_attn_combine(const float* __restrict__ part,
                                                      uint16_t* __restrict__ out, int M, int d,
                                                      int nqb, int items, int per_xcd, int full) {
  const int per = per_xcd - full;                 // split items per XCD (record stride)
  const int si = blockIdx.x, xcd = si / per, k = si % per;
  const int ibeg = xcd * per_xcd, iend = min(items, ibeg + per_xcd);
  const int w = ibeg + full + k;
  if (full >= iend - ibeg || w >= iend) return;
  const int head = w / nqb, ql = threadIdx.x >> 1, hf = threadIdx.x & 1;
  const int q = (w - head * nqb) * 128 + ql;
  if (q >= M) return;
  const float* r0 = part + (size_t(si) * 2 + 0) * 128 * (D + 4) + size_t(ql) * (D + 4);
  const float* r1 = r0 + 128 * (D + 4);
  const float m0 = r0[D], l0 = r0[D + 1], m1 = r1[D], l1 = r1[D + 1];
  const float m = fmaxf(m0, m1);
  const float a0 = __builtin_amdgcn_exp2f(m0 - m), a1 = __builtin_amdgcn_exp2f(m1 - m);
  const float inv = 1.0f / (l0 * a0 + l1 * a1);
  constexpr int DH = D / 2;                       // 32 or 36 dims per thread
  uint16_t* orow = out + size_t(q) * d + head * D + hf * DH;
#pragma unroll
  for (int j = 0; j < DH; j += 4) {
    const float4 x0 = *reinterpret_cast<const float4*>(r0 + hf * DH + j);
    const float4 x1 = *reinterpret_cast<const float4*>(r1 + hf * DH + j);
    ushort4 v;
    v.x = to_bf16((x0.x * a0 + x1.x * a1) * inv);
    v.y = to_bf16((x0.y * a0 + x1.y * a1) * inv);
    v.z = to_bf16((x0.z * a0 + x1.z * a1) * inv);
    v.w = to_bf16((x0.w * a0 + x1.w * a1) * inv);
    *reinterpret_cast<ushort4*>(orow + j) = v;
  }
}

// ---------------------------------------------------------------------------
// k_attn16: head_dim 64 on v_mfma_f32_16x16x32_bf16.  Same work items and tail split as
// k_attn_bf16, but a two-stage K/V^T ring (32 KB of LDS, the next tile's DMA issued
// right after the barrier that frees its stage) and at most 128 VGPRs, so four
// workgroups (four waves per SIMD) are resident: 3 % faster at 17,776 tokens x 30
// heads than three-stage rings at three waves per SIMD.  Per wave: 32 queries as two
// 16-query blocks; the transposed scores S^T come in 16 x 16 blocks (lane: query lane % 16,
// rows 4 (lane / 16) .. + 3 of the block).
//  - The running maximum enters as the C operand of the first score MFMA (four
//    registers holding -m per query block), so scores arrive as s - m.
//  - Each lane's eight P values of a 32-key chunk are the B operand of
//    O^T += V^T P^T directly (K rows permuted, see perm16); the matching V^T operand
//    is one 16-byte LDS read.
//  - The row sum l is one more MFMA per chunk with an all-ones A operand, so the
//    VALU does one exp2 and half a bf16 pack per score and nothing else; numerator
//    and denominator use the same bf16-rounded P.
//  - m comes from the first tile's maximum.  When a tile leaves l at 2^64 or more (a later
//    score more than about 58 above m), m is raised after the tile by the exponent of l, if
//    l and O are finite.  If not (a score more than about 120 above m, or less with huge V),
//    the wave sits out the rest of the pass and the workgroup redoes the item with the tile
//    maximum taken on every tile (the safe pass).  us, one key 80 to 97 above the others,
//    before the raise -> now (as fast as ordinary scores): 2,500 tokens x 30 heads
//    140 -> 64, 17,776 x 30 4,782 -> 1,969; first tile 290 below the rest, the safe pass:
//    2,500 x 30 135 -> 119, 17,776 x 30 4,510 -> 3,235.
// ---------------------------------------------------------------------------
typedef float f32x4 __attribute__((ext_vector_type(4)));

// K rows are read in a permuted order within each 32-key chunk: S^T block row
// 16 h + 4 g + i (h < 2, g < 4, i < 4) holds key 8 g + 4 h + i, so the eight P values
// a lane holds for a chunk (rows 4 g + i of blocks 2c and 2c+1) are keys 8 g .. 8 g + 7
// and the V^T operand is one 16-byte read.  The K swizzle is keyed on the row bits
// that vary across the 16 rows one LDS cycle reads in that order.
__device__ inline int perm16(int p) {
  return (p & 32) | (((p >> 2) & 3) << 3) | (((p >> 4) & 1) << 2) | (p & 3);
}
__device__ inline int swz_k16(int row) { return ((row >> 1) & 1) | ((row >> 2) & 6); }

__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4)))
k_attn16(const uint16_t* __restrict__ qk, const uint16_t* __restrict__ vt, int ldv,
         uint16_t* __restrict__ out, int M, int d, int nqb, int items, int per_xcd, int full,
         float* __restrict__ part) {
  constexpr int D = 64, BKV = 64;
  constexpr int KI = 2, VI = 2;                 // DMA instructions per wave per tile (K, V^T)
  constexpr int STAGE = (KI + VI) * 256;        // 16-byte slots per ring stage
  __shared__ uint4 lds[2 * STAGE];
  __shared__ int redo;
  uint4* const sK0 = lds;
  uint4* const sV0 = lds + KI * 256;
  uint4* const sK1 = lds + STAGE;
  uint4* const sV1 = lds + STAGE + KI * 256;

  const int xcd = blockIdx.x & 7, u = blockIdx.x >> 3;
  const int ibeg = xcd * per_xcd, iend = min(items, ibeg + per_xcd);
  const int nfull = min(full, iend - ibeg);
  int w, half = -1;
  if (u < nfull) {
    w = ibeg + u;
  } else {
    w = ibeg + nfull + ((u - nfull) >> 1);
    half = (u - nfull) & 1;
  }
  if (w >= iend) return;
  const int ntile = (M + BKV - 1) / BKV;
  const int tb = half == 1 ? ntile / 2 : 0;     // key tiles [tb, te)
  const int te = half == 0 ? ntile / 2 : ntile;
  const int head = w / nqb;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int c16 = lane & 15, g4 = lane >> 4;
  const int q0 = (w - head * nqb) * 128 + wave * 32;
  const int ldq = 2 * d;
  const uint16_t* Qb = qk + head * D;
  const uint16_t* Kb = qk + d + head * D;
  const uint16_t* Vb = vt + size_t(head) * D * ldv;
  if (tid == 0) redo = 0;

  // query fragments: lane holds Q[q0 + 16 qb + c16][32 kk + 8 g4 .. + 8]
  bf16x8 qf[2][2];
#pragma unroll
  for (int qb = 0; qb < 2; ++qb)
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) {
      const int q = q0 + 16 * qb + c16;
      uint4 v = make_uint4(0, 0, 0, 0);
      if (q < M) v = *reinterpret_cast<const uint4*>(Qb + size_t(q) * ldq + 32 * kk + 8 * g4);
      qf[qb][kk] = __builtin_bit_cast(bf16x8, v);
    }
  __builtin_amdgcn_s_waitcnt(0x0F70);

  uint32_t offK[KI], offV[VI];
#pragma unroll
  for (int i = 0; i < KI; ++i) {
    const int slot = (wave * KI + i) * 64 + lane;
    const int r = slot >> 3, c = (slot & 7) ^ swz_k16(slot >> 3);
    offK[i] = 2u * uint32_t(r * ldq + 8 * c);
  }
#pragma unroll
  for (int i = 0; i < VI; ++i) {
    const int slot = (wave * VI + i) * 64 + lane;
    const int r = slot >> 3, c = (slot & 7) ^ swz_v(slot >> 3);
    offV[i] = 2u * uint32_t(r * ldv + 8 * c);
  }
  auto issue = [&](uint4* sk, uint4* sv, int t) {
    const uint16_t* kt = Kb + size_t(t) * BKV * ldq;
    const uint16_t* vtt = Vb + t * BKV;
#pragma unroll
    for (int i = 0; i < KI; ++i) dma16(kt, offK[i], sk + (wave * KI + i) * 64);
#pragma unroll
    for (int i = 0; i < VI; ++i) dma16(vtt, offV[i], sv + (wave * VI + i) * 64);
  };

  bf16x8 ones;
#pragma unroll
  for (int e = 0; e < 8; ++e) ones[e] = static_cast<__bf16>(1.0f);

  f32x4 o[4][2], lacc[2], mneg[2];
  bool fail = false;

  // one pass over the key tiles; safe: take the tile maximum on every tile
  auto run = [&](bool safe) {
#pragma unroll
    for (int qb = 0; qb < 2; ++qb) {
#pragma unroll
      for (int i = 0; i < 4; ++i) { lacc[qb][i] = 0.f; mneg[qb][i] = 0.f; }
#pragma unroll
      for (int db = 0; db < 4; ++db)
#pragma unroll
        for (int i = 0; i < 4; ++i) o[db][qb][i] = 0.f;
    }
    fail = false;

    auto rescale = [&](int qb, float up) {      // m += up; O, l *= 2^-up
      // (up < 0 only on the first tile, where O and l are zero and 2^-up may overflow)
      const float a = __builtin_amdgcn_exp2f(fminf(-up, 0.f));
      const float m = up - mneg[qb][0];
#pragma unroll
      for (int i = 0; i < 4; ++i) { lacc[qb][i] *= a; mneg[qb][i] = -m; }
#pragma unroll
      for (int db = 0; db < 4; ++db)
#pragma unroll
        for (int i = 0; i < 4; ++i) o[db][qb][i] *= a;
    };

    // scores of key block kb (16 keys) for both query blocks, with C = -m; with
    // kMask the keys past M are set to -inf (the last tile only, so the common path
    // is one branch-free block the scheduler can interleave)
    auto scores = [&](const uint4* sk, int t, int kb, f32x4 (&sc)[2], auto kMask) {
      const int row = perm16(16 * kb + c16);
      const bf16x8 k0 = __builtin_bit_cast(bf16x8, sk[row * 8 + ((0 + g4) ^ swz_k16(row))]);
      const bf16x8 k1 = __builtin_bit_cast(bf16x8, sk[row * 8 + ((4 + g4) ^ swz_k16(row))]);
#pragma unroll
      for (int qb = 0; qb < 2; ++qb) {
        sc[qb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(k0, qf[qb][0], mneg[qb], 0, 0, 0);
        sc[qb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(k1, qf[qb][1], sc[qb], 0, 0, 0);
      }
      if constexpr (decltype(kMask)::value) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (t * BKV + perm16(16 * kb + 4 * g4 + i) >= M) {
            sc[0][i] = -INFINITY;
            sc[1][i] = -INFINITY;
          }
      }
    };

    // all scores of the tile, then per 32-key chunk: P = 2^(s - m) (bf16), O^T += V^T P^T,
    // l += 1 P^T.  P of chunk c: keys 32 c + 8 g4 .. + 7 (blocks 2c and 2c+1, permuted rows)
    auto body = [&](const uint4* sk, const uint4* sv, int t, auto kMask) {
      f32x4 sb[4][2];
#pragma unroll
      for (int kb = 0; kb < 4; ++kb) scores(sk, t, kb, sb[kb], kMask);
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        bf16x8 pf[2];
#pragma unroll
        for (int qb = 0; qb < 2; ++qb)
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            pf[qb][e] = static_cast<__bf16>(__builtin_amdgcn_exp2f(sb[2 * c][qb][e]));
            pf[qb][4 + e] = static_cast<__bf16>(__builtin_amdgcn_exp2f(sb[2 * c + 1][qb][e]));
          }
#pragma unroll
        for (int db = 0; db < 4; ++db) {
          const int row = 16 * db + c16;
          const bf16x8 vf = __builtin_bit_cast(bf16x8, sv[row * 8 + ((4 * c + g4) ^ swz_v(row))]);
#pragma unroll
          for (int qb = 0; qb < 2; ++qb)
            o[db][qb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf, pf[qb], o[db][qb], 0, 0, 0);
        }
#pragma unroll
        for (int qb = 0; qb < 2; ++qb)
          lacc[qb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ones, pf[qb], lacc[qb], 0, 0, 0);
      }
    };

    // one tile: the tile maximum (first tile, safe pass), P V and l, then the raise check
    auto tile = [&](const uint4* sk, const uint4* sv, int t, auto kMask, bool domax) {
      if (domax) {
        // the tile maximum (a separate pass over the scores, which are recomputed below)
        float mx[2] = {-INFINITY, -INFINITY};
#pragma unroll
        for (int kb = 0; kb < 4; ++kb) {
          f32x4 sc[2];
          scores(sk, t, kb, sc, kMask);
#pragma unroll
          for (int qb = 0; qb < 2; ++qb)
#pragma unroll
            for (int i = 0; i < 4; ++i) mx[qb] = fmaxf(mx[qb], sc[qb][i]);
        }
#pragma unroll
        for (int qb = 0; qb < 2; ++qb) {
          float m = fmaxf(mx[qb], __shfl_xor(mx[qb], 16, 64));
          m = fmaxf(m, __shfl_xor(m, 32, 64));
          const float up = t == tb ? m : fmaxf(m, 0.f);
          if (up != 0.f) rescale(qb, up);
        }
      }
      body(sk, sv, t, kMask);
      // m lags the scores by more than about 58 (l >= 2^64; all rows of lacc hold l).  While l
      // and O are finite nothing has overflowed, and m is raised by the exponent of l (at
      // most 126, so that 2^-up is no denormal); else the item is redone in the safe pass.
      if (!safe) {
        const bool big = !(lacc[0][0] < 0x1p64f && lacc[1][0] < 0x1p64f);
        // a real branch (not a select): it ends the tile's scheduling region, which keeps
        // the compiler from interleaving tiles (that spills), marked unlikely, so that the
        // registers of the loop are not spilled for it either (14 % slower)
        if (__builtin_expect(__builtin_amdgcn_ballot_w64(big) != 0, 0)) {
          float z = 0.f;                        // stays 0 if all are finite
#pragma unroll
          for (int qb = 0; qb < 2; ++qb) {
            if (!(lacc[qb][0] < 0x1p126f)) z = 1.f;
#pragma unroll
            for (int db = 0; db < 4; ++db)
#pragma unroll
              for (int i = 0; i < 4; ++i) z += o[db][qb][i] * 0.f;
          }
          if (__builtin_expect(__builtin_amdgcn_ballot_w64(z != 0.f) != 0, 0)) {
            fail = true;
          } else {
#pragma unroll
            for (int qb = 0; qb < 2; ++qb)
              rescale(qb, lacc[qb][0] < 0x1p64f ? 0.f : float(__builtin_amdgcn_frexp_expf(lacc[qb][0])));
          }
        }
      }
    };
    // two-stage ring: tile t has landed in every wave's view and every wave is done with
    // tile t - 1, whose stage (nk, nv) then takes tile t + 1
    auto sync = [&](int t, uint4* nk, uint4* nv) {
      __builtin_amdgcn_s_waitcnt(0x0F70);
      __builtin_amdgcn_s_barrier();
      if (t + 1 < te) issue(nk, nv, t + 1);
    };
    constexpr std::false_type kFull{};
    constexpr std::true_type kPart{};
    // tile t sits in ring stage (t - tb) % 2.  The first tile and a partial last tile
    // run outside the loop, so the loop body is one branch-free instance per stage.
    const bool part_last = te * BKV > M;
    const int tm = part_last ? te - 1 : te;     // tiles [tb, tm) are full
    issue(sK0, sV0, tb);
    sync(tb, sK1, sV1);
    if (tb < tm) tile(sK0, sV0, tb, kFull, true);
    else tile(sK0, sV0, tb, kPart, true);
    for (int t = tb + 1; t < tm; t += 2) {
      sync(t, sK0, sV0);
      if (__builtin_expect(!fail, 1)) tile(sK1, sV1, t, kFull, safe);
      if (t + 1 >= tm) break;
      sync(t + 1, sK1, sV1);
      if (__builtin_expect(!fail, 1)) tile(sK0, sV0, t + 1, kFull, safe);
    }
    if (part_last && te - 1 > tb) {
      const int t = te - 1, q = (t - tb) % 2;
      sync(t, sK0, sV0);                        // t + 1 = te: nothing to prefetch
      tile(sK0 + q * STAGE, sV0 + q * STAGE, t, kPart, safe);   // one instance, stage by address
    }
  };

  // pass 0 is the fast path; pass 1 (rare) redoes the item with the tile maximum on
  // every tile when any wave gave up (one call site: one inlined copy)
  for (int pass = 0;; ++pass) {
    run(pass > 0);
    if (pass > 0) break;
    if (__builtin_amdgcn_ballot_w64(fail) != 0 && lane == 0) redo = 1;
    __syncthreads();
    if (!redo) break;
    __syncthreads();
  }

  if (half >= 0) {
    const int si = xcd * (per_xcd - full) + (w - ibeg - nfull);
#pragma unroll
    for (int qb = 0; qb < 2; ++qb) {
      float* rec = part + (size_t(si) * 2 + half) * 128 * (D + 4) + size_t(wave * 32 + 16 * qb + c16) * (D + 4);
#pragma unroll
      for (int db = 0; db < 4; ++db)
        *reinterpret_cast<float4*>(rec + 16 * db + 4 * g4) =
            make_float4(o[db][qb][0], o[db][qb][1], o[db][qb][2], o[db][qb][3]);
      if (g4 == 0) {
        rec[D] = -mneg[qb][0];
        rec[D + 1] = lacc[qb][0];
      }
    }
    return;
  }
#pragma unroll
  for (int qb = 0; qb < 2; ++qb) {
    const int q = q0 + 16 * qb + c16;
    if (q >= M) continue;
    const float inv = 1.0f / lacc[qb][0];
    uint16_t* orow = out + size_t(q) * d + head * D;
#pragma unroll
    for (int db = 0; db < 4; ++db) {
      ushort4 v;
      v.x = to_bf16(o[db][qb][0] * inv);
      v.y = to_bf16(o[db][qb][1] * inv);
      v.z = to_bf16(o[db][qb][2] * inv);
      v.w = to_bf16(o[db][qb][3] * inv);
      *reinterpret_cast<ushort4*>(orow + 16 * db + 4 * g4) = v;
    }
  }
}

// ---------------------------------------------------------------------------
// Short sequences: fewer items of 128 queries than compute units leave most of them idle and
// one or two waves per SIMD on the rest (300 tokens x 30 heads: 90 items).  Here a workgroup
// takes 64 queries of one head and its four waves are two query blocks of 32 times two wave
// groups that take alternate key tiles and merge through LDS at the end: twice the
// workgroups, half the serial chain over the keys.  Otherwise as k_attn16 (16x16x32 MFMAs,
// -m as the C operand, the safe pass), with registers to spare at two waves per SIMD.
// head_dim 64: K rows in natural order in LDS, read permuted; l is an all-ones MFMA.
// head_dim 72: K rows stored permuted, 144 bytes each (conflict-free as it is), three 32-wide
// steps of the score product with zeros in Q past the row; O^T has five 16-row blocks, of whose
// last eight rows are used, and the ninth V^T row in LDS holds ones, so that row of O is l.
// ---------------------------------------------------------------------------
template <int D>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2)))
k_attn_keys(const uint16_t* __restrict__ qk, const uint16_t* __restrict__ vt, int ldv,
            uint16_t* __restrict__ out, int M, int d, int nqb, int items, int per_xcd) {
  constexpr int BKV = 64, QW = 2, KS = 2, QR = 32 * QW;   // keys per tile, wave grid, queries
  constexpr int KK = (D + 31) / 32;             // 32-wide steps of the score product
  constexpr int DB = (D + 15) / 16;             // 16-row blocks of O^T
  constexpr int KC = D / 8;                     // 16-byte chunks per K row
  constexpr bool kOnesRow = D % 16 != 0;        // l comes with O (row D of V^T holds ones)
  constexpr int TI = 8 / QW;                    // DMA instructions per wave, tile and operand
  constexpr int KSLOT = BKV * KC, VSLOT = 16 * DB * 8, TILE = KSLOT + VSLOT;   // 16-byte slots
  constexpr int STAGE = KS * TILE;
  static_assert(D == 64 || D == 72, "64 slots more per operand at D = 72");
  __shared__ uint4 lds[2 * STAGE];
  __shared__ int redo;

  const int w = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
  if (w >= items) return;
  const int te = (M + BKV - 1) / BKV;           // key tiles, at least one per group (M > 64)
  const int head = w / nqb;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int qw = wave % QW, ks = wave / QW;
  const int c16 = lane & 15, g4 = lane >> 4;
  const int q0 = (w - head * nqb) * QR + qw * 32;
  const int ldq = 2 * d;
  const uint16_t* Qb = qk + head * D;
  const uint16_t* Kb = qk + d + head * D;
  const uint16_t* Vb = vt + size_t(head) * D * ldv;
  if (tid == 0) redo = 0;
  if constexpr (kOnesRow) {
    // V^T rows D .. 16 DB - 1 of every tile buffer: ones, then zeros (the DMA never writes them)
    for (int e = tid; e < 2 * KS * (16 * DB - D) * 8; e += 256) {
      const int b = e / ((16 * DB - D) * 8), r = e % ((16 * DB - D) * 8);
      const uint32_t v = r < 8 ? 0x3F803F80u : 0u;
      lds[b * TILE + KSLOT + D * 8 + r] = make_uint4(v, v, v, v);
    }
  }

  // query fragments: lane holds Q[q0 + 16 qb + c16][32 kk + 8 g4 .. + 8]
  bf16x8 qf[2][KK];
#pragma unroll
  for (int qb = 0; qb < 2; ++qb)
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) {
      const int q = q0 + 16 * qb + c16;
      uint4 v = make_uint4(0, 0, 0, 0);
      if (q < M && 32 * kk + 8 * g4 < D) v = *reinterpret_cast<const uint4*>(Qb + size_t(q) * ldq + 32 * kk + 8 * g4);
      qf[qb][kk] = __builtin_bit_cast(bf16x8, v);
    }
  __builtin_amdgcn_s_waitcnt(0x0F70);

  // A DMA instruction fills 64 slots; each group fills its own tile of a stage, its two waves four
  // instructions of K and of V^T each.  At head_dim 72 each operand has 64 slots more: wave
  // 2 j takes those of tile j's K, wave 2 j + 1 those of its V^T.
  auto k_off = [&](int slot) {                  // byte offset of a K slot from its tile's first row
    const int r = D == 64 ? slot >> 3 : perm16(slot / KC);
    const int c = D == 64 ? (slot & 7) ^ swz_k16(slot >> 3) : slot % KC;
    return 2u * uint32_t(r * ldq + 8 * c);
  };
  auto v_off = [&](int slot) {
    const int r = slot >> 3, c = (slot & 7) ^ swz_v(r);
    return 2u * uint32_t(r * ldv + 8 * c);
  };
  uint32_t offK[TI], offV[TI], offX = 0;
#pragma unroll
  for (int i = 0; i < TI; ++i) {
    offK[i] = k_off((qw * TI + i) * 64 + lane);
    offV[i] = v_off((qw * TI + i) * 64 + lane);
  }
  if constexpr (D == 72) offX = wave & 1 ? v_off(512 + lane) : k_off(512 + lane);
  auto issue = [&](uint4* stage, int t0) {      // tiles t0, t0 + 1 into a stage
    const int t = t0 + ks;
    if (t < te) {
      uint4* sk = stage + ks * TILE;
      const uint16_t* kt = Kb + size_t(t) * BKV * ldq;
      const uint16_t* vtt = Vb + t * BKV;
#pragma unroll
      for (int i = 0; i < TI; ++i) dma16(kt, offK[i], sk + (qw * TI + i) * 64);
#pragma unroll
      for (int i = 0; i < TI; ++i) dma16(vtt, offV[i], sk + KSLOT + (qw * TI + i) * 64);
    }
    if constexpr (D == 72) {
      const int j = wave >> 1, tx = t0 + j;
      if (tx < te) {
        uint4* sk = stage + j * TILE;
        if (wave & 1) dma16(Vb + tx * BKV, offX, sk + KSLOT + 512);
        else dma16(Kb + size_t(tx) * BKV * ldq, offX, sk + 512);
      }
    }
  };

  bf16x8 ones;
#pragma unroll
  for (int e = 0; e < 8; ++e) ones[e] = static_cast<__bf16>(1.0f);

  f32x4 o[DB][2], lacc[kOnesRow ? 1 : 2], mneg[2];
  float mrow[2];
  bool fail = false;
  // l of query block qb: every lane (ones MFMA), or lanes with g4 == (D % 16) / 4
  auto l_of = [&](int qb) { return kOnesRow ? o[DB - 1][qb][0] : lacc[kOnesRow ? 0 : qb][0]; };
  // the same in every lane
  auto l_all = [&](int qb) { return kOnesRow ? __shfl(l_of(qb), 16 * ((D % 16) / 4) + c16, 64) : l_of(qb); };

  // one pass over the key tiles; safe: take the tile maximum on every tile
  auto run = [&](bool safe) {
#pragma unroll
    for (int qb = 0; qb < 2; ++qb) {
      mrow[qb] = 0.f;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        if constexpr (!kOnesRow) lacc[qb][i] = 0.f;
        mneg[qb][i] = 0.f;
      }
#pragma unroll
      for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int i = 0; i < 4; ++i) o[db][qb][i] = 0.f;
    }
    fail = false;

    auto rescale = [&](int qb, float up) {      // m += up; O, l *= 2^-up
      // (up < 0 only on the first tile, where O and l are zero and 2^-up may overflow)
      const float a = __builtin_amdgcn_exp2f(fminf(-up, 0.f));
      mrow[qb] += up;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        if constexpr (!kOnesRow) lacc[qb][i] *= a;
        mneg[qb][i] = -mrow[qb];
      }
#pragma unroll
      for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int i = 0; i < 4; ++i) o[db][qb][i] *= a;
    };

    // scores of key block kb (16 keys) for both query blocks, with C = -m; with
    // kMask the keys past M are set to -inf (the last tile only, so the common path
    // is one branch-free block the scheduler can interleave).  Chunks past the row (D = 72)
    // re-read its last one: Q is zero there.
    auto scores = [&](const uint4* sk, int t, int kb, f32x4 (&sc)[2], auto kMask) {
#pragma unroll
      for (int kk = 0; kk < KK; ++kk) {
        bf16x8 kf;
        if constexpr (D == 64) {
          const int row = perm16(16 * kb + c16);
          kf = __builtin_bit_cast(bf16x8, sk[row * 8 + ((4 * kk + g4) ^ swz_k16(row))]);
        } else {
          const int ch = 4 * kk + 3 < KC ? 4 * kk + g4 : min(4 * kk + g4, KC - 1);
          kf = __builtin_bit_cast(bf16x8, sk[(16 * kb + c16) * KC + ch]);
        }
#pragma unroll
        for (int qb = 0; qb < 2; ++qb)
          sc[qb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf, qf[qb][kk], kk == 0 ? mneg[qb] : sc[qb], 0, 0, 0);
      }
      if constexpr (decltype(kMask)::value) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (t * BKV + perm16(16 * kb + 4 * g4 + i) >= M) {
            sc[0][i] = -INFINITY;
            sc[1][i] = -INFINITY;
          }
      }
    };

    // all scores of the tile, then per 32-key chunk: P = 2^(s - m) (bf16), O^T += V^T P^T,
    // l += 1 P^T.  P of chunk c: keys 32 c + 8 g4 .. + 7 (blocks 2c and 2c+1, permuted rows)
    auto body = [&](const uint4* sk, const uint4* sv, int t, auto kMask) {
      f32x4 sb[4][2];
#pragma unroll
      for (int kb = 0; kb < 4; ++kb) scores(sk, t, kb, sb[kb], kMask);
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        bf16x8 pf[2];
#pragma unroll
        for (int qb = 0; qb < 2; ++qb)
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            pf[qb][e] = static_cast<__bf16>(__builtin_amdgcn_exp2f(sb[2 * c][qb][e]));
            pf[qb][4 + e] = static_cast<__bf16>(__builtin_amdgcn_exp2f(sb[2 * c + 1][qb][e]));
          }
#pragma unroll
        for (int db = 0; db < DB; ++db) {
          const int row = 16 * db + c16;
          const bf16x8 vf = __builtin_bit_cast(bf16x8, sv[row * 8 + ((4 * c + g4) ^ swz_v(row))]);
#pragma unroll
          for (int qb = 0; qb < 2; ++qb)
            o[db][qb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf, pf[qb], o[db][qb], 0, 0, 0);
        }
        if constexpr (!kOnesRow) {
#pragma unroll
          for (int qb = 0; qb < 2; ++qb)
            lacc[qb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ones, pf[qb], lacc[qb], 0, 0, 0);
        }
      }
    };

    // one tile: the tile maximum (first tile, safe pass), P V and l, then the raise check
    auto tile = [&](const uint4* sk, int t, auto kMask, bool domax, bool first) {
      const uint4* sv = sk + KSLOT;
      if (domax) {
        // the tile maximum (a separate pass over the scores, which are recomputed below)
        float mx[2] = {-INFINITY, -INFINITY};
#pragma unroll
        for (int kb = 0; kb < 4; ++kb) {
          f32x4 sc[2];
          scores(sk, t, kb, sc, kMask);
#pragma unroll
          for (int qb = 0; qb < 2; ++qb)
#pragma unroll
            for (int i = 0; i < 4; ++i) mx[qb] = fmaxf(mx[qb], sc[qb][i]);
        }
#pragma unroll
        for (int qb = 0; qb < 2; ++qb) {
          float m = fmaxf(mx[qb], __shfl_xor(mx[qb], 16, 64));
          m = fmaxf(m, __shfl_xor(m, 32, 64));
          const float up = first ? m : fmaxf(m, 0.f);
          if (up != 0.f) rescale(qb, up);
        }
      }
      body(sk, sv, t, kMask);
      // m lags the scores by more than about 58 (l >= 2^64): raised or redone, as in k_attn16
      if (!safe) {
        bool big = !(l_of(0) < 0x1p64f && l_of(1) < 0x1p64f);
        if constexpr (kOnesRow) big = big && g4 == (D % 16) / 4;
        // a real branch (not a select): it ends the tile's scheduling region, which keeps
        // the compiler from interleaving tiles (that spills)
        if (__builtin_expect(__builtin_amdgcn_ballot_w64(big) != 0, 0)) {
          float z = 0.f;                        // stays 0 if all are finite
#pragma unroll
          for (int qb = 0; qb < 2; ++qb) {
            if (!(l_of(qb) < 0x1p126f)) z = 1.f;
#pragma unroll
            for (int db = 0; db < DB; ++db)
#pragma unroll
              for (int i = 0; i < 4; ++i) z += o[db][qb][i] * 0.f;
          }
          if (__builtin_expect(__builtin_amdgcn_ballot_w64(z != 0.f) != 0, 0)) {
            fail = true;
          } else {
#pragma unroll
            for (int qb = 0; qb < 2; ++qb) {
              const float l = l_all(qb);
              rescale(qb, l < 0x1p64f ? 0.f : float(__builtin_amdgcn_frexp_expf(l)));
            }
          }
        }
      }
    };
    // two-stage ring: the stage's tiles have landed in every wave's view and every wave is done
    // with the stage before, which then takes the KS tiles after
    auto sync = [&](int t0, uint4* next) {
      __builtin_amdgcn_s_waitcnt(0x0F70);
      __builtin_amdgcn_s_barrier();
      if (t0 + KS < te) issue(next, t0 + KS);
    };
    constexpr std::false_type kFull{};
    constexpr std::true_type kPart{};
    uint4* const s0 = lds;
    uint4* const s1 = lds + STAGE;
    // Step i takes tiles 2 i and 2 i + 1 from ring stage i % 2, one per group.  The first step and
    // a last one with a partial or missing tile run outside the loop, so the loop body is
    // one branch-free instance per stage.
    const int nst = (te + KS - 1) / KS;
    const bool ragged = nst * KS * BKV > M;           // the last step is not all full
    const int nfl = ragged ? nst - 1 : nst;
    const int off = ks * TILE;
    issue(s0, 0);
    sync(0, s1);
    if (nfl > 0) tile(s0 + off, ks, kFull, true, true);
    else tile(s0 + off, ks, kPart, true, true);
    for (int i = 1; i < nfl; i += 2) {
      sync(i * KS, s0);
      if (__builtin_expect(!fail, 1)) tile(s1 + off, i * KS + ks, kFull, safe, false);
      if (i + 1 >= nfl) break;
      sync((i + 1) * KS, s1);
      if (__builtin_expect(!fail, 1)) tile(s0 + off, (i + 1) * KS + ks, kFull, safe, false);
    }
    if (ragged && nst > 1) {
      const int i = nst - 1, t = i * KS + ks;
      sync(i * KS, s0);                               // nothing left to prefetch
      if (t < te) tile(lds + (i & 1) * STAGE + off, t, kPart, safe, false);   // one instance, stage by address
    }
  };

  // pass 0 is the fast path; pass 1 (rare) redoes the item with the tile maximum on
  // every tile when any wave gave up (one call site: one inlined copy)
  if constexpr (kOnesRow) __syncthreads();      // the ones rows are written
  for (int pass = 0;; ++pass) {
    run(pass > 0);
    if (pass > 0) break;
    if (__builtin_amdgcn_ballot_w64(fail) != 0 && lane == 0) redo = 1;
    __syncthreads();
    if (!redo) break;
    __syncthreads();
  }

  float l[2];
#pragma unroll
  for (int qb = 0; qb < 2; ++qb) l[qb] = l_all(qb);

  // group 1 leaves O, m and l in LDS (the tiles are done with), group 0 merges
  constexpr int ROW = D + 4;
  static_assert(size_t(QR) * ROW * 4 <= sizeof(lds), "merge space");
  float* const mem = reinterpret_cast<float*>(lds);
  __syncthreads();
  if (ks > 0) {
#pragma unroll
    for (int qb = 0; qb < 2; ++qb) {
      float* rec = mem + (qw * 32 + 16 * qb + c16) * ROW;
#pragma unroll
      for (int db = 0; db < DB; ++db)
        if (16 * db + 4 * g4 < D)
          *reinterpret_cast<float4*>(rec + 16 * db + 4 * g4) =
              make_float4(o[db][qb][0], o[db][qb][1], o[db][qb][2], o[db][qb][3]);
      if (g4 == 0) {
        rec[D] = mrow[qb];
        rec[D + 1] = l[qb];
      }
    }
  }
  __syncthreads();
  if (ks > 0) return;
#pragma unroll
  for (int qb = 0; qb < 2; ++qb) {
    const float* rec = mem + (qw * 32 + 16 * qb + c16) * ROW;
    const float m1 = rec[D], m = fmaxf(mrow[qb], m1);
    const float a0 = __builtin_amdgcn_exp2f(mrow[qb] - m), a1 = __builtin_amdgcn_exp2f(m1 - m);
    l[qb] = l[qb] * a0 + rec[D + 1] * a1;
#pragma unroll
    for (int db = 0; db < DB; ++db)
      if (16 * db + 4 * g4 < D) {
        const float4 x = *reinterpret_cast<const float4*>(rec + 16 * db + 4 * g4);
        o[db][qb][0] = o[db][qb][0] * a0 + x.x * a1;
        o[db][qb][1] = o[db][qb][1] * a0 + x.y * a1;
        o[db][qb][2] = o[db][qb][2] * a0 + x.z * a1;
        o[db][qb][3] = o[db][qb][3] * a0 + x.w * a1;
      }
  }
#pragma unroll
  for (int qb = 0; qb < 2; ++qb) {
    const int q = q0 + 16 * qb + c16;
    if (q >= M) continue;
    const float inv = 1.0f / l[qb];
    uint16_t* orow = out + size_t(q) * d + head * D;
#pragma unroll
    for (int db = 0; db < DB; ++db) {
      if (16 * db + 4 * g4 >= D) continue;
      ushort4 v;
      v.x = to_bf16(o[db][qb][0] * inv);
      v.y = to_bf16(o[db][qb][1] * inv);
      v.z = to_bf16(o[db][qb][2] * inv);
      v.w = to_bf16(o[db][qb][3] * inv);
      *reinterpret_cast<ushort4*>(orow + 16 * db + 4 * g4) = v;
    }
  }
}

}  // namespace

// Resident workgroups of the bf16 attention kernel per XCD on the current device
// (compute units / 8 x workgroups per compute unit), cached per device.
template <int D>
static int attn_slots_per_xcd() {
  static int cache[64] = {0};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 0;
  if (cache[dev] == 0) {
    int cus = 0, per_cu = 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_attn_bf16<D>, 256, 0) != hipSuccess)
      return 0;
    cache[dev] = (cus / 8) * per_cu;
  }
  return cache[dev];
}

static int attn16_slots_per_xcd() {
  static int cache[64] = {0};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 0;
  if (cache[dev] == 0) {
    int cus = 0, per_cu = 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_attn16, 256, 0) != hipSuccess)
      return 0;
    cache[dev] = (cus / 8) * per_cu;
  }
  return cache[dev];
}

// How many of an XCD's items run whole (launch_attn): the items of the last partial round are
// split when their halves fit in one round.
static int whole_items(int per_xcd, int slots, int M, int D, size_t part_bytes) {
  if (slots <= 0 || (M + 63) / 64 < 2) return per_xcd;
  const int f = per_xcd / slots * slots, r = per_xcd - f;
  const size_t need = size_t(8) * r * 2 * 128 * (D + 4) * sizeof(float);
  return r > 0 && 2 * r <= slots && need <= part_bytes ? f : per_xcd;
}

template <int D, bool V16>
static Status launch_attn(const uint16_t* qk, const uint16_t* vt, int ldv, uint16_t* out, const Geo& g,
                          int M, float* part, size_t part_bytes, hipStream_t s) {
  const int nqb = (M + 127) / 128, items = nqb * g.H, per_xcd = (items + 7) / 8;
  const int slots = V16 ? attn16_slots_per_xcd() : attn_slots_per_xcd<D>();
  const int full = whole_items(per_xcd, slots, M, D, part ? part_bytes : 0);
  const int units = full + 2 * (per_xcd - full);
  if constexpr (V16)
    hipLaunchKernelGGL(k_attn16, dim3(8 * units), dim3(256), 0, s, qk, vt, ldv, out, M, g.d, nqb, items,
                       per_xcd, full, part);
  else
    hipLaunchKernelGGL(k_attn_bf16<D>, dim3(8 * units), dim3(256), 0, s, qk, vt, ldv, out, M, g.d, nqb,
                       items, per_xcd, full, part);
  DC_HIP(hipGetLastError());
  if (full < per_xcd) {
    hipLaunchKernelGGL(k_attn_combine<D>, dim3(8 * (per_xcd - full)), dim3(256), 0, s, part, out, M, g.d,
                       nqb, items, per_xcd, full);
    DC_HIP(hipGetLastError());
  }
  return Status::ok();
}

template <int D>
static Status launch_keys(const uint16_t* qk, const uint16_t* vt, int ldv, uint16_t* out, const Geo& g, int M,
                          hipStream_t s) {
  const int nqb = (M + 63) / 64, items = nqb * g.H, per_xcd = (items + 7) / 8;
  hipLaunchKernelGGL(k_attn_keys<D>, dim3(8 * per_xcd), dim3(256), 0, s, qk, vt, ldv, out, M, g.d, nqb, items,
                     per_xcd);
  DC_HIP(hipGetLastError());
  return Status::ok();
}

// Which kernel (256 compute units, us, head_dim 64 unless noted):
//  - k_attn_keys while its items (64 queries of a head) are at most two per compute unit, from two
//    key tiles on: 300 tokens x 30 heads 6.8, k_attn_bf16 12.2; 1,556 x 20 (500 items) 18.9 and
//    34.5; head_dim 72, 2,000 x 16 (512) 29.2 and 38.2, 3,000 x 16 (752) 64.7 and 57.7;
//  - k_attn16 (head_dim 64) from 2.25 items of 128 queries per compute unit: 5,000 x 48 (1,920
//    items) 276, k_attn_bf16 304; 2,500 x 30 (600) 56.9 and 57.7; 5,000 x 12 (480) 87 and 80.5;
//    17,776 x 30 1,916 and 2,127.  How the last rounds fill shifts that by up to 3 % either way:
//    3,597 x 30 (870) 115 and 111.5, 17,000 x 4 (532) 338 and 343;
//  - k_attn_bf16 between, and for head_dim 72.
AttnKernel attention_kernel(int head_dim, int heads, int tokens, int cus) {
  if (tokens > 64 && int64_t(heads) * ((tokens + 63) / 64) <= 2 * int64_t(cus)) return AttnKernel::kKeys;
  if (head_dim == 64 && 4 * int64_t(heads) * ((tokens + 127) / 128) >= 9 * int64_t(cus)) return AttnKernel::k16;
  return AttnKernel::kBf16;
}

bool attention_splits(int head_dim, int heads, int tokens) {
  const AttnKernel k = attention_kernel(head_dim, heads, tokens, compute_units());
  if (k == AttnKernel::kKeys) return false;
  const int slots = k == AttnKernel::k16 ? attn16_slots_per_xcd()
                    : head_dim == 64     ? attn_slots_per_xcd<64>()
                                         : attn_slots_per_xcd<72>();
  const int per_xcd = (heads * ((tokens + 127) / 128) + 7) / 8;
  return whole_items(per_xcd, slots, tokens, head_dim, attn_part_bytes(head_dim)) < per_xcd;
}

Status attention_bf16(const uint16_t* qk, const uint16_t* vt, int ldv, uint16_t* out,
                      const Geo& g, int M, float* part, size_t part_bytes, hipStream_t s) {
  if (ldv % 64 || ldv < M) return Status::shape("attention needs ldv >= M, ldv % 64 == 0");
  // the padding tokens [M, ldv) of vt hold zeros: the bf16 QKV GEMM writes them
  if (g.Dh != 64 && g.Dh != 72) return Status::shape("bf16 attention supports head_dim 64 and 72");
  const int cus = compute_units();
  if (cus <= 0) return Status::make(DC_ERR_HIP, "bf16 attention: no device");
  switch (attention_kernel(g.Dh, g.H, M, cus)) {
    case AttnKernel::kKeys:
      return g.Dh == 64 ? launch_keys<64>(qk, vt, ldv, out, g, M, s) : launch_keys<72>(qk, vt, ldv, out, g, M, s);
    case AttnKernel::k16: return launch_attn<64, true>(qk, vt, ldv, out, g, M, part, part_bytes, s);
    default: break;
  }
  if (g.Dh == 72) return launch_attn<72, false>(qk, vt, ldv, out, g, M, part, part_bytes, s);
  return launch_attn<64, false>(qk, vt, ldv, out, g, M, part, part_bytes, s);
}

}  // namespace dc
