// Final layer + Euler update of the bf16 model in one pass over g (Eq. 1, H_k):
//
//   x += dsigma * unpatchify( (LN(g) (1 + scale) + shift) W_head^T + b_head )
//
// The LayerNorm is folded into the projection.  For one token with mean mu and
// rstd r, and any shift K,
//   sum_k (LN(g)_k (1 + s_k) + sh_k) W_nk
//     = r (sum_k y_k W_nk - (mu - K) cs_n) + shw_n,
//   y_k = (g_k - K)(1 + s_k),  cs_n = sum_k (1 + s_k) W_nk,  shw_n = sum_k sh_k W_nk,
// so g is read once: the matrix cores take y (split v = hi + lo into two bf16
// operands, about 2^-17 relative, against the bf16 weights) while the same pass
// accumulates the row moments of g - K.
//
// Bound by memory: g is read once.  One persistent workgroup per compute unit takes a
// contiguous range of tokens, 16 at a time.  Its 8 waves split d into 32-wide chunks (at d =
// 1920 seven or eight each) and keep their chunks of W_head in registers for the whole kernel.
// Each wave streams its part of the 16 token rows through a ring of LDS of its own by LDS-DMA,
// eight lanes to the 128 contiguous bytes of a row's chunk, and reads the fragments from there:
// loaded straight into the fragment layout, neighbouring lanes lie on different rows and the L1
// takes a line per lane.  The latent values to update and the shifts come by LDS-DMA too, so no
// load in the token loop has a register destination, and the waits for a chunk are counted by
// hand (every wave issues the same instructions, clamped into range) and leave the rest of the
// ring in flight.  The shift K is the row's first value (a sample of the row, so y stays small
// next to g when the row mean is large); cs and shw are computed once per workgroup on the
// matrix cores.  Per token tile the waves leave their 16 x 64 partial products and moments of
// g - K in LDS; every thread then combines two outputs of one token, adds shw + b and applies
// the Euler update to the two latent values they land on.
// 17,776 x 3,072: 55 us (216 MB, 3.9 TB/s; an LN pass and a GEMM on its rows took 115);
// 17,776 x 1,920: 39 us, 42 before; 3,704 x 1,152 (one tile per workgroup): 12.2 us, 15; with a
// residual 13.3 us, 20.  What is left over the stream is the prologue, about 7 us of W_head
// and cs / shw, and the fifth tile of 4.3.
//
// On a reuse step the head input is g = h_in + r (Eq. 1 with the cached r_j): the
// kResid variant reads h_in and the bf16 residual cache and forms g in registers with
// the same fp32 addition as the cache-apply kernel, so g never goes through HBM.
#include <hip/hip_runtime.h>

#include "internal.h"

namespace dc {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

struct HeadGeo { int T, Hl, Wl, p, Hp, Wp; };

constexpr int kWaves = 8;           // waves per workgroup
constexpr int kLdr = 68;            // row stride (floats) of a wave's 16 x 64 partial tile
constexpr int kChunkG = 128;        // 16-byte pieces of a chunk of g: 16 rows x 8
constexpr int kChunkR = 64;         // and of the residual (bf16)

// LDS-DMA: lane i reads 16 bytes at base + off (or 4 bytes at p) and they land at the
// wave-uniform LDS address dst + 16 i (4 i).  Inline assembly, so that the compiler makes no
// LDS read wait for it; the kernel counts its own waits.
__device__ inline void dma16(const void* base, uint32_t off, const void* dst) {
  const uint32_t lds = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(dst));
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1"
               :: "v"(off), "s"(base), "s"(lds) : "memory", "m0");
}
__device__ inline void dma4(const void* p, const void* dst) {
  const uint32_t lds = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(dst));
  asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dword %0, off"
               :: "v"(p), "s"(lds) : "memory", "m0");
}
// s_waitcnt vmcnt(N), the other counters left alone
template <int N>
__device__ inline void wait_vmcnt() {
  static_assert(N >= 0 && N < 64, "vmcnt range");
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | 0x0F70);
  asm volatile("" ::: "memory");
}
__device__ inline void wait_lds() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }
__device__ inline void barrier() {
  wait_lds();
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// latent element that output n of video token m lands on (unpatchify): channel
// c = n / p^2, pixel (p i + a, p j + b) of frame t, (a, b) = ((n / p) % p, n % p);
// the token's and the output's parts add up
__device__ inline size_t latent_of_token(const HeadGeo& hg, int m) {
  const int r = m / hg.Wp, j = m - r * hg.Wp, t = r / hg.Hp, i = r - t * hg.Hp;
  return (size_t(t) * hg.Hl + hg.p * i) * hg.Wl + hg.p * j;
}
__device__ inline size_t latent_of_output(const HeadGeo& hg, int n) {
  const int pp = hg.p * hg.p, c = n / pp, a = (n / hg.p) % hg.p, b = n % hg.p;
  return (size_t(c) * hg.T * hg.Hl + a) * hg.Wl + b;
}

// chunks [chunk_begin(w), chunk_begin(w + 1)) of the nch chunks of d belong to wave w
__device__ inline int chunk_begin(int w, int nch) { return (w * nch) / kWaves; }

// NC: chunks per wave at most, the last NL of whose W fragments stay in LDS instead of registers;
// RING <= NC: chunks of the token rows a wave has in flight.
template <bool kResid, int NC, int NL, int RING>
__global__ void __launch_bounds__(512) k_head_euler_bf16(const float* __restrict__ gin,
                                                         const uint16_t* __restrict__ resid,
                                                         const uint16_t* __restrict__ W,
                                                         const float* __restrict__ bias,
                                                         const float* __restrict__ shift,
                                                         const float* __restrict__ scale,
                                                         float* __restrict__ x, float dsigma,
                                                         int Nv, int d, float eps, HeadGeo hg) {
  constexpr int kSlot = kChunkG + (kResid ? kChunkR : 0);
  constexpr int kDma = kResid ? 3 : 2;                    // DMA instructions per chunk
  constexpr int kPer = (NC * kWaves * 32 + 511) / 512;    // elements of scale per thread
  static_assert(RING <= NC, "a tile's shifts and latent values arrive in time");
  __shared__ uint4 s_ring[kWaves][RING][kSlot];
  __shared__ float s_x[kWaves][2][64];                    // latent values of a tile, by thread
  __shared__ float* s_xn[32];                             // where outputs 2 i of token 0 land
  __shared__ float* s_px[512];                            // and a tile's outputs, by thread
  __shared__ float s_k[2][kWaves][64];                    // shifts: g, and the residual's dword
  __shared__ float s_sc1[NC * kWaves * 32];               // 1 + scale
  __shared__ float2 s_st[kWaves][16];                     // per wave and row: sum, sum sq of g - K
  __shared__ uint4 s_w[kWaves][NL > 0 ? NL : 1][NL > 0 ? 256 : 1];   // [nb][lane] of a chunk
  __shared__ float s_cs[kWaves][64];                      // cs and shw over each wave's chunks
  __shared__ float s_shw[kWaves][64];
  // Staging of W_head (a chunk of each wave, 4 KB), then scale and shift in bf16, then the
  // per-wave partial products of a token tile: one region, used in that order.
  __shared__ __attribute__((aligned(16))) float s_big[kWaves * 16 * kLdr];
  static_assert(kWaves * 16 * kLdr * 4 >= kWaves * 4096 && kWaves * 16 * kLdr * 4 >= NC * kWaves * 32 * 8,
                "the region holds each of its uses");
  __bf16* const s_ab = reinterpret_cast<__bf16*>(s_big);  // [4][d]: (1 + scale), shift as hi / lo

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int c16 = lane & 15, g4 = lane >> 4;
  const int nch = d >> 5;
  const int cb = chunk_begin(wave, nch);
  const int kc = chunk_begin(wave + 1, nch) - cb;         // may be 0 (d = 128)
  const int last = max(kc - 1, 0);
  // this workgroup's tokens [r0, r1), balanced over the grid
  const int G = gridDim.x, bid = blockIdx.x;
  const int base = Nv / G, extra = Nv % G;
  const int r0 = bid * base + min(bid, extra);
  const int r1 = r0 + base + (bid < extra ? 1 : 0);
  const int ntile = (r1 - r0 + 15) >> 4;

  // Ring: chunk j of the 16 rows of tile t.  Rows past the range, tiles past the last and
  // chunks past kc are clamped (they re-read lines already fetched).  The 16-byte pieces of a
  // row are XOR-swizzled by the row, so that the fragment reads spread over the banks.
  const float* const gb = gin + size_t(r0) * d + 32 * cb;
  const uint16_t* const rb = kResid ? resid + size_t(r0) * d + 32 * cb : nullptr;
  auto row_of = [&](int t, int r) { return min(16 * min(t, ntile - 1) + r, r1 - r0 - 1); };
  struct Off { uint32_t g[2], r; };
  auto offsets = [&](int t) {
    Off o;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int r = 8 * h + (lane >> 3);
      o.g[h] = uint32_t(row_of(t, r) * d) * 4u + 16u * ((lane & 7) ^ ((r >> 1) & 7));
    }
    o.r = kResid ? uint32_t(row_of(t, lane >> 2) * d) * 2u + 16u * ((lane & 3) ^ ((lane >> 4) & 3)) : 0u;
    return o;
  };
  auto fetch = [&](const Off& o, int j, int slot) {
    const int c = 32 * min(j, last);
    uint4* const to = s_ring[wave][slot];
    dma16(gb + c, o.g[0], to);
    dma16(gb + c, o.g[1], to + 64);
    if constexpr (kResid) dma16(rb + c, o.r, to + kChunkG);
  };
  // epilogue role of a thread: token er = tid % 16 of a tile, outputs n = 2 eq and 2 eq + 1
  // with eq = tid / 16
  if (tid < 32) s_xn[tid] = x + latent_of_output(hg, 2 * tid);   // (read after the barriers below)
  const size_t xd = hg.p > 1 ? 1 : size_t(hg.T) * hg.Hl * hg.Wl;      // output 2 eq is an even pixel
  // the latent values of tile t that this thread updates, and where they are
  auto fetch_x = [&](int t) {
    int id = tid;
    asm volatile("" : "+v"(id));                // (as at the end of a tile)
    float* const px = s_xn[id >> 4] + latent_of_token(hg, r0 + row_of(t, id & 15));
    s_px[id] = px;
    dma4(px, s_x[wave][0]);
    dma4(px + xd, s_x[wave][1]);
  };
  // the shifts of tile t
  auto fetch_k = [&](int t) {
    const size_t first = size_t(r0 + row_of(t, c16)) * d;
    const char* pk = reinterpret_cast<const char*>(gin + first);
    if (kResid && (lane & 16)) pk = reinterpret_cast<const char*>(resid + first);
    dma4(pk, s_k[t & 1][wave]);
  };
  Off off = offsets(0);
  fetch_k(0);
#pragma unroll
  for (int q = 0; q < RING; ++q) fetch(off, q, q);

  // scale and shift (k = tid + 512 i), written to LDS once W is staged
  float scv[kPer], shv[kPer];
  auto load_mod = [&] {
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
      const int k = min(tid + 512 * i, d - 1);
      scv[i] = scale[k];
      shv[i] = shift[k];
    }
  };
  if constexpr (NC <= 8) load_mod();            // (wider: W leaves no registers to wait in)
  // W_head fragments (B operand: column n = 16 nb + c16, k = 8 g4 + e of the chunk), each chunk
  // through the wave's 4 KB slab (a load instruction reads 16 rows x 64 contiguous bytes), the
  // four 16-byte pieces of a row XOR-swizzled.  Chunks j >= kc (unused) repeat the last.
  bf16x8 wf[NC - NL][4];
  {
    uint4* const slab = reinterpret_cast<uint4*>(s_big) + wave * 256;
    constexpr int kRound = NC > 8 ? 3 : NC;               // chunks whose loads go out together
#pragma unroll
    for (int j0 = 0; j0 < NC; j0 += kRound) {
      uint4 v[kRound][4];
#pragma unroll
      for (int j = 0; j < kRound; ++j)
#pragma unroll
        for (int i = 0; i < 4; ++i)
          v[j][i] = *reinterpret_cast<const uint4*>(W + size_t(16 * i + (lane >> 2)) * d +
                                                    32 * (cb + min(j0 + j, last)) + 8 * (lane & 3));
#pragma unroll
      for (int j = 0; j < kRound; ++j) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int row = 16 * i + (lane >> 2);
          slab[row * 4 + ((lane & 3) ^ ((row >> 2) & 3))] = v[j][i];
        }
#pragma unroll
        for (int nb = 0; nb < 4; ++nb)
        {
          const uint4 f = slab[(16 * nb + c16) * 4 + (g4 ^ ((c16 >> 2) & 3))];
          if (j0 + j < NC - NL) wf[j0 + j < NC - NL ? j0 + j : 0][nb] = __builtin_bit_cast(bf16x8, f);
          else s_w[wave][NL > 0 ? j0 + j - (NC - NL) : 0][64 * nb + lane] = f;
        }
      }
    }
  }
  if constexpr (NC > 8) load_mod();
  auto frag = [&](int j, int nb) -> bf16x8 {
    if (j < NC - NL) return wf[j < NC - NL ? j : 0][nb];
    return __builtin_bit_cast(bf16x8, s_w[wave][NL > 0 ? j - (NC - NL) : 0][64 * nb + lane]);
  };
  barrier();                                    // every slab is read: the region takes
#pragma unroll                                  // (1 + scale) and shift split to bf16 hi / lo
  for (int i = 0; i < kPer; ++i) {
    const int k = tid + 512 * i;
    if (k < d) {
      const float f = 1.0f + scv[i];
      s_sc1[k] = f;
      const __bf16 fh = static_cast<__bf16>(f), sh = static_cast<__bf16>(shv[i]);
      s_ab[k] = fh;
      s_ab[d + k] = static_cast<__bf16>(f - static_cast<float>(fh));
      s_ab[2 * d + k] = sh;
      s_ab[3 * d + k] = static_cast<__bf16>(shv[i] - static_cast<float>(sh));
    }
  }
  barrier();

  // cs_w and shw_w on the matrix cores: A rows 0 / 1 = (1 + scale) hi / lo, rows 2 / 3
  // = shift hi / lo, the other rows zero.  Rows 0..3 of the result are registers 0..3
  // of lanes 0..15.
  {
    f32x4 pc[4];
#pragma unroll
    for (int nb = 0; nb < 4; ++nb) pc[nb] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int j = 0; j < NC; ++j) {
      if (j < kc) {
        uint4 a = *reinterpret_cast<const uint4*>(s_ab + min(c16, 3) * d + 32 * (cb + j) + 8 * g4);
        if (c16 >= 4) a = make_uint4(0, 0, 0, 0);
        const bf16x8 af = __builtin_bit_cast(bf16x8, a);
#pragma unroll
        for (int nb = 0; nb < 4; ++nb)
          pc[nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af, frag(j, nb), pc[nb], 0, 0, 0);
      }
    }
    if (g4 == 0)
#pragma unroll
      for (int nb = 0; nb < 4; ++nb) {
        s_cs[wave][16 * nb + c16] = pc[nb][0] + pc[nb][1];
        s_shw[wave][16 * nb + c16] = pc[nb][2] + pc[nb][3];
      }
  }
  barrier();
  if (tid < 64) {                               // over all waves, into the first one's row
    float v = bias[tid], c = 0.f;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
      v += s_shw[w][tid];
      c += s_cs[w][tid];
    }
    s_shw[0][tid] = v;                          // (read after the barriers of the first tile)
    s_cs[0][tid] = c;
  }
  const float inv_d = 1.0f / float(d);

  int slot = 0;
  for (int t = 0; t < ntile; ++t) {
    fetch_x(t);
    fetch_k(t + 1);
    f32x4 acc[4];
#pragma unroll
    for (int nb = 0; nb < 4; ++nb) acc[nb] = f32x4{0.f, 0.f, 0.f, 0.f};
    float s1 = 0.f, s2 = 0.f, kcur = 0.f;
#pragma unroll
    for (int j = 0; j < NC; ++j) {
      // The chunk has landed when at most the RING - 1 newer ones are outstanding (the other
      // loads and stores among them only make this wait for more).  The tile's shifts were
      // issued NC >= RING chunks ago, so they are there for the first chunk, and by the wait
      // for the last chunk the tile's latent values are too.
      wait_vmcnt<kDma * (RING - 1)>();
      if (j == 0) {
        kcur = s_k[t & 1][wave][c16];
        if constexpr (kResid) kcur += __uint_as_float(__float_as_uint(s_k[t & 1][wave][16 + c16]) << 16);
      }
      const uint4* const from = s_ring[wave][slot];
      const int pr = c16 * 8, sw = (c16 >> 1) & 7;
      const float4 va = __builtin_bit_cast(float4, from[pr + ((2 * g4) ^ sw)]);
      const float4 vb = __builtin_bit_cast(float4, from[pr + ((2 * g4 + 1) ^ sw)]);
      uint4 rw = make_uint4(0, 0, 0, 0);
      if constexpr (kResid) rw = from[kChunkG + c16 * 4 + (g4 ^ ((c16 >> 2) & 3))];
      const int k0 = 32 * (cb + min(j, last)) + 8 * g4;
      const float4 sa = *reinterpret_cast<const float4*>(s_sc1 + k0);
      const float4 sb = *reinterpret_cast<const float4*>(s_sc1 + k0 + 4);
      wait_lds();                               // read: the slot takes the chunk RING ahead
      if (j == NC - RING) off = offsets(t + 1);
      fetch(off, j + RING < NC ? j + RING : j + RING - NC, slot);
      slot = slot + 1 == RING ? 0 : slot + 1;
      if (j < kc) {
        float e[8] = {va.x, va.y, va.z, va.w, vb.x, vb.y, vb.z, vb.w};
        if constexpr (kResid) {                 // g = h_in + r, the cache-apply addition
          const uint32_t r[4] = {rw.x, rw.y, rw.z, rw.w};
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            e[2 * i] += __uint_as_float(r[i] << 16);
            e[2 * i + 1] += __uint_as_float(r[i] & 0xFFFF0000u);
          }
        }
        const float sc[8] = {sa.x, sa.y, sa.z, sa.w, sb.x, sb.y, sb.z, sb.w};
        bf16x8 ah, al, fw[4];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          const float u = e[i] - kcur;
          s1 += u;
          s2 = fmaf(u, u, s2);
          const float y = u * sc[i];
          const __bf16 h = static_cast<__bf16>(y);
          ah[i] = h;
          al[i] = static_cast<__bf16>(y - static_cast<float>(h));
        }
#pragma unroll
        for (int nb = 0; nb < 4; ++nb) fw[nb] = frag(j, nb);
#pragma unroll
        for (int nb = 0; nb < 4; ++nb) acc[nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah, fw[nb], acc[nb], 0, 0, 0);
#pragma unroll
        for (int nb = 0; nb < 4; ++nb) acc[nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(al, fw[nb], acc[nb], 0, 0, 0);
      }
    }

    // From here to the end of the tile everything is computed from a copy of the thread index
    // that the compiler cannot see through: addresses kept over the chunks would be spilled, and
    // a reload waits for the whole ring.
    int id = tid;
    asm volatile("" : "+v"(id));
    const int ln = id & 63, c = ln & 15, q4 = ln >> 4, er = id & 15, eq = id >> 4;
    // this wave's moments of each row (the row's four lane groups) and partial products
    s1 += __shfl_xor(s1, 16, 64);
    s1 += __shfl_xor(s1, 32, 64);
    s2 += __shfl_xor(s2, 16, 64);
    s2 += __shfl_xor(s2, 32, 64);
    barrier();                                  // the last tile's partials are combined
    if (q4 == 0) s_st[wave][c] = make_float2(s1, s2);
    float* const pa = s_big + wave * 16 * kLdr + 4 * q4 * kLdr + c;
#pragma unroll
    for (int nb = 0; nb < 4; ++nb)
#pragma unroll
      for (int i = 0; i < 4; ++i) pa[i * kLdr + 16 * nb] = acc[nb][i];
    barrier();

    // combine: mean - K and variance of the token, then
    // r (sum_w acc_w - (mu - K) cs) + shw + b
    float t1 = 0.f, t2 = 0.f, o0 = 0.f, o1 = 0.f;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
      const float2 st = s_st[w][er];
      const float2 a = *reinterpret_cast<const float2*>(&s_big[(w * 16 + er) * kLdr + 2 * eq]);
      t1 += st.x;
      t2 += st.y;
      o0 += a.x;
      o1 += a.y;
    }
    const float dm = t1 * inv_d;                               // mu - K
    const float var = fmaxf(t2 * inv_d - dm * dm, 0.f);
    const float rs = 1.0f / sqrtf(var + eps);
    if (r0 + 16 * t + er < r1) {
      float* const px = s_px[id];
      const float2 cs = *reinterpret_cast<const float2*>(&s_cs[0][2 * eq]);
      const float2 shw = *reinterpret_cast<const float2*>(&s_shw[0][2 * eq]);
      px[0] = s_x[wave][0][ln] + dsigma * (rs * (o0 - dm * cs.x) + shw.x);
      px[xd] = s_x[wave][1][ln] + dsigma * (rs * (o1 - dm * cs.y) + shw.y);
    }
  }
  wait_vmcnt<0>();                              // the chunks past the last tile land before the LDS goes
}

template <int NC, int NL, int RG, int RR>
Status launch(int grid, const float* gin, const uint16_t* resid, const uint16_t* W, const float* bias,
              const float* shift, const float* scale, float* x, float dsigma, const Geo& g, hipStream_t s) {
  const HeadGeo hg{g.T, g.Hl, g.Wl, g.p, g.Hp, g.Wp};
  if constexpr (RR > 0) {
    if (resid) {
      hipLaunchKernelGGL((k_head_euler_bf16<true, NC, NL, RR>), dim3(grid), dim3(512), 0, s, gin, resid, W, bias, shift,
                         scale, x, dsigma, g.Nv, g.d, g.eps, hg);
      DC_HIP(hipGetLastError());
      return Status::ok();
    }
  }
  if (resid) return Status::shape("bf16 head with a residual input needs d <= 2048");
  hipLaunchKernelGGL((k_head_euler_bf16<false, NC, NL, RG>), dim3(grid), dim3(512), 0, s, gin, resid, W, bias, shift,
                     scale, x, dsigma, g.Nv, g.d, g.eps, hg);
  DC_HIP(hipGetLastError());
  return Status::ok();
}

}  // namespace

bool head_takes_resid(const Geo& g) { return g.bf16 && g.d <= 2048; }

Status head_euler_bf16(const float* gin, const uint16_t* resid, const uint16_t* W, const float* bias,
                       const float* shift, const float* scale, float* x, float dsigma, const Geo& g,
                       hipStream_t s) {
  if (g.Nv <= 0) return Status::ok();
  if (g.P != 64 || g.d % 128 || g.d > 3072) return Status::shape("bf16 head needs 64 outputs, d % 128 == 0 and d <= 3072");
  const int cus = compute_units();
  if (cus <= 0) return Status::make(DC_ERR_HIP, "bf16 head: no device");
  const int tiles = (g.Nv + 15) / 16, grid = cus < tiles ? cus : tiles;
  // Chunks per wave, d / 256 rounded up, decide the registers for W and what is loaded past
  // the last chunk; the ring takes what LDS is left, six chunks (four with a residual) at most.
  const int nc = (g.d + 255) / 256;
  if (nc <= 3) return launch<3, 0, 3, 3>(grid, gin, resid, W, bias, shift, scale, x, dsigma, g, s);
  if (nc <= 5) return launch<5, 0, 5, 4>(grid, gin, resid, W, bias, shift, scale, x, dsigma, g, s);
  if (nc <= 8) return launch<8, 0, 6, 4>(grid, gin, resid, W, bias, shift, scale, x, dsigma, g, s);
  return launch<12, 1, 4, 0>(grid, gin, resid, W, bias, shift, scale, x, dsigma, g, s);
}

}  // namespace dc
