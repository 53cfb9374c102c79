// Patch embedding with the text rows, one launch for all samples:
//
//   h_in[n] = patch(x)[n] W_pe^T + b + pos[n]  (n < N_v),   h_in[N_v + i] = txt[i]
//
// bf16 model: fp32 latent and fp32 W_pe at fp32 accuracy on bf16 MFMA: each operand is split v = hi + lo
// (hi = bf16(v), lo = bf16(v - hi)) and the product is hi*Whi + lo*Whi + hi*Wlo (the dropped
// lo*Wlo is about 2^-18 relative).
//
// Bound by memory: h_in is written and the positions are read once.  A wave owns 64 columns,
// whose split weights (64 x 64) stay in registers; the four waves of a workgroup (256 columns)
// walk the same tokens, 64 at a time.  Each wave gathers and splits the patch vectors of one
// strip of 16 of them and leaves the fragments in LDS, so that work is done once for 256
// columns; all loads of a step go out one step ahead.  Column 4 c + j of the 64 goes to lane c
// of MFMA j, so a lane ends up with four consecutive columns of four tokens and 16 neighbouring
// lanes store 256 contiguous bytes of a row straight from the accumulators.  (With the operands
// the other way round, neighbouring lanes storing 16 bytes to different rows, the L1 took a line
// per lane: half the speed.)  The weights come through a slab of LDS for the same reason.
// 17,776 x 1,920: 43 us (208 MB, 4.9 TB/s), 62 before; 17,776 x 3,072: 57 us (5.7 TB/s), 91;
// 3,704 x 1,152: 10.4 us, 18.  Before, a workgroup staged W in LDS for 256 tokens x 128 columns;
// 1,035 of them on 512 slots took a third round for eleven, and the text rows were copied by a
// launch of their own.
//
// fp32 model: v_mfma_f32_16x16x4_f32, 16 tokens x 32 columns a wave; calls of a few hundred
// tokens, bound by launches and one chain of loads and 32 MFMAs.  256 tokens x 256: 4.9 us for what
// took 2.9 + 3.8 + 1.5 in three launches (a sample of ten steps 973 -> 867 us).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "internal.h"

namespace dc {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2u __attribute__((ext_vector_type(2), aligned(4)));   // two floats at any element

constexpr int kStrip = 16;          // tokens per strip
constexpr int kCols = 64;           // columns per wave
constexpr int kPeWaves = 4;         // waves per workgroup
constexpr int kPePerCu = 2;         // workgroups per compute unit (three would spill: 50 us at 17,776 x 1,920)

struct PatchGeo {
  int T, Hl, Wl, p, lp, Hp, Wp;     // lp = log2(p)
  int Nv, d, groups;                // groups of kPeWaves * kCols columns
  int steps, run;                   // steps of kPeWaves strips in a sample, and per workgroup
  int items, per_xcd;               // groups x runs, and their share of an XCD
  size_t latent, h_stride;          // elements per sample of x and of h_in
  size_t txt4;                      // 16-byte pieces of a sample's text rows
};

inline bool al16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; }

__device__ inline void split8(const float (&v)[8], bf16x8& hi, bf16x8& lo) {
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const __bf16 h = static_cast<__bf16>(v[e]);
    hi[e] = h;
    lo[e] = static_cast<__bf16>(v[e] - static_cast<float>(h));
  }
}

// Every wave's LDS accesses before it are done; global accesses stay in flight.
__device__ inline void barrier() {
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// V consecutive floats
template <int V>
__device__ inline void load_v(const float* p, float* dst) {
  if constexpr (V == 4) {
    const float4 a = *reinterpret_cast<const float4*>(p);
    dst[0] = a.x; dst[1] = a.y; dst[2] = a.z; dst[3] = a.w;
  } else if constexpr (V == 2) {
    const float2 a = *reinterpret_cast<const float2*>(p);
    dst[0] = a.x; dst[1] = a.y;
  } else {
    dst[0] = p[0];
  }
}

// V = patch-vector entries that lie next to each other in the latent and are read at once
template <int V>
__global__ void __launch_bounds__(kPeWaves * 64, kPePerCu)
k_patch_embed_bf16(const float* __restrict__ x, const float* __restrict__ W, const float* __restrict__ bias,
                   const uint16_t* __restrict__ pos, const float4* __restrict__ txt, float* __restrict__ out,
                   IdxList idx, PatchGeo g) {
  // the weights' slab of each wave, then the fragments of two steps: [2][strip][xh, xo][lane]
  __shared__ float4 lds[kPeWaves * kCols * 8];
  const int b = idx.v[blockIdx.y];
  float* const ob = out + size_t(b) * g.h_stride;
  if (int(blockIdx.x) >= 8 * g.per_xcd) {        // the workgroups past the strips copy the text rows
    const size_t i = size_t(blockIdx.x - 8 * g.per_xcd) * (kPeWaves * 64) + threadIdx.x;
    float4* dst = reinterpret_cast<float4*>(ob + size_t(g.Nv) * g.d);
    if (i < g.txt4) dst[i] = txt[size_t(b) * g.txt4 + i];
    return;
  }
  // each XCD takes a contiguous range of tokens with all of their columns
  const int item = (blockIdx.x & 7) * g.per_xcd + (blockIdx.x >> 3);
  if (item >= g.items) return;
  const int lane = threadIdx.x & 63, c16 = lane & 15, g4 = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int n = ((item % g.groups) * kPeWaves + wave) * kCols;
  const bool active = n < g.d;                   // the last group may have fewer columns
  const int n0 = active ? n : 0;
  const int s0 = (item / g.groups) * g.run, s1 = min(s0 + g.run, g.steps);
  const float* const xb = x + size_t(b) * g.latent;

  // entry q of a patch vector: channel q >> 2 lp, pixel ((q >> lp) % p, q % p).  Entry
  // 32 kk + 8 g4 + e of a token: the three parts have disjoint bits, so their offsets add up.
  auto entry = [&](int q) {
    const int c = q >> (2 * g.lp), a = (q >> g.lp) & (g.p - 1), bb = q & (g.p - 1);
    return (size_t(c) * g.T * g.Hl + a) * g.Wl + bb;
  };
  const float* const xl = xb + entry(8 * g4);
  auto gather = [&](int s, float (&v)[2][8]) {  // this wave's strip of step s
    const int m = min(kStrip * (kPeWaves * s + wave) + c16, g.Nv - 1);
    const int row = m / g.Wp, j = m - row * g.Wp, t = row / g.Hp, i = row - t * g.Hp;
    const float* px = xl + (size_t(t) * g.Hl + g.p * i) * g.Wl + g.p * j;
#pragma unroll
    for (int kk = 0; kk < 2; ++kk)
#pragma unroll
      for (int e = 0; e < 8; e += V) {
        load_v<V>(px + entry(32 * kk + e), &v[kk][e]);
        if (V == 1 && e % 4 == 3) __builtin_amdgcn_sched_barrier(0);   // 16 live addresses would spill
      }
  };
  // this lane's columns n0 + 4 c16 .. + 3 of the tokens 4 g4 + i of strip q
  const int nc = n0 + 4 * c16;
  // (element offset from strip q's first token, whose row is uniform; rows past the last token
  // are clamped to it: t0 >= N_v in strips that lie past it altogether)
  auto first = [&](int s, int q) { return min(kStrip * (kPeWaves * s + q), g.Nv - 1); };
  auto row_off = [&](int t0, int i) { return uint32_t(min(4 * g4 + i, g.Nv - 1 - t0) * g.d + nc); };
  auto load_pos = [&](int s, int q, uint2 (&pv)[4]) {
    const int t0 = first(s, q);
    const uint16_t* r = pos + size_t(t0) * g.d;
#pragma unroll
    for (int i = 0; i < 4; ++i) pv[i] = *reinterpret_cast<const uint2*>(r + row_off(t0, i));
  };
  float v[2][8];
  uint2 pv[kPeWaves][4];
  gather(s0, v);
#pragma unroll
  for (int q = 0; q < kPeWaves; ++q) load_pos(s0, q, pv[q]);
  const float4 bv = *reinterpret_cast<const float4*>(bias + nc);

  // W[n0 .. n0 + 64)[0 .. 64): half of the rows' columns at a time through the wave's slab, the
  // eight 16-byte pieces of a half row XOR-swizzled; fragment nt takes row 4 c16 + nt
  bf16x8 wh[4][2], wl[4][2];
  {
    float4* const slab = lds + wave * kCols * 8;
    float4 w[2][8];
#pragma unroll
    for (int kk = 0; kk < 2; ++kk)
#pragma unroll
      for (int i = 0; i < 8; ++i)
        w[kk][i] = *reinterpret_cast<const float4*>(W + size_t(n0 + 8 * i + (lane >> 3)) * 64 + 32 * kk + 4 * (lane & 7));
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) {
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const int row = 8 * i + (lane >> 3);
        slab[row * 8 + ((lane & 7) ^ ((row >> 2) & 7))] = w[kk][i];
      }
#pragma unroll
      for (int nt = 0; nt < 4; ++nt) {
        const int row = 4 * c16 + nt;
        const float4 a = slab[row * 8 + ((2 * g4) ^ (c16 & 7))], c = slab[row * 8 + ((2 * g4 + 1) ^ (c16 & 7))];
        const float f[8] = {a.x, a.y, a.z, a.w, c.x, c.y, c.z, c.w};
        split8(f, wh[nt][kk], wl[nt][kk]);
      }
    }
  }

  bf16x8* const frag = reinterpret_cast<bf16x8*>(lds);
  auto step = [&](int s, auto computes) {
    bf16x8* const mine = frag + ((s & 1) * kPeWaves + wave) * 256 + lane;
    bf16x8 fh, fl;
    if (s == s0) barrier();                      // every wave has read its slab
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) {
      split8(v[kk], fh, fl);
      mine[128 * kk] = fh;
      mine[128 * kk + 64] = fl;
    }
    const int sn = min(s + 1, s1 - 1);           // past the run: re-reads the last step
    gather(sn, v);
    barrier();                                   // (the other half of lds is read until the next one)
    if constexpr (!decltype(computes)::value) return;
#pragma unroll
    for (int q = 0; q < kPeWaves; ++q) {
      const bf16x8* const f = frag + ((s & 1) * kPeWaves + q) * 256 + lane;
      f32x4 acc[4];
      acc[0] = f32x4{bv.x, bv.x, bv.x, bv.x};
      acc[1] = f32x4{bv.y, bv.y, bv.y, bv.y};
      acc[2] = f32x4{bv.z, bv.z, bv.z, bv.z};
      acc[3] = f32x4{bv.w, bv.w, bv.w, bv.w};
#pragma unroll
      for (int kk = 0; kk < 2; ++kk) {
        const bf16x8 xh = f[128 * kk], xo = f[128 * kk + 64];
#pragma unroll
        for (int nt = 0; nt < 4; ++nt) acc[nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xh, wl[nt][kk], acc[nt], 0, 0, 0);
#pragma unroll
        for (int nt = 0; nt < 4; ++nt) acc[nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xo, wh[nt][kk], acc[nt], 0, 0, 0);
#pragma unroll
        for (int nt = 0; nt < 4; ++nt) acc[nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xh, wh[nt][kk], acc[nt], 0, 0, 0);
      }
      float4 o[4];
#pragma unroll
      for (int i = 0; i < 4; ++i)
        o[i] = make_float4(acc[0][i] + __uint_as_float(pv[q][i].x << 16), acc[1][i] + __uint_as_float(pv[q][i].x & 0xFFFF0000u),
                           acc[2][i] + __uint_as_float(pv[q][i].y << 16), acc[3][i] + __uint_as_float(pv[q][i].y & 0xFFFF0000u));
      load_pos(sn, q, pv[q]);
      // Rows past the last token hold that token's values and store them again: without a
      // branch around the stores, the waits for the next step's loads leave them in flight.
      // (A strip that lies past it altogether holds the last token in every row.)
      const int t0 = first(s, q);
      float* const orow = ob + size_t(t0) * g.d;
#pragma unroll
      for (int i = 0; i < 4; ++i) *reinterpret_cast<float4*>(orow + row_off(t0, i)) = o[i];
    }
  };
  if (active)
    for (int s = s0; s < s1; ++s) step(s, std::true_type{});
  else
    for (int s = s0; s < s1; ++s) step(s, std::false_type{});
}

// Lane (c16, g4) holds the entries 16 g4 + e (e < 16) of token c16 and of its two weight rows;
// MFMA step e takes entry e on both sides.  Two chains of sums per tile.
template <int V>
__global__ void __launch_bounds__(kPeWaves * 64)
k_patch_embed_f32(const float* __restrict__ x, const float* __restrict__ W, const float* __restrict__ bias,
                  const float* __restrict__ pos, const float4* __restrict__ txt, float* __restrict__ out,
                  IdxList idx, PatchGeo g) {
  const int b = idx.v[blockIdx.y];
  float* const ob = out + size_t(b) * g.h_stride;
  if (int(blockIdx.x) >= g.items) {              // the workgroups past the strips copy the text rows
    const size_t i = size_t(blockIdx.x - g.items) * (kPeWaves * 64) + threadIdx.x;
    float4* dst = reinterpret_cast<float4*>(ob + size_t(g.Nv) * g.d);
    if (i < g.txt4) dst[i] = txt[size_t(b) * g.txt4 + i];
    return;
  }
  const int lane = threadIdx.x & 63, c16 = lane & 15, g4 = lane >> 4, wave = threadIdx.x >> 6;
  const int t0 = int(blockIdx.x) / g.groups * kStrip;
  const int nc = (int(blockIdx.x) % g.groups * kPeWaves + wave) * 32 + 2 * c16;   // two columns per lane
  auto entry = [&](int q) {
    const int c = q >> (2 * g.lp), a = (q >> g.lp) & (g.p - 1), bb = q & (g.p - 1);
    return (size_t(c) * g.T * g.Hl + a) * g.Wl + bb;
  };
  const int m = min(t0 + c16, g.Nv - 1);
  const int row = m / g.Wp, j = m - row * g.Wp, t = row / g.Hp, i = row - t * g.Hp;
  const float* px = x + size_t(b) * g.latent + entry(16 * g4) + (size_t(t) * g.Hl + g.p * i) * g.Wl + g.p * j;
  float v[16], w[2][16];
#pragma unroll
  for (int e = 0; e < 16; e += V) load_v<V>(px + entry(e), &v[e]);
#pragma unroll
  for (int k = 0; k < 2; ++k)
#pragma unroll
    for (int e = 0; e < 16; e += 4) load_v<4>(W + size_t(nc + k) * 64 + 16 * g4 + e, &w[k][e]);
  f32x2u pv[4];
#pragma unroll
  for (int r = 0; r < 4; ++r)
    pv[r] = *reinterpret_cast<const f32x2u*>(pos + size_t(min(t0 + 4 * g4 + r, g.Nv - 1)) * g.d + nc);
  const f32x2u bv = *reinterpret_cast<const f32x2u*>(bias + nc);
  f32x4 acc[2][2];
#pragma unroll
  for (int k = 0; k < 2; ++k) acc[k][0] = acc[k][1] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int e = 0; e < 16; ++e)
#pragma unroll
    for (int k = 0; k < 2; ++k)
      acc[k][e & 1] = __builtin_amdgcn_mfma_f32_16x16x4f32(v[e], w[k][e], acc[k][e & 1], 0, 0, 0);
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int mr = t0 + 4 * g4 + r;
    if (mr < g.Nv)
      *reinterpret_cast<f32x2u*>(ob + size_t(mr) * g.d + nc) =
          f32x2u{((acc[0][0][r] + acc[0][1][r]) + bv.x) + pv[r].x, ((acc[1][0][r] + acc[1][1][r]) + bv.y) + pv[r].y};
  }
}

// what both kernels take of the geometry, and how many floats of the latent are read at once:
// its rows are multiples of the patch long, so a patch's row starts at a multiple of 4 * p
// bytes from the base; a base that is aligned to less is read an element at a time
PatchGeo patch_geo(const Geo& g, int lp) {
  PatchGeo pg{};
  pg.T = g.T; pg.Hl = g.Hl; pg.Wl = g.Wl; pg.p = g.p; pg.lp = lp; pg.Hp = g.Hp; pg.Wp = g.Wp;
  pg.Nv = g.Nv; pg.d = g.d;
  pg.latent = size_t(g.C) * g.T * g.Hl * g.Wl;
  pg.h_stride = size_t(g.N) * g.d;
  pg.txt4 = size_t(g.Nt) * g.d / 4;
  return pg;
}
int vector_width(const Geo& g, const float* x) {
  const uintptr_t base = reinterpret_cast<uintptr_t>(x);
  return g.p >= 4 && base % 16 == 0 ? 4 : g.p >= 2 && base % 8 == 0 ? 2 : 1;
}

}  // namespace

Status patch_embed_f32(const float* x, const float* W, const float* bias, const float* pos, const float* txt,
                       float* out, const IdxList& idx, const Geo& g, hipStream_t s) {
  if (idx.n <= 0 || g.N <= 0) return Status::ok();
  int lp = 0;
  while ((1 << lp) < g.p) ++lp;
  if ((1 << lp) != g.p || g.P != 64 || g.d % 128)
    return Status::shape("fp32 patch embedding needs 64-entry patches, a power-of-two patch, d % 128 == 0");
  PatchGeo pg = patch_geo(g, lp);
  pg.groups = g.d / (kPeWaves * 32);
  pg.items = (g.Nv + kStrip - 1) / kStrip * pg.groups;
  const dim3 grid(unsigned(pg.items + (pg.txt4 + kPeWaves * 64 - 1) / (kPeWaves * 64)), unsigned(idx.n));
  const float4* t4 = reinterpret_cast<const float4*>(txt);
  switch (vector_width(g, x)) {
    case 4: hipLaunchKernelGGL(k_patch_embed_f32<4>, grid, dim3(kPeWaves * 64), 0, s, x, W, bias, pos, t4, out, idx, pg); break;
    case 2: hipLaunchKernelGGL(k_patch_embed_f32<2>, grid, dim3(kPeWaves * 64), 0, s, x, W, bias, pos, t4, out, idx, pg); break;
    default: hipLaunchKernelGGL(k_patch_embed_f32<1>, grid, dim3(kPeWaves * 64), 0, s, x, W, bias, pos, t4, out, idx, pg);
  }
  DC_HIP(hipGetLastError());
  return Status::ok();
}

Status patch_embed_bf16(const float* x, const float* W, const float* bias, const uint16_t* pos, const float* txt,
                        float* out, const IdxList& idx, const Geo& g, hipStream_t s) {
  if (idx.n <= 0 || g.N <= 0) return Status::ok();
  if (g.P != 64 || g.d % 128) return Status::shape("bf16 patch embedding needs 64-entry patches, d % 128 == 0");
  int lp = 0;
  while ((1 << lp) < g.p) ++lp;
  if ((1 << lp) != g.p) return Status::shape("bf16 patch embedding needs a power-of-two patch");
  if (!al16(out) || !al16(bias) || !al16(pos) || !al16(W))
    return Status::arg("bf16 patch embedding needs 16-byte aligned device buffers");
  const int cus = compute_units();
  if (cus <= 0) return Status::make(DC_ERR_HIP, "bf16 patch embedding: no device");
  PatchGeo pg = patch_geo(g, lp);
  pg.groups = (g.d + kPeWaves * kCols - 1) / (kPeWaves * kCols);
  pg.steps = (g.Nv + kStrip * kPeWaves - 1) / (kStrip * kPeWaves);
  // about as many workgroups as are resident at once, since W is read once per run (runs that do
  // not divide a sample's steps, and the text rows, can make it a few more)
  const int64_t work = int64_t(pg.steps) * pg.groups * idx.n;
  pg.run = std::max(1, int((work + kPePerCu * cus - 1) / (kPePerCu * cus)));   // (no video tokens: no steps)
  pg.items = pg.groups * ((pg.steps + pg.run - 1) / pg.run);
  pg.per_xcd = (pg.items + 7) / 8;
  const dim3 grid(unsigned(8 * pg.per_xcd + (pg.txt4 + kPeWaves * 64 - 1) / (kPeWaves * 64)), unsigned(idx.n));
  const float4* t4 = reinterpret_cast<const float4*>(txt);
  switch (vector_width(g, x)) {
    case 4: hipLaunchKernelGGL(k_patch_embed_bf16<4>, grid, dim3(kPeWaves * 64), 0, s, x, W, bias, pos, t4, out, idx, pg); break;
    case 2: hipLaunchKernelGGL(k_patch_embed_bf16<2>, grid, dim3(kPeWaves * 64), 0, s, x, W, bias, pos, t4, out, idx, pg); break;
    default: hipLaunchKernelGGL(k_patch_embed_bf16<1>, grid, dim3(kPeWaves * 64), 0, s, x, W, bias, pos, t4, out, idx, pg);
  }
  DC_HIP(hipGetLastError());
  return Status::ok();
}

}  // namespace dc
