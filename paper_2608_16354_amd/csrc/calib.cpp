// Anchor calibration of the run tables on the GPU (Sec. 3.1 after Eq. 4; Eq. 5-7).
//
// For one anchor clip the full (uncached) denoising trace stores, per step k, the latent
// x_k the step starts from, the backbone input u_k (block 0's modulated input of the
// video rows) and the backbone output r_k = h_out - h_in over the video rows.  For a run
// that refreshes at step j and reuses r_j for h steps:
//   Eq. 5  d_{j,h} = ||u_{j+h} - u_j||_2 / (||u_{j+h}||_2 + eps);
//   Eq. 6  e_{j,l} = H_{j+l}(x_{j+l}, r_j) - H_{j+l}(x_{j+l}, r_{j+l}), H_k(x, r) the
//          denoiser output of the head for g = h_in(x)[video] + r;
//   Eq. 7  G_{j,h} = sum_{l <= h} P_{j+l} e_{j,l},  q_{j,h} = ||G_{j,h}||_2 / (||x_out||_2 + eps),
//          with P_t e the tangent of the terminal latent when the denoiser output of step
//          t moves by e: dx = (sigma_{t+1} - sigma_t) e, then for every later step k
//          dx += (sigma_{k+1} - sigma_k) J_k dx, J_k the Jacobian of the full network at
//          x_k (a Jacobian-vector product: the network run in tangent mode).
// J_k does not depend on the perturbation, so the runs are taken in groups of up to T tangents
// (ordered by t = j + h) that go through the steps together: one network pass per step
// carries the primal activations and every active tangent of the group, stacked as rows of the
// same GEMMs.  T fills about 4,096 rows; one tangent at a time (the small fp32 model: 64 passes
// of the network with its tangent, 2,900 launches, a wait per norm) took 15.5 ms, the groups
// take 3.7 ms.  The norms are read back once, at the end.
// Runs with j + h > K price nothing and stay 0.  The trace runs the library's own
// kernels for the model's dtype (bf16 models: bf16 MFMA blocks); r, u, the perturbations
// and every tangent are fp32 (calib.hip and the fp32 GEMMs, with bf16 weights widened
// exactly on load).
#include <algorithm>
#include <cmath>

#include "internal.h"

namespace dc {

Status time_modulation(const Geo& g, const dc_model_weights* w, const double* sigmas, int K,
                       float* mod, void* ws, size_t ws_bytes, hipStream_t s);
Status patch_embed(const Geo& g, const dc_model_weights* w, const float* x, const float* txt,
                   float* h_in, const IdxList& il, void* ws, size_t ws_bytes, hipStream_t s);
Status block_forward(const Geo& g, const dc_block_weights* bw, const float* mod, float* h,
                     const IdxList& il, void* ws, size_t ws_bytes, hipStream_t s);
Status head_euler(const Geo& g, const dc_model_weights* w, const float* head_mod, const float* gin,
                  float* x, float dsigma, const IdxList& il, void* ws, size_t ws_bytes,
                  hipStream_t s, const void* resid);

namespace {

inline size_t al256(size_t v) { return (v + 255) & ~size_t(255); }

struct CalibLayout {
  size_t blk, blk_bytes, mod, xs, us, rs, h_in, h, a, qkv, o, z, patches, v, dx, G, red, norms, total;
  int T;                 // tangents per group
};

// one (j, h) entry: a run refreshed at j, perturbed at step t = j + h
struct Run { int j, h, t; };

inline int max_runs(int K) { return K * (K - 1) / 2; }    // j + h <= K, any h_max

CalibLayout calib_layout(const Geo& g, int K) {
  CalibLayout c{};
  size_t off = 0;
  auto take = [&](size_t bytes) { const size_t o = off; off = al256(off + bytes); return o; };
  const size_t N = size_t(g.N), Nv = size_t(g.Nv), d = size_t(g.d), F = size_t(g.F);
  const size_t lat = size_t(g.C) * g.T * g.Hl * g.Wl;
  c.T = std::max(1, std::min(kMaxTangents, 4096 / std::max(1, g.N)));     // (a model may have no token)
  const size_t R = size_t(c.T + 1) * N;            // rows of a stack: the primal and T tangents
  c.blk_bytes = workspace_layout(g, 1).total;
  c.blk = take(c.blk_bytes);
  c.mod = take(size_t(K) * (g.L + 1) * 6 * d * 4);
  c.xs = take(size_t(K + 1) * lat * 4);
  c.us = take(size_t(K) * Nv * d * 4);
  c.rs = take(size_t(K) * Nv * d * 4);
  c.h_in = take(N * d * 4);
  c.h = take(R * d * 4);
  c.a = take(R * d * 4);
  c.qkv = take(R * 3 * d * 4);
  c.o = take(R * d * 4);
  c.z = take(R * F * 4);
  c.patches = take(size_t(c.T) * N * 64 * 4);
  c.v = take(size_t(c.T + 1) * lat * 4);
  c.dx = take(size_t(c.T) * lat * 4);
  c.G = take(size_t(K) * lat * 4);
  c.red = take(sumsq_scratch_doubles() * 8);
  c.norms = take((2 * size_t(max_runs(K)) + 1) * 2 * 8);
  c.total = off;
  return c;
}

template <class T> T* at(void* base, size_t off) {
  return reinterpret_cast<T*>(static_cast<char*>(base) + off);
}

struct Calib {
  const Geo& g;
  const dc_model_weights* w;
  const float* txt;
  const double* sig;
  int K;
  void* ws;
  CalibLayout L;
  hipStream_t s;
  IdxList one;
  size_t lat, mstride;

  void* blk() const { return at<void>(ws, L.blk); }
  float* F(size_t off) const { return at<float>(ws, off); }
  const float* mod_k(int k) const { return F(L.mod) + size_t(k - 1) * mstride; }
  float* x_at(int k) const { return F(L.xs) + size_t(k - 1) * lat; }        // x_k, k = 1..K+1
  float* u_at(int k) const { return F(L.us) + size_t(k - 1) * g.Nv * g.d; }
  float* r_at(int k) const { return F(L.rs) + size_t(k - 1) * g.Nv * g.d; }
  float* G_at(int j) const { return F(L.G) + size_t(j - 1) * lat; }         // sum of P e over the run
  float* dx_at(int i) const { return F(L.dx) + size_t(i) * lat; }           // tangent i of the group
  float dsig(int k) const { return float(sig[k] - sig[k - 1]); }            // step k: sigma_{k+1} - sigma_k

  // full trace: x_1..x_{K+1}, u_k, r_k
  Status trace(const float* x1) {
    DC_HIP(hipMemcpyAsync(x_at(1), x1, lat * 4, hipMemcpyDeviceToDevice, s));
    for (int k = 1; k <= K; ++k) {
      const float* mk = mod_k(k);
      DC_TRY(patch_embed(g, w, x_at(k), txt, F(L.h_in), one, blk(), L.blk_bytes, s));
      DC_TRY(ln_modulate(F(L.h_in), g.Nv, g.d, mk, mk + g.d, u_at(k), g.d, false, g, s));
      DC_TRY(copy_rows(F(L.h_in), F(L.h), size_t(g.N) * g.d, s));
      for (int l = 0; l < g.L; ++l)
        DC_TRY(block_forward(g, &w->blocks[l], mk + size_t(l) * 6 * g.d, F(L.h), one, blk(), L.blk_bytes, s));
      DC_TRY(lincomb(r_at(k), F(L.h), 1.0f, F(L.h_in), -1.0f, size_t(g.Nv) * g.d, s));   // r = h_out - h_in
      DC_HIP(hipMemcpyAsync(x_at(k + 1), x_at(k), lat * 4, hipMemcpyDeviceToDevice, s));
      DC_TRY(head_euler(g, w, mk + size_t(g.L) * 6 * g.d, F(L.h), x_at(k + 1), dsig(k), one, blk(),
                        L.blk_bytes, s, nullptr));
    }
    return Status::ok();
  }

  // dx of runs [i0, i1) of the group, all perturbed at step t: the Euler step of Eq. 6's e.
  // H_t(x_t, r) is the head of g = h_in(x_t)[video] + r, as x = 0 + 1 v.
  Status perturb(const Run* runs, int i0, int i1, int t) {
    const float* mt = mod_k(t);
    const int n = i1 - i0;
    const float* r[kMaxTangents + 1];
    for (int i = 0; i < n; ++i) r[i] = r_at(runs[i0 + i].j);
    r[n] = r_at(t);
    DC_TRY(patch_embed(g, w, x_at(t), txt, F(L.h_in), one, blk(), L.blk_bytes, s));
    DC_TRY(add_each(F(L.h_in), r, n + 1, size_t(g.Nv) * g.d, F(L.h), size_t(g.N) * g.d, s));
    DC_HIP(hipMemsetAsync(F(L.v), 0, size_t(n + 1) * lat * 4, s));
    int32_t ids[kMaxTangents + 1];
    for (int i = 0; i <= n; ++i) ids[i] = i;
    IdxList il;
    DC_TRY(make_idx(ids, n + 1, il));
    DC_TRY(head_euler(g, w, mt + size_t(g.L) * 6 * g.d, F(L.h), F(L.v), 1.0f, il, blk(), L.blk_bytes, s, nullptr));
    for (int i = 0; i < n; ++i)
      DC_TRY(scaled_diff(dx_at(i0 + i), F(L.v) + size_t(i) * lat, F(L.v) + size_t(n) * lat, dsig(t), lat, s));
    return Status::ok();
  }

  // one block on the stack h of the primal and n tangents
  Status block_jvp(int l, const float* m6, int n) {
    const dc_block_weights& b = w->blocks[l];
    const int N = g.N, d = g.d, Fh = g.F, R = (n + 1) * N;
    const float *sh1 = m6, *sc1 = m6 + d, *g1 = m6 + 2 * d, *sh2 = m6 + 3 * d, *sc2 = m6 + 4 * d,
                *g2 = m6 + 5 * d;
    DC_TRY(ln_mod_jvp(F(L.h), n, N, d, sh1, sc1, F(L.a), g.eps, s));
    DC_TRY(gemm_f32_rows(F(L.a), d, b.w_qkv, g.bf16, d, b.b_qkv, N, F(L.qkv), 3 * d, R, 3 * d, d, s));
    DC_TRY(attention_jvp_f32(F(L.qkv), n, g, N, F(L.o), s));
    DC_TRY(gemm_f32_gate_residual_rows(F(L.o), d, b.w_o, g.bf16, d, b.b_o, N, g1, F(L.h), d, R, d, d, s));
    DC_TRY(ln_mod_jvp(F(L.h), n, N, d, sh2, sc2, F(L.a), g.eps, s));
    DC_TRY(gemm_f32_rows(F(L.a), d, b.w_1, g.bf16, d, b.b_1, N, F(L.z), Fh, R, Fh, d, s));
    DC_TRY(gelu_jvp(F(L.z), n, size_t(N) * Fh, s));
    return gemm_f32_gate_residual_rows(F(L.z), Fh, b.w_2, g.bf16, Fh, b.b_2, N, g2, F(L.h), d, R, d, Fh, s);
  }

  // dx += (sigma_{k+1} - sigma_k) J_k dx for the first n tangents of the group: the whole
  // network at x_k, primal and tangents
  Status step_jvp(int k, int n) {
    const float* mk = mod_k(k);
    const int d = g.d, N = g.N;
    DC_TRY(patch_embed(g, w, x_at(k), txt, F(L.h), one, blk(), L.blk_bytes, s));
    DC_TRY(patchify_tangents(F(L.dx), F(L.patches), g, n, s));            // text rows carry no tangent
    DC_TRY(gemm_f32_rows(F(L.patches), 64, w->w_pe, false, 64, w->b_pe, 0, F(L.h) + size_t(N) * d, d, n * N, d, 64,
                         s));                                             // (no row gets the bias)
    for (int l = 0; l < g.L; ++l) DC_TRY(block_jvp(l, mk + size_t(l) * 6 * d, n));
    const float* hm = mk + size_t(g.L) * 6 * d;
    DC_TRY(ln_mod_jvp(F(L.h), n, N, d, hm, hm + d, F(L.a), g.eps, s));
    return gemm_f32_head_tangents(F(L.a) + size_t(N) * d, w->w_head, g.bf16, F(L.dx), dsig(k), g, n, s);
  }
};

}  // namespace

size_t calibrate_workspace_bytes(const Geo& g, int K) { return calib_layout(g, K).total; }

Status calibrate_tables(const Geo& g, const dc_model_weights* w, const float* x1, const float* txt,
                        const double* sigmas, int K, int h_max, double eps, double* q, double* dtab,
                        void* ws, size_t ws_bytes, hipStream_t s) {
  if (!w || !x1 || !sigmas || !q || !dtab || !ws || (g.Nt > 0 && !txt)) return Status::arg("NULL argument");
  if (g.Dh != 64) return Status::shape("calibration supports head_dim 64");
  if (K < 2 || h_max < 1) return Status::arg("calibration needs K >= 2 and h_max >= 1");
  if (!(eps >= 0.0)) return Status::arg("eps must be >= 0");
  if (!w->blocks || !w->w_head || !w->b_head || !w->w_pe) return Status::arg("weight pointer is NULL");
  for (int l = 0; l < g.L; ++l)
    if (!w->blocks[l].w_qkv || !w->blocks[l].w_o || !w->blocks[l].w_1 || !w->blocks[l].w_2 ||
        !w->blocks[l].b_qkv || !w->blocks[l].b_o || !w->blocks[l].b_1 || !w->blocks[l].b_2)
      return Status::arg("block weight pointer is NULL");
  const CalibLayout L = calib_layout(g, K);
  if (reinterpret_cast<uintptr_t>(ws) % 256) return Status::make(DC_ERR_WORKSPACE, "workspace must be 256-byte aligned");
  if (ws_bytes < L.total) return Status::make(DC_ERR_WORKSPACE, "calibration workspace too small");
  Calib c{g, w, txt, sigmas, K, ws, L, s, {}, size_t(g.C) * g.T * g.Hl * g.Wl, size_t(g.L + 1) * 6 * g.d};
  const int32_t zero = 0;
  DC_TRY(make_idx(&zero, 1, c.one));
  DC_HIP(hipMemsetAsync(c.F(L.G), 0, size_t(K) * c.lat * 4, s));
  DC_TRY(time_modulation(g, w, sigmas, K, c.F(L.mod), c.blk(), L.blk_bytes, s));
  DC_TRY(c.trace(x1));

  // every run, ordered by the step it is perturbed at (and by h, so the sums of Eq. 7 grow in order)
  std::vector<Run> runs;
  for (int t = 2; t <= K; ++t)
    for (int h = 1; h <= h_max && h < t; ++h) runs.push_back({t - h, h, t});
  const int n_runs = int(runs.size());

  // norms: n_runs of Eq. 5, then n_runs of Eq. 7, then the terminal latent's
  double* norms = at<double>(ws, L.norms);
  {
    std::vector<const float*> a, b;
    for (const Run& r : runs) {
      a.push_back(c.u_at(r.t));
      b.push_back(c.u_at(r.j));
    }
    DC_TRY(sumsq(a.data(), b.data(), n_runs, size_t(g.Nv) * g.d, at<double>(ws, L.red), norms, s));
    const float* out = c.x_at(K + 1);
    DC_TRY(sumsq(&out, nullptr, 1, c.lat, at<double>(ws, L.red), norms + 4 * size_t(n_runs), s));
  }
  for (int g0 = 0; g0 < n_runs; g0 += L.T) {
    const Run* grp = runs.data() + g0;
    const int n = std::min(L.T, n_runs - g0);
    for (int i = 0; i < n;) {
      int e = i + 1;
      while (e < n && grp[e].t == grp[i].t) ++e;
      DC_TRY(c.perturb(grp, i, e, grp[i].t));
      i = e;
    }
    for (int k = grp[0].t + 1, active = 0; k <= K; ++k) {
      while (active < n && grp[active].t < k) ++active;
      DC_TRY(c.step_jvp(k, active));
    }
    for (int i = 0; i < n; ++i) {
      float* G = c.G_at(grp[i].j);                        // G_{j,h} = G_{j,h-1} + P_{j+h} e
      DC_TRY(lincomb(G, G, 1.0f, c.dx_at(i), 1.0f, c.lat, s));
      const float* Gc = G;
      DC_TRY(sumsq(&Gc, nullptr, 1, c.lat, at<double>(ws, L.red), norms + 2 * size_t(n_runs + g0 + i), s));
    }
  }
  std::vector<double> host(2 * (2 * size_t(n_runs) + 1));
  DC_HIP(hipMemcpyAsync(host.data(), norms, host.size() * sizeof(double), hipMemcpyDeviceToHost, s));
  DC_HIP(hipStreamSynchronize(s));

  const size_t T = size_t(K - 1) * h_max;
  std::fill(q, q + T, 0.0);
  std::fill(dtab, dtab + T, 0.0);
  const double xn = std::sqrt(host[4 * size_t(n_runs) + 1]);
  for (int i = 0; i < n_runs; ++i) {
    const size_t e = size_t(runs[size_t(i)].j - 1) * h_max + (runs[size_t(i)].h - 1);
    dtab[e] = std::sqrt(host[2 * size_t(i)]) / (std::sqrt(host[2 * size_t(i) + 1]) + eps);
    q[e] = std::sqrt(host[2 * size_t(n_runs + i) + 1]) / (xn + eps);
  }
  return Status::ok();
}

}  // namespace dc
