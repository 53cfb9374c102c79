// Internal declarations shared by the library's host and device sources.
#pragma once

#include <cstdint>
#include <string>
#include <vector>

#include <hip/hip_runtime.h>

#include "../../include/dc.h"

namespace dc {

// ---------------------------------------------------------------------------
// status
// ---------------------------------------------------------------------------
struct Status {
  dc_status code = DC_OK;
  std::string msg;
  static Status ok() { return {}; }
  static Status make(dc_status c, std::string m) { Status s; s.code = c; s.msg = std::move(m); return s; }
  static Status arg(std::string m) { return make(DC_ERR_ARG, std::move(m)); }
  static Status shape(std::string m) { return make(DC_ERR_SHAPE, std::move(m)); }
  explicit operator bool() const { return code == DC_OK; }
};

Status hip_status(hipError_t e, const char* what);
#define DC_HIP(call)                                              \
  do {                                                            \
    hipError_t e_ = (call);                                       \
    if (e_ != hipSuccess) return ::dc::hip_status(e_, #call);     \
  } while (0)
#define DC_TRY(expr)                        \
  do {                                      \
    ::dc::Status s_ = (expr);               \
    if (!s_) return s_;                     \
  } while (0)

// ---------------------------------------------------------------------------
// host schedule (sched.cpp)
// ---------------------------------------------------------------------------
struct SceneTables {
  int K = 0, H = 0;
  double L = 0, Theta = 0, zL = 0, zTh = 0, D = 0;
  bool in_support = false;
  std::vector<int64_t> chat;   // [(K-1) * H], 2^-40 units
  std::vector<double> dbar;    // [(K-1) * H]
  int64_t cost(int j, int h) const { return chat[size_t(j - 1) * H + (h - 1)]; }
  double threshold(int j, int h) const { return dbar[size_t(j - 1) * H + (h - 1)]; }
};
Status validate_problem(const dc_sched_problem& p);
Status scene_tables(const dc_sched_problem& p, SceneTables& t);
Status schedule(const dc_sched_problem& p, const SceneTables& t, std::vector<uint8_t>& reuse,
                int32_t& n_reuse, int64_t& cost_q);
Status select_tau(const dc_sched_problem* probs, int n, double rho, int64_t& tau);
void motion_statistics(const double* xy, const double* yaw, int n_pose, double& L, double& Th);
Status select_anchors(const double* L, const double* Th, int n, double eps, int& i0, int& i1);

// ---------------------------------------------------------------------------
// model geometry
// ---------------------------------------------------------------------------
struct Geo {
  int L, d, H, Dh, F, C, T, Hl, Wl, p, Hp, Wp, Nv, Nt, N, P;
  bool bf16;
  float eps;
  size_t esz;            // bytes per element of the model dtype
};
Status make_geo(const dc_model_cfg* cfg, Geo& g);

// Kernel classes that can be timed (dc_profile_*); the numbering is part of the ABI.
enum class KClass { kAttention = 0, kGemmQKV, kGemmOut, kGemmUp, kGemmDown, kLnModulate,
                    kPatchEmbed, kDrift, kCacheStore, kCacheApply, kHead, kHeadReuse, kCount };

// RAII: brackets the launches made in its scope with events when the class is enabled.
class ProfScope {
 public:
  ProfScope(KClass c, hipStream_t s);
  ~ProfScope();
  ProfScope(const ProfScope&) = delete;
  ProfScope& operator=(const ProfScope&) = delete;

 private:
  int cls_;
  hipStream_t stream_;
  hipEvent_t start_ = nullptr;
};

// Selected samples of a batch, passed to kernels by value.
struct IdxList {
  int32_t n;
  int32_t v[DC_MAX_BATCH];
};
Status make_idx(const int32_t* idx, int32_t n, IdxList& out);

// Workspace layout (offsets in bytes, each 256-aligned).
struct Workspace {
  size_t a, qk, vt, o, ff, drift_part, attn_part, attn_part_bytes, tm_e, tm_h, tm_c, tm_s, tm_m, total;
  int ldv;               // row stride of the transposed value buffer (tokens, padded)
};
Workspace workspace_layout(const Geo& g, int batch);

// split-tail partials of the bf16 attention: up to 64 split items per XCD, two halves of
// 128 queries x (head_dim + 4) floats each
inline size_t attn_part_bytes(int head_dim) { return size_t(8) * 64 * 2 * 128 * (head_dim + 4) * sizeof(float); }

constexpr int kModSteps = 64;       // denoising steps per pass of the modulation
constexpr int kDriftBlocks = 1024;  // fixed grid per sample: reproducible reductions

// Compute units of the current device (looked up once per device); 0 if there is none.
int compute_units();

// ---------------------------------------------------------------------------
// kernel launchers (kernels_*.hip, gemm.hip, attention.hip)
// ---------------------------------------------------------------------------
enum class Act { kNone, kSilu };

// fp32 GEMM, C = A W^T (+ epilogue).  A [M, K] (lda), W [N, K] (ldw); K % 64 == 0.
Status gemm_f32_bias_act(const float* A, int lda, const float* W, int ldw, const float* bias,
                         float* out, int ldo, int M, int N, int K, Act act, hipStream_t s);
// out = A W^T + bias and silu_out = SiLU(out)
Status gemm_f32_bias_and_silu(const float* A, int lda, const float* W, int ldw, const float* bias,
                              float* out, float* silu_out, int ldo, int M, int N, int K, hipStream_t s);
Status gemm_f32_gate_residual(const float* A, int lda, const float* W, int ldw, const float* bias,
                              const float* gate, float* h, int ldh, int M, int N, int K,
                              hipStream_t s);
Status gemm_f32_gelu(const float* A, int lda, const float* W, int ldw, const float* bias,
                     float* out, int ldo, int M, int N, int K, hipStream_t s);
Status gemm_f32_head(const float* A, int lda, const float* W, const float* bias, float* x,
                     float dsigma, const Geo& g, int M, hipStream_t s);
// The calibration's GEMMs: rows from bias_rows on (tangents stacked below a primal activation)
// get no bias; weights fp32, or bf16 (w_bf16) widened exactly on load.
Status gemm_f32_rows(const float* A, int lda, const void* W, bool w_bf16, int ldw, const float* bias,
                     int bias_rows, float* out, int ldo, int M, int N, int K, hipStream_t s);
Status gemm_f32_gate_residual_rows(const float* A, int lda, const void* W, bool w_bf16, int ldw,
                                   const float* bias, int bias_rows, const float* gate, float* h, int ldh,
                                   int M, int N, int K, hipStream_t s);
// n tangents da [n, N, d] through the head: x [n, latent] += dsigma unpatchify(da[:, :Nv] W^T)
Status gemm_f32_head_tangents(const float* A, const void* W, bool w_bf16, float* x, float dsigma,
                              const Geo& g, int n, hipStream_t s);

// bf16 MFMA GEMM variants.  block_gemm_tile: which of its six tiles a call takes (gemm.hip, kTiles).
int block_gemm_tile(int M, int N, int K, int cus);
Status gemm_bf16_qkv(const uint16_t* A, const uint16_t* W, const float* bias, uint16_t* qk,
                     uint16_t* vt, int ldv, const Geo& g, int M, hipStream_t s);
Status gemm_bf16_gate_residual(const uint16_t* A, int lda, const uint16_t* W, const float* bias,
                               const float* gate, float* h, int ldh, int M, int N, int K,
                               hipStream_t s);
Status gemm_bf16_gelu(const uint16_t* A, int lda, const uint16_t* W, const float* bias,
                      uint16_t* out, int ldo, int M, int N, int K, hipStream_t s);
// h_in of the samples idx: patchify + patch embedding + bias + positions, and the text rows
// (patch_embed.hip).
Status patch_embed_bf16(const float* x, const float* W, const float* bias, const uint16_t* pos, const float* txt,
                        float* out, const IdxList& idx, const Geo& g, hipStream_t s);
Status patch_embed_f32(const float* x, const float* W, const float* bias, const float* pos, const float* txt,
                       float* out, const IdxList& idx, const Geo& g, hipStream_t s);
// bf16 model: LN-modulation + head projection + unpatchify + Euler update of one sample's
// latent in one pass over its N_v video rows of g (head.hip).  With resid != NULL the input
// is g = gin + resid (bf16), formed in registers (reuse steps); head_takes_resid says whether
// the model's width allows that.
bool head_takes_resid(const Geo& g);
Status head_euler_bf16(const float* gin, const uint16_t* resid, const uint16_t* W, const float* bias,
                       const float* shift, const float* scale, float* x, float dsigma, const Geo& g,
                       hipStream_t s);

// Attention over one sample: qk [M, 2d] (Q | K), vt [heads][Dh][ldv], out [M, d].
// part: scratch for the split tail items (unnormalised partial outputs), part_bytes its size;
// with too little scratch the tail is not split.
Status attention_bf16(const uint16_t* qk, const uint16_t* vt, int ldv, uint16_t* out,
                      const Geo& g, int M, float* part, size_t part_bytes, hipStream_t s);
// Which of its kernels that call takes, and whether items of its last round are split (with the
// scratch of a workspace; false without a device).
enum class AttnKernel { kKeys, kBf16, k16 };
AttnKernel attention_kernel(int head_dim, int heads, int tokens, int cus);
bool attention_splits(int head_dim, int heads, int tokens);
// fp32 attention over qkv [M, 3d] (Q | K | V), out [M, d] (attention_f32.hip).
Status attention_f32(const float* qkv, float* out, const Geo& g, int M, hipStream_t s);

// Elementwise / row kernels.
Status ln_modulate(const float* x, int rows, int ldx, const float* shift, const float* scale,
                   void* out, int ldo, bool out_bf16, const Geo& g, hipStream_t s);
Status cache_store(const float* h_out, const float* h_in, void* resid, const IdxList& idx,
                   const Geo& g, hipStream_t s);
Status cache_apply(const float* h_in, const void* resid, float* gout, const IdxList& idx,
                   const Geo& g, hipStream_t s);
Status drift(const float* h_in, const float* mod0, void* u_ref, bool snapshot, double* sums,
             const IdxList& idx, const Geo& g, double* part, hipStream_t s);
// drift() with the partial sums in the library's fixed per-GPU scratch array (no workspace)
Status drift_noalloc(const float* h_in, const float* mod0, void* u_ref, bool snapshot, double* sums,
                     const IdxList& idx, const Geo& g, hipStream_t s);

// Anchor calibration (Eq. 5-7): tangent-mode kernels of the fp32 network (calib.hip) and the
// driver (calib.cpp).  Activations are stacked: the primal [rows], then n tangents [rows] each.
constexpr int kMaxTangents = 32;
// per row of the stack [1 + n, rows, d]: a = LN(x)(1+scale)+shift and its n tangents
Status ln_mod_jvp(const float* x, int n, int rows, int d, const float* shift, const float* scale, float* a,
                  float eps, hipStream_t s);
// qkv [1 + n, M, 3d] -> o [1 + n, M, d]: attention and its n tangents (attention_f32.hip)
Status attention_jvp_f32(const float* qkv, int n, const Geo& g, int M, float* o, hipStream_t s);
// z [1 + n, count] <- GELU(z) and its n tangents
Status gelu_jvp(float* z, int n, size_t count, hipStream_t s);
// patches [n, N, 64] of n latents dx (text rows zero)
Status patchify_tangents(const float* dx, float* patches, const Geo& g, int n, hipStream_t s);
// out[i] [Nv, d] (stride `stride`) = x + r[i], i < n <= kMaxTangents + 1; r: host array of device pointers
Status add_each(const float* x, const float* const* r, int n, size_t count, float* out, size_t stride,
                hipStream_t s);
// out = alpha x + beta y
Status lincomb(float* out, const float* x, float alpha, const float* y, float beta, size_t n,
               hipStream_t s);
// out = alpha (x - y)
Status scaled_diff(float* out, const float* x, const float* y, float alpha, size_t n, hipStream_t s);
// out2[i] = (sum (a[i]-b[i])^2, sum a[i]^2) for i < count (b[i] may be NULL) in a fixed order, with
// sumsq_scratch_doubles() doubles of scratch; a, b: host arrays of device pointers
size_t sumsq_scratch_doubles();
Status sumsq(const float* const* a, const float* const* b, int count, size_t n, double* scratch, double* out2,
             hipStream_t s);
size_t calibrate_workspace_bytes(const Geo& g, int K);
Status calibrate_tables(const Geo& g, const dc_model_weights* w, const float* x1, const float* txt,
                        const double* sigmas, int K, int h_max, double eps, double* q, double* dtab,
                        void* ws, size_t ws_bytes, hipStream_t s);
Status copy_rows(const float* src, float* dst, size_t count, hipStream_t s);
// e [K, n_freq] from the host noise levels (K <= kModSteps)
Status time_features(const double* sig, int K, float* e, int n_freq, hipStream_t s);
// mod [K, L+1, 6, d] from m [K, 6, d], c [K, d], the L per-block offsets (host array of device
// pointers) and the head's offset
Status assemble_modulation(const float* m, const float* c, const float* const* offsets,
                           const float* head_mod, int K, const Geo& g, float* mod, hipStream_t s);

}  // namespace dc
