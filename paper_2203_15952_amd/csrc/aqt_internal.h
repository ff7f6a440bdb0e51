// Internal declarations shared by the HIP translation units of libaqt.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "aqt.h"

// Per-tile timelines (tracing builds only, -DAQT_TIMELINE; see paper_2203_15952_amd/timeline.py):
// wavefront 0 of every workgroup stamps the shader clock at its phase boundaries and leaves
// eight 64-bit words per workgroup in a device array of the translation unit, which an
// extern "C" accessor copies out.  The product build contains none of this.
#ifdef AQT_TIMELINE
#define AQT_TL_SLOTS (1 << 15)
#define AQT_TL_DECL long long aqt_tl_[5] = {0, 0, 0, 0, 0}
#define AQT_TL(i) aqt_tl_[i] = __builtin_readcyclecounter()
#define AQT_TL_WRITE(buf, tag)                                                        \
  do {                                                                                \
    if ((threadIdx.x & 63) == 0 && (threadIdx.x >> 6) == 0 && blockIdx.x < AQT_TL_SLOTS) { \
      unsigned hw_, xcc_;                                                             \
      asm volatile("s_getreg_b32 %0, hwreg(HW_REG_HW_ID)" : "=s"(hw_));               \
      asm volatile("s_getreg_b32 %0, hwreg(HW_REG_XCC_ID)" : "=s"(xcc_));             \
      long long *o_ = (buf) + static_cast<long long>(blockIdx.x) * 8;                 \
      o_[0] = aqt_tl_[0]; o_[1] = aqt_tl_[1]; o_[2] = aqt_tl_[2]; o_[3] = aqt_tl_[3];  \
      o_[4] = aqt_tl_[4]; o_[5] = hw_; o_[6] = xcc_; o_[7] = (tag);                    \
    }                                                                                 \
  } while (0)
#else
#define AQT_TL_DECL
#define AQT_TL(i)
#define AQT_TL_WRITE(buf, tag)
#endif

namespace aqt {

extern thread_local int g_last_hip_error;

#define AQT_HIP(expr)                                   \
  do {                                                  \
    hipError_t e__ = (expr);                            \
    if (e__ != hipSuccess) {                            \
      aqt::g_last_hip_error = static_cast<int>(e__);    \
      return AQT_ERR_HIP;                               \
    }                                                   \
  } while (0)

#define AQT_TRY(expr)                 \
  do {                                \
    aqt_status s__ = (expr);          \
    if (s__ != AQT_OK) return s__;    \
  } while (0)

constexpr int kMaxPartials = 4096;  // per-block abs-max slots at the head of a quantize workspace
constexpr int kWeightSlabs = 16;    // fan-in slabs whose per-channel maxima the weight quantizer folds

#ifdef __HIPCC__
// What lanes of this wavefront wrote to LDS in front of it, its other lanes may read behind it, and the other way round.  The hardware
// executes a wavefront's LDS operations in order; the fences keep the compiler from exchanging them (the barrier by itself only
// binds its scheduling) and cost no instruction.
__device__ __forceinline__ void wave_lds_order() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}
#endif

// Whether the n bytes at a and the m bytes at b have one in common (a null pointer has none).
inline bool overlap(const void *a, size_t n, const void *b, size_t m) {
  const uintptr_t p = reinterpret_cast<uintptr_t>(a), q = reinterpret_cast<uintptr_t>(b);
  return a && b && p < q + m && q < p + n;
}

inline int qmax_of(int bits) { return (1 << (bits - 1)) - 1; }
inline bool bits_ok(int bits) { return bits >= 2 && bits <= 8; }
inline bool packed4(int bits_w) { return bits_w <= 4; }
inline size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }
__host__ __device__ inline int64_t cdiv(int64_t a, int64_t b) { return (a + b - 1) / b; }

// ---- quantizers (quantize.hip) ------------------------------------------------
aqt_status launch_quantize(const float *x, int64_t rows, int64_t cols, int64_t ldx, int bits, int axis,
                           int8_t *q, float *scale, uint32_t *mask, float *partials, hipStream_t st,
                           int32_t *dev_status);
aqt_status launch_quantize_with_absmax(const float *x, int64_t rows, int64_t cols, int64_t ldx, int bits,
                                       const uint32_t *absmax_bits, int8_t *q, float *scale, uint32_t *mask,
                                       hipStream_t st, int32_t *dev_status);
aqt_status launch_quantize_with_scale(const float *x, int64_t rows, int64_t cols, int64_t ldx, int bits,
                                      int axis, const float *scale, int8_t *q, uint32_t *mask,
                                      hipStream_t st);
// Up to eight matrices through the weight quantizer in one launch pair.
struct WeightJob {
  const float *w;
  int64_t K, N;
  int bits_w;
  void *wq_packed;
  float *s_w;
  int8_t *wq_kn;       // nullable
  uint32_t *mask_w;    // nullable
  uint32_t *part;      // kWeightSlabs x N words of its own
  void *wfrag;         // nullable
};
constexpr int kWeightJobsMax = 8;
aqt_status launch_quantize_weights_group(const WeightJob *jobs, int n, hipStream_t st, int32_t *dev_status);
struct DenseSource;
// The activations (per tensor) and the weights of one dense layer; one launch pair where the activations are aligned, want no mask
// and share no memory with what the weights leave behind (in two pairs x has been read by then).
aqt_status launch_quantize_dense(const float *x, int64_t rows, int64_t cols, int bits_x, int8_t *q, float *scale, uint32_t *mask,
                                 float *partials, const WeightJob &w, hipStream_t st, int32_t *dev_status,
                                 DenseSource *later = nullptr);   // later: the second launch is described there (xq set) where a product can take it
inline size_t weight_ws_bytes(int64_t N) { return align_up(static_cast<size_t>(kWeightSlabs) * N * 4, 256); }
aqt_status launch_unpack_weights(const void *wq_packed, int64_t K, int64_t N, int bits_w,
                                 int8_t *codes_kn, hipStream_t st);

// ---- forward contraction (gemm_fwd.hip) -----------------------------------------
aqt_status launch_dense_fwd_q(const int8_t *xq, const float *s_x, const void *wq_packed,
                              const float *s_w, int64_t M, int64_t K, int64_t N, int bits_w,
                              const float *bias, int epilogue, float *y, int32_t *acc_out, uint32_t *y_absmax,
                              void *ws, hipStream_t st, float *dact = nullptr, bool ws_is_prepared = false,
                              bool absmax_is_zero = false);
// True when the matrix-core kernel takes the shape (then its weight operand may be handed over
// already in fragment order: from the weight quantizer, or from launch_prepare_weights).
bool fwd_q_takes_fragments(int64_t M, int64_t K, int64_t N, int epilogue);
// True when it is also the kernel launch_dense_fwd_q picks, given the forward operand in its canonical form as well.
bool fwd_q_uses_fragments(int64_t M, int64_t K, int64_t N, int epilogue);
aqt_status launch_prepare_weights(const void *wq_packed, int64_t K, int64_t N, int bits_w, void *wprep,
                                  hipStream_t st);
size_t fwd_q_workspace_bytes(int64_t K, int64_t N);
aqt_status static_scratch_address(void **out);   // the library's own scratch array on the current device
size_t fwd_wonly_workspace_bytes(int64_t K, int64_t N);
aqt_status launch_dense_fwd_wonly(const float *x, const void *wq_packed, const float *s_w, int64_t M, int64_t K,
                                  int64_t N, int bits_w, const float *bias, int epilogue, float *y, void *ws,
                                  hipStream_t st);

// ---- contractions straight from the caller's tensors (gemm_any.hip): the forward for any shape; the float ones for small
// problems on the tuned kernels' grid, which gemm_bwd.hip checks -----------
aqt_status launch_dense_fwd_any(const int8_t *xq, const float *s_x, const void *wq_packed, const float *s_w, int64_t M,
                                int64_t K, int64_t N, int bits_w, const float *bias, int epilogue, float *y,
                                int32_t *acc_out, uint32_t *y_absmax, float *dact, hipStream_t st);
aqt_status launch_dense_fwd_wonly_any(const float *x, const void *wq_packed, const float *s_w, int64_t M, int64_t K,
                                      int64_t N, int bits_w, const float *bias, int epilogue, float *y, hipStream_t st);
aqt_status launch_bwd_dx_any(const float *dy, const int8_t *wq_kn, const float *s_w, const float *s_x, const uint32_t *mask_x,
                             const float *factor, int64_t M, int64_t K, int64_t N, float *dx, hipStream_t st);
int dw_any_slabs(int64_t M, int64_t K, int64_t N);   // slabs of rows: K x N floats each in `partial`, K / 128 x N doubles
                                                     // each in `bias_part` (dbias not null)
bool bwd_small_ok(int64_t M, int64_t K, int64_t N);
aqt_status launch_bwd_small_any(const float *dy, const int8_t *wq_kn, const float *s_w, const float *s_x, const uint32_t *mask_x,
                                const float *factor, const int8_t *xq, const uint32_t *mask_w, int64_t M, int64_t K, int64_t N,
                                float *dx, float *dw, float *dbias, hipStream_t st);
aqt_status launch_bwd_dw_any(const float *dy, const int8_t *xq, const float *s_x, const float *s_w, const uint32_t *mask_w,
                             int64_t M, int64_t K, int64_t N, float *dw, float *partial, float *dbias, double *bias_part,
                             hipStream_t st);

// ---- the float ones in float64, off the tuned kernels' grid (gemm_any_f64.hip) -------------------------
aqt_status launch_bwd_dx_f64(const float *dy, const int8_t *wq_kn, const float *s_w, const float *s_x, const uint32_t *mask_x,
                             const float *factor, int64_t M, int64_t K, int64_t N, float *dx, hipStream_t st);
aqt_status launch_dense_fwd_wonly_f64(const float *x, const void *wq_packed, const float *s_w, int64_t M, int64_t K,
                                      int64_t N, int bits_w, const float *bias, int epilogue, float *y, hipStream_t st);
int dw_f64_slabs(int64_t M, int64_t K, int64_t N);   // K x N doubles each in `partial`, cdiv(K, 64) x N each in `bias_part`
aqt_status launch_bwd_dw_f64(const float *dy, const int8_t *xq, const float *s_x, const float *s_w, const uint32_t *mask_w,
                             int64_t M, int64_t K, int64_t N, float *dw, double *partial, int max_slabs, float *dbias,
                             double *bias_part, hipStream_t st);

aqt_status launch_dw_f64_fold(const double *partial, int slabs, int64_t K, int64_t N, const float *s_x, const float *s_w,
                              const uint32_t *mask_w, float *dw, const double *bias_part, int bias_rows, float *dbias,
                              hipStream_t st);

// ---- the same sums on the int8 matrix cores, where there is enough work (gemm_exact.hip) -------------------------
bool f32_codes_exact_ok(int64_t M, int64_t R, int64_t C);   // M x R results, contraction C
aqt_status launch_bwd_dx_exact(const float *dy, const int8_t *wq_kn, const float *s_w, const float *s_x, const uint32_t *mask_x,
                               const float *factor, int64_t M, int64_t K, int64_t N, float *dx, hipStream_t st);
aqt_status launch_dense_fwd_wonly_exact(const float *x, const void *wq_packed, const float *s_w, int64_t M, int64_t K,
                                        int64_t N, int bits_w, const float *bias, int epilogue, float *y, hipStream_t st);
bool dw_exact_ok(int64_t M, int64_t K, int64_t N, int slabs);
int dw_exact_slabs(int64_t M, int64_t K, int64_t N);
aqt_status launch_bwd_dw_exact(const float *dy, const int8_t *xq, const float *s_x, const float *s_w, const uint32_t *mask_w,
                               int64_t M, int64_t K, int64_t N, float *dw, double *partial, int slabs, float *dbias,
                               double *bias_part, hipStream_t st);

// ---- straight-through backward (gemm_bwd.hip) -------------------------------------
size_t bwd_workspace_bytes(int64_t M, int64_t K, int64_t N);
// dx_factor (optional, [M,K]): dx leaves multiplied elementwise by it (the previous layer's activation derivative)
aqt_status launch_dense_bwd(const float *dy, const aqt_saved *sv, int64_t M, int64_t K, int64_t N,
                            float *dx, float *dw, float *dbias, void *ws, size_t ws_bytes,
                            hipStream_t st, const float *dx_factor = nullptr);

// Float32 rows [M,K] whose codes are still to be made, by the product that takes them: launch_quantize_with_absmax inside
// gemm_any.hip's forward.  x is 16-byte and q 4-byte aligned.
struct RowSource {
  const float *x;
  const uint32_t *absmax;
  int qmax;
  int8_t *q;
  float *scale;
  int32_t *dev_status;
};
bool dense_fwd_rows_ok(int64_t M, int64_t K, int64_t N);
aqt_status launch_dense_fwd_rows(const RowSource &src, const void *wq_packed, const float *s_w, int64_t M, int64_t K, int64_t N,
                                 int bits_w, const float *bias, float *y, hipStream_t st);

// A dense layer's float32 tensors and where its codes go, behind the pass that takes the maxima (absmax_dense_kernel): the second
// launch of launch_quantize_dense and the product in one.  x, w 16-byte, the codes 4-byte aligned, no clip masks.
struct DenseSource {
  const float *x;
  const uint32_t *partial;   // nparts maxima of |x|
  int nparts, qmax_x;
  int8_t *xq;
  float *s_x;
  const float *w;
  const uint32_t *part;      // slabs x N maxima of |w|
  int slabs, qmax_w, packed;
  uint8_t *wq_packed;
  float *s_w;
  int8_t *wq_kn;             // nullable
  int32_t *dev_status;
};
bool dense_fwd_raw_ok(int64_t M, int64_t K, int64_t N, int epilogue);
aqt_status launch_dense_fwd_raw(const DenseSource &src, int64_t M, int64_t K, int64_t N, const float *bias, int epilogue, float *y,
                                float *dact, hipStream_t st);

// ---- block pieces (block.hip) -----------------------------------------------------------
size_t layernorm_ws_bytes(int64_t M);
// res / alpha / sum_out (optional): normalise x + alpha * res instead of x and leave that sum in sum_out.
// zero_word (optional): a word the first pass clears, e.g. the abs-max word of a producer launched after it
// (which is then told absmax_is_zero and needs no clearing launch of its own).
aqt_status launch_layernorm_quantize(const float *x, int64_t M, int64_t D, const float *gamma, const float *beta,
                                     float eps, int bits, int8_t *q, float *scale, float *y_out, float *row_stats,
                                     void *ws, hipStream_t st, int32_t *dev_status, const float *res = nullptr,
                                     float alpha = 0.0f, float *sum_out = nullptr, uint32_t *zero_word = nullptr);
size_t layernorm_bwd_ws_bytes(int64_t D);
// The column sums of a normalisation's backward, left to be folded (its workspace has to last until then).
struct LnFold {
  const float *part;
  float *dgamma, *dbeta;   // nullable
  int parts;
};
constexpr int kLnFoldsMax = 5;
aqt_status launch_ln_folds(const LnFold *jobs, int n, int64_t D, hipStream_t st);
// later (optional): the fold is not launched, but described there
aqt_status launch_layernorm_bwd(const float *x, const float *stats, const float *gamma, const float *dy,
                                const float *add, int64_t M, int64_t D, float *dx, float *dgamma, float *dbeta,
                                void *ws, hipStream_t st, float *half = nullptr, LnFold *later = nullptr);
aqt_status launch_scale(const float *m, float alpha, float *out, int64_t n, hipStream_t st);
aqt_status launch_dact_mul(const float *dout, const float *dact, int64_t M, int64_t N, int64_t oc, float *dv,
                           hipStream_t st);
aqt_status launch_residual_add(const float *x, const float *m, float alpha, float *out, int64_t n, hipStream_t st);
aqt_status launch_fake_matmul_f32(const int8_t *xq, const int8_t *wq_kn, int64_t M, int64_t K, int64_t N, float *out,
                                  hipStream_t st);

// ---- depthwise convolution of the convolution module (conv.hip) ---------------------------
size_t dwconv_bwd_ws_bytes(int64_t C, int kw);
bool dwconv_takes_gate(int64_t M, int64_t C, int kw);   // M = B * T frames: the backward multiplies by the gate itself
aqt_status launch_dwconv_fwd(const float *x, const float *w, const float *bias, const float *na, const float *nb,
                             int swish, int64_t B, int64_t T, int64_t C, int kw, int pad_left, float *out, float *dfac,
                             uint32_t *absmax, hipStream_t st, bool absmax_is_zero = false);
aqt_status launch_dwconv_bwd(const float *dout, const float *dmul, const float *x, const float *w, int64_t B, int64_t T,
                             int64_t C, int kw, int pad_left, float *dx, float *dw, float *dbias, void *ws,
                             hipStream_t st, const float *gate = nullptr, float *dv = nullptr);   // with gate: dv [B T, 2 C] is wanted, dx scratch (not used where dwconv_takes_gate)

// ---- attention core of the self-attention module (attention.hip, attention_fwd.hip, attention_bwd.hip) -------------
struct AttnShape {
  int64_t B, D;
  int T;                        // frames: positions within an utterance are 32-bit (2^31 - 1 here: too long for that)
  int heads, dh, left, right;   // left / right < 0: no limit on that side, otherwise at most T
  int qtiles;                   // tiles per utterance: of 128 frames, or of the 32 that a workgroup of the backward for small batches owns
  float scale_log2e, scale;     // log2(e) / sqrt(dh), 1 / sqrt(dh)
};
// Heads of a multiple of four on 16-byte aligned tensors; dsum [B*T, heads].
bool attention_rows_ok(const AttnShape &g, const void *a, const void *b, const void *c, const void *d);
bool attention_few_ok(const AttnShape &g);   // ... and so few tiles of 128 queries that attention_few.hip's of 16 are faster
aqt_status launch_attention_few(const float *qkv, const AttnShape &g, float *ctx, uint32_t *absmax, float *lse, hipStream_t st);
aqt_status launch_attention_rows(const float *qkv, const AttnShape &g, float *ctx, uint32_t *absmax, float *lse, hipStream_t st);
bool attention_bwd_few_ok(const AttnShape &g);   // ... whether its form for few workgroups is the faster
aqt_status launch_attention_bwd_rows(const float *qkv, const float *ctx, const float *dctx, const float *lse, const AttnShape &g,
                                      float *dqkv, float *dsum, hipStream_t st);
bool attention_shape_ok(int64_t B, int64_t T, int64_t D, int heads);
aqt_status launch_attention(const float *qkv, int64_t B, int64_t T, int64_t D, int heads, int left, int right,
                            float *ctx, uint32_t *absmax, float *lse, hipStream_t st, bool absmax_is_zero = false);
size_t attention_bwd_ws_bytes(int64_t B, int64_t T, int heads);
aqt_status launch_attention_bwd(const float *qkv, const float *ctx, const float *dctx, const float *lse, int64_t B,
                                int64_t T, int64_t D, int heads, int left, int right, float *dqkv, void *ws,
                                hipStream_t st);

}  // namespace aqt
