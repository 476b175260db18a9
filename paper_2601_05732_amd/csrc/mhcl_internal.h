// Host-side declarations shared by the translation units of libmhcl.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "../../include/mhcl.h"

namespace mhcl {

inline int host_factorial(int n) { return n <= 1 ? 1 : n * host_factorial(n - 1); }
inline int res_logits(const mhcl_desc &d) {
  if (d.res_mode == MHCL_RES_LITE) return host_factorial(d.n);
  if (d.res_mode == MHCL_RES_SUBSET) return d.n_perm;
  return d.n * d.n;
}
// A workspace is sized for every token count up to T, so that one made for a caller's largest batch serves
// its smaller ones: the number of slices rises as T falls.  `parts1` slices at one token, and never
// more than `most` slices times tokens while there is more than one.
inline int64_t slice_tokens(int64_t T, int parts1, int64_t most) {
  const int64_t split = parts1 * T < most ? parts1 * T : most;
  return split > T ? split : T;
}
// the cache between the L2s and HBM
constexpr int64_t kLastLevelCache = int64_t{256} << 20;

inline size_t align_up(size_t v, size_t a = 256) { return (v + a - 1) / a * a; }

// Carves a caller-provided workspace into 256-byte aligned pieces.
struct WsCursor {
  char *base;
  size_t off = 0;
  explicit WsCursor(void *p) : base(static_cast<char *>(p)) {}
  template <typename T>
  T *take(size_t count) {
    T *p = base ? reinterpret_cast<T *>(base + off) : nullptr;
    off += align_up(count * sizeof(T));
    return p;
  }
};

// floats of a token's coefficient record, whole 16-byte pieces
constexpr int token_rec_floats(int n) { return (n * n + 2 * n + 1 + 3) / 4 * 4; }
template <int N>
constexpr int token_rec() { return token_rec_floats(N); }

// Per-token results of the backward's coefficient stage, all [T, ...] fp32.
struct BwdTokenBufs {
  float *rec;     // [T, token_rec<n>()] H_res | H_pre | H_post | coefx = (r^2 / nC) <vr, u_raw>
  float *vr;      // [T, 16 ceil(M / 16)] r * alpha_g * g_z (the vector multiplied with W and x), zero-padded
  float *gz;      // [gz_rows(d), M+3] sums over a block's tokens of g_z and of the per-group g_z u
};

// Layers of a stack whose kernels share launches (mhcl_coeffs_logits_layers).
constexpr int kJointLayers = 8;
struct JointLayers {
  const void *x[kJointLayers];
  const float *W[kJointLayers], *b[kJointLayers], *alpha[kJointLayers];
  int64_t stride;   // floats from a layer's u_raw to the next one's, and of sumsq
};

// ---- stream kernels: any n in 1..8, bf16 or f32 streams -----
hipError_t launch_pre(const mhcl_desc &d, const void *x, const float *H_pre, void *h, hipStream_t s);
hipError_t launch_post(const mhcl_desc &d, const void *x, const void *y, const float *H_res,
                       const float *H_post, void *x_out, hipStream_t s);
hipError_t launch_post_bwd(const mhcl_desc &d, const void *x, const void *y, const float *H_res,
                           const float *H_post, const void *g_xout, void *g_x, void *g_y,
                           float *g_H_res, float *g_H_post, hipStream_t s);
hipError_t launch_pre_bwd(const mhcl_desc &d, const void *x, const float *H_pre, const void *g_h,
                          void *g_x, float *g_H_pre, hipStream_t s);
// x = n copies of x0, out = the sum of x's streams
hipError_t launch_streams_in(const mhcl_desc &d, const void *x0, void *x, hipStream_t s);
hipError_t launch_streams_out(const mhcl_desc &d, const void *x, void *out, hipStream_t s);
// dots only: g_H_res = <g_xout[i], x[j]>, g_H_post = <g_xout[i], y>, g_H_pre = <g_h, x[j]>
hipError_t launch_bwd_dots(const mhcl_desc &d, const void *x, const void *y, const void *g_xout,
                           const void *g_h, float *g_H_res, float *g_H_post, float *g_H_pre,
                           hipStream_t s);
hipError_t launch_copy(void *dst, const void *src, size_t bytes, hipStream_t s);
// a fill kernel (safe under graph capture, unlike a memset node)
hipError_t launch_fill_zero(float *p, size_t count, hipStream_t s);

// ---- full-precision products on the matrix cores: any C, bf16 or f32 streams -----
// whether u_raw, sumsq come from the fp64 projection below (else from launch_proj_mfma)
bool proj_fullprec_used(const mhcl_desc &d);
int64_t few_tokens(const mhcl_desc &d);   // up to so many where the other could run too
int proj_fullprec_parts(const mhcl_desc &d);   // slices it writes: one in fp32, 2, 4, 8, 16 or 32 in fp64
// floats that the slices of one logit take, at most, of T tokens or fewer
int64_t proj_fullprec_slice_floats(const mhcl_desc &d);
hipError_t launch_proj_fullprec(const mhcl_desc &d, int M, const void *x, const float *W,
                                float *u_raw, float *sumsq, hipStream_t s);
hipError_t launch_proj_fullprec_layers(const mhcl_desc &d, int M, const JointLayers &layers, int L, float *u_raw,
                                       float *sumsq, hipStream_t s);
// What a projection leaves for the per-token stage, where the slices are added in order: u_raw
// [parts][T][M] and sumsq [parts][T], in fp64 if `wide`.
struct RawSums {
  const float *u_raw, *sumsq;
  int parts;
  bool wide;
};
// the sums over fp64 slices take the place of the first one, which alone is left
hipError_t add_wide_slices(const mhcl_desc &d, RawSums &raw, hipStream_t s);
// as launch_proj_fullprec or launch_proj_mfma left them
RawSums projected(const mhcl_desc &d, const float *u_raw, const float *sumsq);
// g_W from x and vr (rows as in BwdTokenBufs); `partials` holds gw_chunks_fullprec(d) results
// of [nC, M] when that is more than one
int gw_chunks_fullprec(const mhcl_desc &d);
hipError_t launch_gw_fullprec(const mhcl_desc &d, int M, const void *x, const float *vr,
                              float *partials, float *g_W, hipStream_t s);
// fused == true : g_x = H_res^T g_xout + H_pre g_h + W vr - x coefx ; g_y = H_post g_xout
// fused == false: g_x += W vr - x coefx
hipError_t launch_gx_fullprec(const mhcl_desc &d, int M, bool fused, const void *x, const float *W,
                             const void *g_xout, const void *g_h, const BwdTokenBufs &o, void *g_x,
                             void *g_y, hipStream_t s);

// What does not wait for each other, as one launch: launch_proj_fullprec with launch_bwd_dots where joint_proj_dots_ok;
// launch_gx_fullprec with launch_gw_fullprec and the sums behind g_b and g_alpha (gz_count rows) where joint_fullprec_ok
bool joint_proj_dots_ok(const mhcl_desc &d);
bool joint_fullprec_ok(const mhcl_desc &d);
hipError_t launch_proj_dots(const mhcl_desc &d, int M, const void *x, const float *W, const void *y,
                            const void *g_xout, const void *g_h, float *u_raw, float *sumsq, float *g_H_res,
                            float *g_H_post, float *g_H_pre, hipStream_t s);
hipError_t launch_gx_gw_fullprec(const mhcl_desc &d, int M, bool fused, const void *x, const float *W,
                                 const void *g_xout, const void *g_h, const BwdTokenBufs &o, void *g_x, void *g_y,
                                 float *partials, float *g_W, int64_t gz_count, float *g_b, float *g_alpha,
                                 hipStream_t s);

// ---- per-token stage of the other forms (n <= 4, Sinkhorn-Knopp) --------------
bool token_stage_many(const mhcl_desc &d, bool backward);   // the variant for many tokens
bool token_per_lane(const mhcl_desc &d, bool backward);     // more tokens still
hipError_t launch_token_coeffs(const mhcl_desc &d, const RawSums &raw, const float *b,
                               const float *alpha, float *H_res, float *H_pre, float *H_post,
                               hipStream_t s);
// the coefficients and, in the same launch, h = H_pre x, where token_coeffs_pre_ok
bool token_coeffs_pre_ok(const mhcl_desc &d, const RawSums &raw);
hipError_t launch_token_coeffs_pre(const mhcl_desc &d, const RawSums &raw, const float *b, const float *alpha,
                                   const void *x, float *H_res, float *H_pre, float *H_post, void *h,
                                   hipStream_t s);
// the same with the logits z [T,M] and spread [T] (see launch_logits) where token_logits_ok
bool token_logits_ok(const mhcl_desc &d, const RawSums &raw);
hipError_t launch_token_coeffs_logits(const mhcl_desc &d, const RawSums &raw, const float *b,
                                      const float *alpha, float *H_res, float *H_pre, float *H_post,
                                      float *z, float *spread, hipStream_t s);
// several layers' launches shared, where joint_layers_ok: `raw` is the first one's, the outputs are stacks [layer][T][...]
bool joint_layers_ok(const mhcl_desc &d);
hipError_t launch_token_layers(const mhcl_desc &d, const RawSums &raw, const JointLayers &layers, int count, float *H_res,
                               float *z, float *spread, hipStream_t s);
hipError_t launch_token_bwd_full(const mhcl_desc &d, const RawSums &raw, const float *b,
                                 const float *alpha, const float *g_H_res, const float *g_H_pre,
                                 const float *g_H_post, const BwdTokenBufs &o, hipStream_t s);

// ---- permutation-subset form (run-time table d.perm, n up to 8) --------------
// eight lanes per token: permutation subsets and the full form at n = 5
bool coeffs_group_ok(const mhcl_desc &d);
// rows of the g_z sums that the per-token stage of the backward (`fast`: of the fast path) leaves
// for launch_bwd_finish
int64_t gz_rows(const mhcl_desc &d, bool fast);
int64_t gz_rows_reserved(const mhcl_desc &d);   // at most, of T tokens or fewer
hipError_t launch_coeffs_group(const mhcl_desc &d, const RawSums &raw, const float *b,
                               const float *alpha, float *H_res, float *H_pre, float *H_post,
                               hipStream_t s);
bool group_coeffs_pre_ok(const mhcl_desc &d);   // with h in the same launch
hipError_t launch_coeffs_pre_group(const mhcl_desc &d, const RawSums &raw, const float *b, const float *alpha,
                                   const void *x, float *H_res, float *H_pre, float *H_post, void *h,
                                   hipStream_t s);
hipError_t launch_coeffs_bwd_group(const mhcl_desc &d, const RawSums &raw, const float *b,
                                   const float *alpha, const float *g_H_res, const float *g_H_pre,
                                   const float *g_H_post, const BwdTokenBufs &o, hipStream_t s);

// ---- diagnostics ----------------------------------------------------------
// z [T,M] and spread [T] (max - min of the residual logits); either may be null
hipError_t launch_logits(const mhcl_desc &d, int M, const RawSums &raw, const float *b,
                         const float *alpha, float *z, float *spread, hipStream_t s);
hipError_t launch_ds_chain(int n, int L, int64_t T, const float *H, float *colsum, float *l1,
                           float *prod, float *prod_colsum, float *prod_l1, hipStream_t s);

// ---- bf16 fast path (MFMA projections); needs fast_path_ok(desc) ---------
bool fast_path_ok(const mhcl_desc &d);
// Either projection may split K over several blocks per token tile (the MFMA one over up to
// kMaxMfmaParts); u_raw and sumsq then hold that many slices ([parts][T][M], [parts][T]).
constexpr int kMaxMfmaParts = 16;
int proj_ksplit(const mhcl_desc &d);
int mfma_ksplit(const mhcl_desc &d);   // slices of launch_proj_mfma
int64_t mfma_slices(const mhcl_desc &d);         // slices x tokens that the forward's workspace holds
int64_t mfma_slice_tokens(const mhcl_desc &d);   // slices x tokens of launch_proj_mfma, at most, of T tokens or fewer
size_t packed_w_b_bytes(const mhcl_desc &d, int M);
// packs W (B layout) and, in the same launch, clears `nzero` floats at `zero`
hipError_t launch_pack_w_b(const mhcl_desc &d, int M, const float *W, void *Wp, hipStream_t s,
                           float *zero = nullptr, size_t nzero = 0);
// reads W itself where proj_mfma_direct(d), else Wp (W packed by launch_pack_w_b or launch_pack_w_ab)
bool proj_mfma_direct(const mhcl_desc &d);
hipError_t launch_proj_mfma(const mhcl_desc &d, int M, const void *x, const void *Wp, const float *W,
                            float *u_raw, float *sumsq, hipStream_t s);
// (W as it is: where proj_mfma_direct)
hipError_t launch_proj_mfma_layers(const mhcl_desc &d, int M, const JointLayers &layers, int L, float *u_raw, float *sumsq,
                                   hipStream_t s);

// Single-read forward (projection slices, H_pre and h from one read of x): bf16 fast path
// with at most 32 logits, C a multiple of 256 from 1024 to 8192, enough tokens to fill the pipeline.
bool fwd_once_ok(const mhcl_desc &d);
struct OnceWs {
  float *u_part, *sumsq_part;   // [parts][T][M], [parts][T]: one slice per 256-column part
  char *Wp;                     // packed W (B layout)
  unsigned long long *xchg;     // exchange rings of the kernel (zeroed by its launcher)
  size_t xchg_words, bytes;
  int parts;
  OnceWs(const mhcl_desc &d, void *ws);
};
// *usable == false on return with hipSuccess: this device cannot hold the kernel's grid at
// once (the caller then takes the two-kernel path).
hipError_t prepare_fwd_once(const mhcl_desc &d, int M, bool *usable);
// the kernel itself; w.Wp must hold the packed W and the w.xchg_words words at w.xchg must be
// zero (tags count from 1 in every launch)
hipError_t launch_fwd_once(const mhcl_desc &d, int M, const void *x, const float *b,
                           const float *alpha, const OnceWs &w, void *h, hipStream_t s);

// fused backward on the fast path (needs fast_bwd_ok(desc))
bool fast_bwd_ok(const mhcl_desc &d);
bool fast_bwd_whi(const mhcl_desc &d);    // wide case, n >= 5, where W fits LDS as one fp16 part: that pass 2 as one kernel
bool fast_bwd_wide(const mhcl_desc &d);   // n >= 5 or a subset: pass 2 split into W vr and the mixing
int gw_chunks_fast(const mhcl_desc &d);
int reduce_parts(const mhcl_desc &d);     // slices that launch_bwd_reduce writes
struct FastBwdWs {
  // gz: [gz_rows(d)][M+3] sums of g_z and g_z u over each block's tokens
  // wmax_part: partial maxima of |W|; wscale: {scale, 1 / scale} of the fp16 copy of W
  float *u_raw, *sumsq, *gH_res, *gH_pre, *gH_post, *cpk, *gz, *partials, *D, *wmax_part, *wscale;
  uint16_t *vr_hi, *vr_lo, *vrT_hi, *vrT_lo;
  char *Wp, *Wa;
  int CP, MP32, MP16, parts, gparts;   // slices of u_raw, sumsq and of gH_*
  bool wide_sums;                      // the former are fp64
  RawSums raw() const { return {u_raw, sumsq, parts, wide_sums}; }
  size_t bytes;
  FastBwdWs(const mhcl_desc &d, void *ws);
};
hipError_t launch_pack_w_ab(const mhcl_desc &d, int M, const float *W, const FastBwdWs &w,
                            hipStream_t s);
// whether the two passes of n <= 4 take W as it is (else packed by launch_pack_w_ab)
bool narrow_direct(const mhcl_desc &d);
hipError_t launch_bwd_reduce(const mhcl_desc &d, int M, const void *x, const void *y, const float *W,
                             const void *g_xout, const void *g_h, const FastBwdWs &w,
                             hipStream_t s);
hipError_t launch_bwd_dots_fast(const mhcl_desc &d, const void *x, const void *y, const void *g_xout,
                                const void *g_h, const FastBwdWs &w, hipStream_t s);
// per-token stage between the two passes: coefficients again, g_z and what pass 2 reads
hipError_t launch_token_bwd_fast(const mhcl_desc &d, const float *b, const float *alpha,
                                 const FastBwdWs &w, hipStream_t s);
// the same stage for the permutation-subset form (run-time table)
hipError_t launch_bwd_epilogue_group(const mhcl_desc &d, const float *b, const float *alpha,
                                     const FastBwdWs &w, hipStream_t s);
hipError_t launch_bwd_out_wide(const mhcl_desc &d, int M, const void *x, const void *g_xout,
                               const void *g_h, const FastBwdWs &w, void *g_x, void *g_y,
                               hipStream_t s);
// (with one chunk of tokens also g_b and g_alpha, from the gz_count rows of g_z sums)
hipError_t launch_bwd_out_gw(const mhcl_desc &d, int M, const void *x, const float *W, const void *g_xout,
                             const void *g_h, const FastBwdWs &w, void *g_x, void *g_y, float *g_W,
                             int64_t gz_count, float *g_b, float *g_alpha, hipStream_t s);
hipError_t launch_bwd_gw(const mhcl_desc &d, int M, const void *x, const FastBwdWs &w, float *g_W,
                         hipStream_t s);
// g_W from the chunks' partial sums (none if chunks == 1) and g_b, g_alpha from the
// [rows, M+3] sums of g_z (none if rows == 0), in one launch
hipError_t launch_bwd_finish(const float *partials, size_t size, int chunks, float *g_W,
                             const float *gz_rows, int64_t rows, int M, float *g_b, float *g_alpha,
                             hipStream_t s);
int fast_gw_chunks(const mhcl_desc &d);

}  // namespace mhcl
