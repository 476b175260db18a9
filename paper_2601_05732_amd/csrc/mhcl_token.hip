// Per-token stage of the compile-time forms (all n! permutations for n <= 4, Sinkhorn-Knopp):
// from the raw projection to the coefficients, and in the backward on to g_z and the operands of
// what follows.  The work of one token is a few hundred dependent instructions, so it is spread
// over a group of lanes: 16 for n <= 4 (lane 4 i + j owns entry (i, j) of H_res, and the
// residual logits l, l + 16), four where there are many tokens (a row of H_res each), eight for n = 5
// (likewise).  Sums over the group are DPP steps.  With more tokens still, one lane per token.
#include "mhcl_common.h"
#include "mhcl_internal.h"
#include "mhcl_mfma.h"
#include "mhcl_pre.h"

namespace mhcl {

namespace {

// tokens and threads per block
template <int L>
constexpr int kTokBlock = L == 4 ? 64 : 32;
template <int L>
constexpr int kTokThreads = L * kTokBlock<L>;

// kinds of output (kOutLogits: the forward's with the logits)
enum { kOutForward, kOutLogits, kOutFast, kOutFull };
constexpr bool out_bwd(int out) { return out == kOutFast || out == kOutFull; }

template <int CTRL>
__device__ __forceinline__ float dpp(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, true));
}
constexpr int kRor1 = 0x121, kRor2 = 0x122, kRor4 = 0x124, kRor8 = 0x128;   // rotate in rows of 16 lanes
constexpr int kXor1 = 0xB1, kXor2 = 0x4E;                                   // exchange in quads
constexpr int kHalfMirror = 0x141;                                          // reverse eight lanes

// over all lanes of a token's group (every lane gets the same bits: each step adds a pair)
template <int L, typename OP>
__device__ __forceinline__ float group_reduce(float v, OP op) {
  if constexpr (L == 16) {
    v = op(v, dpp<kRor8>(v));
    v = op(v, dpp<kRor4>(v));
    v = op(v, dpp<kRor2>(v));
    v = op(v, dpp<kRor1>(v));
  } else {
    v = op(v, dpp<kXor2>(v));
    v = op(v, dpp<kXor1>(v));
    if constexpr (L == 8) v = op(v, dpp<kHalfMirror>(v));
  }
  return v;
}
struct Add {
  __device__ __forceinline__ float operator()(float a, float b) const { return lane_add(a, b); }
};
struct Max {
  __device__ __forceinline__ float operator()(float a, float b) const { return fmaxf(a, b); }
};
// Sums over the rows i (one per column that the lane has entries of) and over the columns j (one:
// a lane's entries are of one row) of a matrix spread over the group.
template <int L, int CC>
__device__ __forceinline__ void column_sums(const float (&v)[CC], float (&s)[CC]) {
#pragma unroll
  for (int c = 0; c < CC; ++c) {
    s[c] = v[c];
    if constexpr (L == 16) {
      s[c] = lane_add(s[c], dpp<kRor8>(s[c]));
      s[c] = lane_add(s[c], dpp<kRor4>(s[c]));
    } else {
      s[c] = lane_add(s[c], dpp<kXor2>(s[c]));
      s[c] = lane_add(s[c], dpp<kXor1>(s[c]));
      if constexpr (L == 8) s[c] = lane_add(s[c], dpp<kHalfMirror>(s[c]));
    }
  }
}
template <int L, int CC>
__device__ __forceinline__ float row_sum(const float (&v)[CC]) {
  // (the same sums whether a lane has a row, up to four entries, or an entry)
  if constexpr (CC == 4) return lane_add(lane_add(v[0], v[1]), lane_add(v[2], v[3]));
  float s = v[0];
#pragma unroll
  for (int c = 1; c < CC; ++c) s = lane_add(s, v[c]);
  if constexpr (L == 16) {
    s = lane_add(s, dpp<kXor1>(s));
    s = lane_add(s, dpp<kXor2>(s));
  }
  return s;
}

// 1 / s of a Sinkhorn-Knopp half step (s at most n: the entries are at most 1): v_rcp_f32 and one Newton-Raphson step in fused
// multiply-adds.  Scaled by 2^60, so that sums below the normal range keep their reciprocals; of 0, where the division
// gives infinity, it is NaN, as the entries of such a line become either way (0 times infinity).
// The division's bits: compared for every positive float below 8, subnormals too.  (The step's error before its one rounding is 2^-44, which
// does not settle sums next to a tie, such as 1 - 2^-24: these hold because of what the instruction returns there.)
// Five instructions for the division's eleven, which were half of a half step: the stage of six layers, n = 4, 8192
// tokens, 20 iterations 20.6 / 16.5 us, steps n = 4, C = 768, 3001 tokens 70.9 / 69.6, n = 5, C = 512, 20000 tokens 344 / 339.
__device__ __forceinline__ float reciprocal(float s) {
  const float t = s * 0x1p60f, r = __builtin_amdgcn_rcpf(t);
  return fmaf(fmaf(-t, r, 1.f), r, r) * 0x1p60f;
}

// bit k set: permutation k has its 1 of row i in column j
template <int N>
constexpr uint32_t cell_mask(int i, int j) {
  uint32_t m = 0;
  for (int k = 0; k < factorial(N); ++k)
    if (Perm<N>::tab.s[k][i] == j) m |= 1u << k;
  return m;
}
// the columns of permutation k, two bits each
template <int N>
constexpr uint32_t perm_bits(int k) {
  uint32_t b = 0;
  for (int i = 0; i < N; ++i) b |= static_cast<uint32_t>(Perm<N>::tab.s[k][i]) << (2 * i);
  return b;
}
template <int N, int... C>
__device__ __forceinline__ uint32_t select_mask(int cell, std::integer_sequence<int, C...>) {
  uint32_t m = 0;
  ((m = cell == C ? std::integral_constant<uint32_t, cell_mask<N>(C / N, C % N)>::value : m), ...);
  return m;
}
template <int N, int... K>
__device__ __forceinline__ uint32_t select_perm(int k, std::integer_sequence<int, K...>) {
  uint32_t b = 0;
  ((b = k == K ? std::integral_constant<uint32_t, perm_bits<N>(K)>::value : b), ...);
  return b;
}

struct TokenIn {
  const float *u_raw, *sumsq;              // [parts][T][M], [parts][T], in fp64 if `wide`
  int parts;
  bool wide;
  const float *gH_res, *gH_pre, *gH_post;  // backward: [gparts][T][n*n], [gparts][T][n]
  int gparts;
  const float *b, *alpha;
  int nC;
  float eps;
  int sk_iters;
  int64_t T;
};
struct TokenOut {
  float *H_res, *H_pre, *H_post;                     // forward
  float *z, *spread;                                 // kOutLogits: logits, max - min of the residual ones
  float *rec;                                        // backward: records of `rec_ld` floats
  int rec_ld;
  uint16_t *vr_hi, *vr_lo, *vrT_hi, *vrT_lo;         // fast
  float *vr;                                         // full
  float *gz_sums;                                    // [blocks][M + 3]
};

// dst[tok][0..W) = the sums over the slices of src [slices][T][W], tokens t0 ... of the block
// (past the last token: some valid element again).  begin() requests the first slice, so that
// several arrays can be on their way together; finish() requests eight more slices at a time
// and adds them in order.
template <int W, int L>
struct StageSums {
  static constexpr int THREADS = kTokThreads<L>, BT = kTokBlock<L>;
  static constexpr int IT = (BT * W + THREADS - 1) / THREADS;
  const float *src;
  size_t stride, e[IT];
  float s[IT];
  __device__ __forceinline__ void begin(const float *p, int64_t T, int64_t t0) {
    src = p;
    stride = static_cast<size_t>(T) * W;
#pragma unroll
    for (int i = 0; i < IT; ++i) {
      const size_t at = static_cast<size_t>(t0) * W + threadIdx.x + i * THREADS;
      e[i] = at < stride ? at : stride - 1;
      s[i] = src[e[i]];
    }
  }
  __device__ __forceinline__ void finish(int slices, float *dst, int ld) {
    for (int p0 = 1; p0 < slices; p0 += 8) {
      float v[IT][8];
#pragma unroll
      for (int i = 0; i < IT; ++i)
#pragma unroll
        for (int k = 0; k < 8; ++k) v[i][k] = src[(p0 + k < slices ? p0 + k : slices - 1) * stride + e[i]];
#pragma unroll
      for (int i = 0; i < IT; ++i)
#pragma unroll
        for (int k = 0; k < 8; ++k)
          if (p0 + k < slices) s[i] += v[i][k];
    }
#pragma unroll
    for (int i = 0; i < IT; ++i) {
      const int idx = threadIdx.x + i * THREADS;
      if (idx < BT * W) dst[(idx / W) * ld + idx % W] = s[i];
    }
  }
};

// the same for slices in fp64, rounded once: a row that was split sums as a whole one does.  E elements per
// thread and all their slices are on their way together.
template <int W, int L, int S, int E>
__device__ __forceinline__ void stage_wide_pass(const double *src, int64_t T, int64_t t0, float *dst, int ld) {
  constexpr int THREADS = kTokThreads<L>, ALL = kTokBlock<L> * W;
  const int64_t stride = T * W;
  for (int e0 = threadIdx.x; e0 < ALL; e0 += E * THREADS) {
    double v[E][S];
#pragma unroll
    for (int i = 0; i < E; ++i) {
      const int64_t at = t0 * W + e0 + i * THREADS, e = at < stride ? at : stride - 1;
#pragma unroll
      for (int k = 0; k < S; ++k) v[i][k] = src[k * stride + e];
    }
#pragma unroll
    for (int i = 0; i < E; ++i) {
      double s = v[i][0];
#pragma unroll
      for (int k = 1; k < S; ++k) s += v[i][k];
      const int e = e0 + i * THREADS;
      if (e < ALL) dst[(e / W) * ld + e % W] = static_cast<float>(s);
    }
  }
}
// slices: 2, 4, 8, 16 or 32 (proj_fullprec_parts)
template <int W, int L>
__device__ __forceinline__ void stage_wide(const float *src, int slices, int64_t T, int64_t t0, float *dst, int ld) {
  constexpr int IT = (kTokBlock<L> * W + kTokThreads<L> - 1) / kTokThreads<L>;
  const double *p = reinterpret_cast<const double *>(src);
  switch (slices) {
    case 2: stage_wide_pass<W, L, 2, IT>(p, T, t0, dst, ld); break;
    case 4: stage_wide_pass<W, L, 4, IT>(p, T, t0, dst, ld); break;
    case 8: stage_wide_pass<W, L, 8, IT < 4 ? IT : 4>(p, T, t0, dst, ld); break;
    case 16: stage_wide_pass<W, L, 16, IT < 2 ? IT : 2>(p, T, t0, dst, ld); break;
    default: stage_wide_pass<W, L, 32, 1>(p, T, t0, dst, ld);
  }
}

// floats of dynamic LDS per Sinkhorn-Knopp iteration: the divisors of its two half steps and their
// reciprocals, one pair per line and token of a pass (backward only)
template <int N, int L>
constexpr int kLines = L == 16 ? 4 : N;   // lines per token, as they are spaced
template <int N, int MODE, int OUT, int L>
constexpr int kSkPerIter = (MODE == MHCL_RES_SK && out_bwd(OUT))
                               ? 2 * 2 * kTokBlock<L> * kLines<N, L> : 0;

template <int N, int MODE, int OUT, int L>
__device__ __forceinline__ void token_stage(const TokenIn &in, const TokenOut &out) {
  constexpr int R = Dims<N, MODE>::R, M = Dims<N, MODE>::M, NN = N * N;
  constexpr int THREADS = kTokThreads<L>, BT = kTokBlock<L>, NP = kLines<N, L>;
  constexpr int CC = L == 16 ? 1 : N;                          // entries of H_res per lane
  constexpr int KK = MODE == MHCL_RES_LITE ? (R + L - 1) / L : CC;   // residual logits per lane
  constexpr int GG = (2 * N + L - 1) / L;                      // gates per lane
  constexpr int MP32 = (M + 31) / 32 * 32, MP16 = (M + 15) / 16 * 16;
  constexpr bool BWD = out_bwd(OUT), F16ROWS = OUT == kOutFast && N == 5;
  static_assert(MODE == MHCL_RES_SK || N <= 4, "the table of n = 5 does not fit these lanes");
  static_assert(N <= 4 ? L == 4 || L == 16 : L == 8, "lanes per token");
  constexpr int UL = (M + 2) | 1;                              // odd row lengths keep banks apart
  constexpr int AL = (R + 3) / 4 * 4 + 4;
  __shared__ float u_s[BT][UL];
  __shared__ __align__(16) float a_s[MODE == MHCL_RES_LITE ? BT : 1][AL];
  __shared__ float g_s[BWD ? BT : 1][(NN + 2 * N) | 1];
  __shared__ float v_s[BWD ? BT : 1][MP32 + 1];         // vr, zero past the last logit
  __shared__ float z_s[BWD ? BT : 1][(M + 3) | 1];      // g_z and the per-group sums of g_z u
  __shared__ float sc_s[BT];                            // scale of the token's fp16 row
  extern __shared__ float2 sk_s[];                             // {s, 1 / s} of every half step
  const int tid = threadIdx.x;
  const int64_t T = in.T, t0 = static_cast<int64_t>(blockIdx.x) * BT;

  StageSums<M, L> su;
  StageSums<1, L> ss;
  StageSums<NN, L> sr;
  StageSums<N, L> sp, sq;
  constexpr bool WIDE = L != 4;   // (the fp64 slices are those of few tokens)
  su.begin(in.u_raw, T, t0);      // (of fp64 slices: some of their halves, not used)
  ss.begin(in.sumsq, T, t0);
  if constexpr (BWD) {
    sr.begin(in.gH_res, T, t0);
    sp.begin(in.gH_pre, T, t0);
    sq.begin(in.gH_post, T, t0);
  }
  const int l = tid % L;
  const int li = L == 16 ? l / 4 : l, lj0 = L == 16 ? l % 4 : 0;   // row, column of the first entry
  const bool row_ok = li < N, cell_ok = row_ok && lj0 < N;         // (all CC entries or none)
  const int cell0 = cell_ok ? li * N + lj0 : 0;
  // residual logit kk of this lane
  auto logit = [&](int kk) { return MODE == MHCL_RES_LITE ? l + L * kk : cell0 + kk; };
  auto owns = [&](int kk) { return MODE == MHCL_RES_LITE ? l + L * kk < R : cell_ok; };
  const float a_res = in.alpha[0], a_pre = in.alpha[1], a_post = in.alpha[2];
  float bk[KK], bg[GG], a_gate[GG];
#pragma unroll
  for (int kk = 0; kk < KK; ++kk) bk[kk] = in.b[owns(kk) ? logit(kk) : 0];
#pragma unroll
  for (int gi = 0; gi < GG; ++gi) {   // gate l + L gi of pre | post
    const int gt = l + L * gi < 2 * N ? l + L * gi : 0;
    bg[gi] = in.b[R + gt];
    a_gate[gi] = gt < N ? a_pre : a_post;
  }
  uint32_t mask[CC], pbits[KK];
  if constexpr (MODE == MHCL_RES_LITE) {
#pragma unroll
    for (int c = 0; c < CC; ++c)
      mask[c] = cell_ok ? select_mask<N>(cell0 + c, std::make_integer_sequence<int, NN>{}) : 0u;
#pragma unroll
    for (int kk = 0; kk < KK; ++kk)
      pbits[kk] = BWD ? select_perm<N>(l + L * kk, std::make_integer_sequence<int, R>{}) : 0u;
  }
  if (WIDE && in.wide) {
    stage_wide<M, L>(in.u_raw, in.parts, T, t0, &u_s[0][0], UL);
    stage_wide<1, L>(in.sumsq, in.parts, T, t0, &u_s[0][M], UL);
  } else {
    su.finish(in.parts, &u_s[0][0], UL);
    ss.finish(in.parts, &u_s[0][M], UL);
  }
  if constexpr (BWD) {
    constexpr int GL = (NN + 2 * N) | 1, PAD = MP32 - M > 0 ? MP32 - M : 1;
    sr.finish(in.gparts, &g_s[0][0], GL);
    sp.finish(in.gparts, &g_s[0][NN], GL);
    sq.finish(in.gparts, &g_s[0][NN + N], GL);
    for (int e = tid; e < BT * (MP32 - M); e += THREADS) v_s[e / PAD][M + e % PAD] = 0.f;
  }
  __syncthreads();

  {
    const int tok = tid / L;
    const int64_t t = t0 + tok;
    const bool live = t < T;
    const float *u = u_s[tok];
    const float r = rms_factor(u[M], in.nC, in.eps);

    // residual logits of this lane, softmax weights / Sinkhorn-Knopp input a, entries H of H_res
    float a[KK], uk[KK], H[CC];
    float zmax = -INFINITY;
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) {
      uk[kk] = u[owns(kk) ? logit(kk) : 0];
      a[kk] = owns(kk) ? logit_of(a_res, r, uk[kk], bk[kk]) : -INFINITY;
      zmax = fmaxf(zmax, a[kk]);
    }
    zmax = group_reduce<L>(zmax, Max{});
    if constexpr (OUT == kOutLogits) {
      float zneg = -INFINITY;
#pragma unroll
      for (int kk = 0; kk < KK; ++kk) {
        zneg = fmaxf(zneg, owns(kk) ? -a[kk] : -INFINITY);
        if (live && owns(kk)) out.z[t * M + logit(kk)] = a[kk];
      }
      zneg = group_reduce<L>(zneg, Max{});
      if (live && l == 0) out.spread[t] = zmax + zneg;
    }
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) a[kk] = owns(kk) ? expf(a[kk] - zmax) : 0.f;
    // Sinkhorn-Knopp: one pair of floats per line, columns in the even half steps, rows in the odd
    // ones; kHalf pairs per half step
    constexpr int kHalf = BT * NP;
    float2 *sk = MODE == MHCL_RES_SK ? sk_s + (tid / L) * NP : nullptr;
    if constexpr (MODE == MHCL_RES_LITE) {
      float s = 0.f;
#pragma unroll
      for (int kk = 0; kk < KK; ++kk) s += a[kk];
      s = group_reduce<L>(s, Add{});
#pragma unroll
      for (int kk = 0; kk < KK; ++kk) {
        a[kk] = a[kk] / s;
        if (owns(kk)) a_s[tok][l + L * kk] = a[kk];
      }
      __builtin_amdgcn_wave_barrier();   // (a token's lanes are one wave's: LDS serves it in order)
      const float *at = a_s[tok];
#pragma unroll
      for (int c = 0; c < CC; ++c) H[c] = 0.f;
#pragma unroll
      for (int k = 0; k < R; ++k) {   // k ascending
        const float w = at[k];
#pragma unroll
        for (int c = 0; c < CC; ++c) H[c] += (mask[c] >> k) & 1u ? w : 0.f;
      }
    } else {
#pragma unroll
      for (int c = 0; c < CC; ++c) H[c] = a[c];
      for (int it = 0; it < in.sk_iters; ++it) {
        float s[CC], inv[CC];
        column_sums<L>(H, s);
#pragma unroll
        for (int c = 0; c < CC; ++c) {
          inv[c] = L == 16 && !cell_ok ? 0.f : reciprocal(s[c]);   // (entries that are none stay 0)
          if (BWD && li == 0) sk[(2 * it) * kHalf + lj0 + c] = make_float2(s[c], inv[c]);
          H[c] *= inv[c];
        }
        const float rs = row_sum<L>(H), rinv = cell_ok ? reciprocal(rs) : 0.f;
        if (BWD && lj0 == 0 && row_ok) sk[(2 * it + 1) * kHalf + li] = make_float2(rs, rinv);
#pragma unroll
        for (int c = 0; c < CC; ++c) H[c] *= rinv;
      }
      __builtin_amdgcn_wave_barrier();
    }
    float ug[GG], gate[GG];
#pragma unroll
    for (int gi = 0; gi < GG; ++gi) {
      const int gt = l + L * gi < 2 * N ? l + L * gi : 0;
      ug[gi] = u[R + gt];
      const float zg = logit_of(a_gate[gi], r, ug[gi], bg[gi]), sg = sigmoidf(zg);
      gate[gi] = gt < N ? sg : 2.f * sg;
      if constexpr (OUT == kOutLogits) {
        if (live && l + L * gi < 2 * N) out.z[t * M + R + gt] = zg;
      }
    }

    if constexpr (!BWD) {
      if (live) {
        if (cell_ok) {
#pragma unroll
          for (int c = 0; c < CC; ++c) out.H_res[t * NN + cell0 + c] = H[c];
        }
        if (OUT == kOutLogits && out.H_pre == nullptr) return;   // (of several layers: not asked for)
#pragma unroll
        for (int gi = 0; gi < GG; ++gi) {
          const int gt = l + L * gi;
          if (gt < N) out.H_pre[t * N + gt] = gate[gi];
          else if (gt < 2 * N) out.H_post[t * N + gt - N] = gate[gi];
        }
      }
    } else {
      float *rec = out.rec + t * out.rec_ld;
      if (live) {
        if (cell_ok) {
#pragma unroll
          for (int c = 0; c < CC; ++c) rec[cell0 + c] = H[c];
        }
#pragma unroll
        for (int gi = 0; gi < GG; ++gi)
          if (l + L * gi < 2 * N) rec[NN + l + L * gi] = gate[gi];
      }
      // gradient on this lane's residual logits
      const float *g = g_s[tok];
      float gz[KK];
      if constexpr (MODE == MHCL_RES_LITE) {
        float mean = 0.f;
#pragma unroll
        for (int kk = 0; kk < KK; ++kk) {   // g_a[k] = sum_i g_H[i][sigma_k(i)]
          gz[kk] = 0.f;
#pragma unroll
          for (int i = 0; i < N; ++i) gz[kk] += g[i * N + ((pbits[kk] >> (2 * i)) & 3u)];
          mean += owns(kk) ? a[kk] * gz[kk] : 0.f;
        }
        mean = group_reduce<L>(mean, Add{});
#pragma unroll
        for (int kk = 0; kk < KK; ++kk) gz[kk] = a[kk] * (gz[kk] - mean);
      } else {
        // back through the half steps: for Y = X / s, g_X = (g_Y - sum(g_Y Y)) / s and X = Y s
        float gh[CC], p[CC], d[CC];
#pragma unroll
        for (int c = 0; c < CC; ++c) gh[c] = cell_ok ? g[cell0 + c] : 0.f;
        for (int it = in.sk_iters - 1; it >= 0; --it) {
          const float2 rs = sk[(2 * it + 1) * kHalf + (row_ok ? li : 0)];
          float2 cs[CC];
#pragma unroll
          for (int c = 0; c < CC; ++c) cs[c] = sk[(2 * it) * kHalf + lj0 + c];
#pragma unroll
          for (int c = 0; c < CC; ++c) p[c] = gh[c] * H[c];
          const float dr = row_sum<L>(p);
#pragma unroll
          for (int c = 0; c < CC; ++c) {
            gh[c] = cell_ok ? (gh[c] - dr) * rs.y : 0.f;
            H[c] = cell_ok ? H[c] * rs.x : 0.f;
            p[c] = gh[c] * H[c];
          }
          column_sums<L>(p, d);
#pragma unroll
          for (int c = 0; c < CC; ++c) {
            gh[c] = cell_ok ? (gh[c] - d[c]) * cs[c].y : 0.f;
            H[c] = cell_ok ? H[c] * cs[c].x : 0.f;
          }
        }
#pragma unroll
        for (int c = 0; c < CC; ++c) gz[c] = gh[c] * a[c];
      }
      // gradient on this lane's gates, vr = r alpha g_z and the sums (selected, not multiplied by
      // zero, where a lane has no logit or a block no token: what stands there may be infinite)
      float dot = 0.f, ga0 = 0.f, ga1 = 0.f, ga2 = 0.f, vmax = 0.f;
#pragma unroll
      for (int gi = 0; gi < GG; ++gi) {
        const int gt = l + L * gi;
        const bool ok = live && gt < 2 * N;
        const float gg = g[NN + (gt < 2 * N ? gt : 0)];
        const float gzg = !ok ? 0.f : (gt < N ? gg * gate[gi] * (1.f - gate[gi])
                                              : gg * gate[gi] * (1.f - 0.5f * gate[gi]));
        const float v = ok ? r * a_gate[gi] * gzg : 0.f;
        dot += ok ? v * ug[gi] : 0.f;
        vmax = fmaxf(vmax, fabsf(v));
        const float gag = ok ? gzg * (r * ug[gi]) : 0.f;
        if (gt < N) ga1 += gag;
        else ga2 += gag;
        if (gt < 2 * N) { z_s[tok][R + gt] = gzg; v_s[tok][R + gt] = v; }
      }
#pragma unroll
      for (int kk = 0; kk < KK; ++kk) {
        const bool ok = live && owns(kk);
        if (!ok) gz[kk] = 0.f;
        const float v = ok ? r * a_res * gz[kk] : 0.f;
        ga0 += ok ? gz[kk] * (r * uk[kk]) : 0.f;
        dot += ok ? v * uk[kk] : 0.f;
        vmax = fmaxf(vmax, fabsf(v));
        if (owns(kk)) { z_s[tok][logit(kk)] = gz[kk]; v_s[tok][logit(kk)] = v; }
      }
      dot = group_reduce<L>(dot, Add{});
      ga0 = group_reduce<L>(ga0, Add{});
      ga1 = group_reduce<L>(ga1, Add{});
      ga2 = group_reduce<L>(ga2, Add{});
      if constexpr (F16ROWS) vmax = group_reduce<L>(vmax, Max{});
      if (l == 0) {
        z_s[tok][M] = ga0;
        z_s[tok][M + 1] = ga1;
        z_s[tok][M + 2] = ga2;
        if (live) rec[NN + 2 * N] = (r * r / static_cast<float>(in.nC)) * dot;
        if constexpr (F16ROWS) {
          const float sc = vmax > 0.f ? vmax : 1.f;
          sc_s[tok] = 1.f / sc;
          if (live) rec[NN + 2 * N + 1] = sc;
        }
      }
    }
  }
  if constexpr (BWD) {
    __syncthreads();
    if constexpr (OUT == kOutFull) {
      for (int e = tid; e < BT * MP16; e += THREADS) {
        const int tk = e / MP16, m = e % MP16;
        if (t0 + tk < T) out.vr[(t0 + tk) * MP16 + m] = v_s[tk][m];
      }
    } else {
      // (tokens up to the next multiple of 64 exist in these arrays; past T they are zeros)
      // rows [Tpad][MP32]: eight logits of a token per thread; then, by the next threads, tokens
      // innermost [Tpad/32][MP16][32]: eight tokens of a logit
      constexpr int kRows = BT * MP32 / 8, kCols = MP16 * BT / 8;
      for (int e = tid; e < kRows + kCols; e += THREADS) {
        u32x4 hi, lo;
        float v[8];
        if (e < kRows) {
          const int tk = e / (MP32 / 8), v8 = e % (MP32 / 8);
          const float inv = F16ROWS ? sc_s[tk] : 1.f;
#pragma unroll
          for (int i = 0; i < 8; ++i) v[i] = v_s[tk][8 * v8 + i] * inv;
          split8(v, std::bool_constant<F16ROWS>{}, hi, lo);
          const size_t off = static_cast<size_t>(t0 + tk) * MP32 + 8 * v8;
          *reinterpret_cast<u32x4 *>(out.vr_hi + off) = hi;
          *reinterpret_cast<u32x4 *>(out.vr_lo + off) = lo;
        } else {
          const int half = (e - kRows) / (4 * MP16), m = ((e - kRows) / 4) % MP16, tg = (e - kRows) & 3;
#pragma unroll
          for (int i = 0; i < 8; ++i) v[i] = v_s[32 * half + tg * 8 + i][m];
          split8(v, std::false_type{}, hi, lo);
          const size_t off = ((static_cast<size_t>(blockIdx.x) * (BT / 32) + half) * MP16 + m) * 32 + tg * 8;
          *reinterpret_cast<u32x4 *>(out.vrT_hi + off) = hi;
          *reinterpret_cast<u32x4 *>(out.vrT_lo + off) = lo;
        }
      }
    }
    // sums over the block's tokens (zeros past T), pairwise, by the last threads
    for (int m = THREADS - 1 - tid; m < M + 3; m += THREADS)
      out.gz_sums[static_cast<int64_t>(blockIdx.x) * (M + 3) + m] =
          pairwise_sum<BT>([&](int tk) { return z_s[tk][m]; });
  }
}

template <int N, int MODE, int OUT, int L>
__global__ __launch_bounds__(kTokThreads<L>) void token_stage_kernel(TokenIn in, TokenOut out) {
  token_stage<N, MODE, OUT, L>(in, out);
}
// gridDim.y layers of a stack side by side: H_res, logits and spreads in stacks [layer][T][...]
template <int N, int MODE, int L>
__global__ __launch_bounds__(kTokThreads<L>) void token_layers_kernel(TokenIn in, TokenOut out, JointLayers layers) {
  const int l = blockIdx.y;
  in.u_raw += l * layers.stride;
  in.sumsq += l * layers.stride;
  in.b = layers.b[l];
  in.alpha = layers.alpha[l];
  out.H_res += l * in.T * (N * N);
  out.z += l * in.T * Dims<N, MODE>::M;
  out.spread += l * in.T;
  token_stage<N, MODE, kOutLogits, L>(in, out);
}
// the forward's stage, and from block p.first on the pre-aggregate
template <int N, int MODE, int L, typename IO>
__global__ __launch_bounds__(kTokThreads<L>) void token_pre_kernel(TokenIn in, TokenOut out, PreArgs p) {
  if (blockIdx.x < p.first)
    token_stage<N, MODE, kOutForward, L>(in, out);
  else
    pre_from_slices<IO, N, kTokThreads<L>>(p, blockIdx.x - p.first, in.u_raw, in.sumsq, in.parts, in.wide, in.b,
                                           in.alpha, in.eps, in.T, Dims<N, MODE>::R);
}

template <int OUT>
hipError_t launch_token_stage(const mhcl_desc &d, const TokenIn &in,
                              const TokenOut &out, hipStream_t s) {
  const bool many = token_stage_many(d, out_bwd(OUT));
  const int64_t blocks64 = (d.T + 63) / 64;
  const unsigned blocks = static_cast<unsigned>(many ? blocks64 : 2 * blocks64);
  auto go = [&](auto nn, auto mm) {
    constexpr int N = decltype(nn)::value, MODE = decltype(mm)::value;
    constexpr int LF = N <= 4 ? 16 : 8;   // lanes per token with few tokens
    auto kern = token_stage_kernel<N, MODE, OUT, LF>;
    int threads = kTokThreads<LF>, per_iter = kSkPerIter<N, MODE, OUT, LF>;
    if constexpr (N <= 4 && (MODE == MHCL_RES_LITE || !out_bwd(OUT))) {
      if (many) {
        kern = token_stage_kernel<N, MODE, OUT, 4>;
        threads = kTokThreads<4>;
        per_iter = kSkPerIter<N, MODE, OUT, 4>;
      }
    }
    const size_t lds = static_cast<size_t>(per_iter) * d.sk_iters * sizeof(float);
    if (MODE == MHCL_RES_SK && lds > 16 * 1024) {   // (with the static arrays it may pass 64 KiB)
      // the kernel's limit, not this call's need: another thread may be about to launch with more iterations
      const int most = per_iter * kMaxSkIters * static_cast<int>(sizeof(float));
      hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kern),
                                         hipFuncAttributeMaxDynamicSharedMemorySize, most);
      if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(kern, dim3(blocks), dim3(threads), MODE == MHCL_RES_SK ? lds : 0, s, in, out);
    return hipGetLastError();
  };
  using L = std::integral_constant<int, MHCL_RES_LITE>;
  using S = std::integral_constant<int, MHCL_RES_SK>;
  const bool lite = d.res_mode == MHCL_RES_LITE;
  switch (d.n) {
    case 1: return lite ? go(std::integral_constant<int, 1>{}, L{}) : go(std::integral_constant<int, 1>{}, S{});
    case 2: return lite ? go(std::integral_constant<int, 2>{}, L{}) : go(std::integral_constant<int, 2>{}, S{});
    case 3: return lite ? go(std::integral_constant<int, 3>{}, L{}) : go(std::integral_constant<int, 3>{}, S{});
    case 4: return lite ? go(std::integral_constant<int, 4>{}, L{}) : go(std::integral_constant<int, 4>{}, S{});
    case 5: return lite ? hipErrorInvalidValue : go(std::integral_constant<int, 5>{}, S{});
  }
  return hipErrorInvalidValue;
}

// ---------------------------------------------------------------------------
// One token per lane, for many tokens.  In the Sinkhorn-Knopp form a group of lanes shortens the chain of one
// token but repeats its divisions (every lane of a column divides by that column's sum): about 28
// instructions per iteration in each of 16 lanes at n <= 4 and 90 in each of eight at n = 5, against
// 24 (n = 1) to 190 (n = 5) in one lane.  Once there are waves enough to hide the chain the count of
// instructions is what bounds the stage; so it is, with far more tokens, in the forward of the permutation
// form.  `token_per_lane` has the lines and both sides' times.
struct LaneParams {
  float alpha_res, alpha_pre, alpha_post, eps;
  int nC, sk_iters;
};

template <int N>
__device__ __forceinline__ void lane_gates(const float *u, float r, const float *b, const LaneParams &p,
                                           float *H_pre, float *H_post) {
#pragma unroll
  for (int j = 0; j < N; ++j) {
    H_pre[j] = sigmoidf(logit_of(p.alpha_pre, r, u[j], b[j]));
    H_post[j] = 2.f * sigmoidf(logit_of(p.alpha_post, r, u[N + j], b[N + j]));
  }
}

// a weight into the entries of permutation K
template <int N, int K, int... I>
__device__ __forceinline__ void add_perm(float w, float *H, std::integer_sequence<int, I...>) {
  ((H[std::integral_constant<int, I * N + Perm<N>::tab.s[K][I]>::value] += w), ...);
}
// softmax over all N! logits, a = its weights; H_res = sum_k a_k P_k, k ascending
template <int N, int... K>
__device__ __forceinline__ void lite_token(const float *u, float sumsq, const float *b,
                                           const LaneParams &p, float *H_res, float *H_pre,
                                           float *H_post, float *a, std::integer_sequence<int, K...>) {
  constexpr int R = sizeof...(K);
  const float r = rms_factor(sumsq, p.nC, p.eps);
  float zmax = -INFINITY, s = 0.f;
#pragma unroll
  for (int k = 0; k < R; ++k) {
    a[k] = logit_of(p.alpha_res, r, u[k], b[k]);
    zmax = fmaxf(zmax, a[k]);
  }
#pragma unroll
  for (int k = 0; k < R; ++k) { a[k] = expf(a[k] - zmax); s += a[k]; }
#pragma unroll
  for (int k = 0; k < R; ++k) a[k] = a[k] / s;
#pragma unroll
  for (int e = 0; e < N * N; ++e) H_res[e] = 0.f;
  (add_perm<N, K>(a[K], H_res, std::make_integer_sequence<int, N>{}), ...);
  lane_gates<N>(u + R, r, b + R, p, H_pre, H_post);
}

// Sinkhorn-Knopp: the 2 sk_iters N divisors go to `sums` if that is not null; a = exp(z - max), the input of the
// iteration; returns r.
template <int N>
__device__ __forceinline__ float sk_token(const float *u, float sumsq, const float *b, const LaneParams &p,
                                          float *H_res, float *H_pre, float *H_post, float *a,
                                          float *sums) {
  constexpr int R = N * N;
  const float r = rms_factor(sumsq, p.nC, p.eps);
  float zmax = -INFINITY;
#pragma unroll
  for (int k = 0; k < R; ++k) {
    a[k] = logit_of(p.alpha_res, r, u[k], b[k]);
    zmax = fmaxf(zmax, a[k]);
  }
#pragma unroll
  for (int k = 0; k < R; ++k) { a[k] = expf(a[k] - zmax); H_res[k] = a[k]; }
  for (int it = 0; it < p.sk_iters; ++it) {
#pragma unroll
    for (int j = 0; j < N; ++j) {
      float s = 0.f;
#pragma unroll
      for (int i = 0; i < N; ++i) s += H_res[i * N + j];
      const float inv = reciprocal(s);
#pragma unroll
      for (int i = 0; i < N; ++i) H_res[i * N + j] *= inv;
      if (sums) sums[(2 * it) * N + j] = s;
    }
#pragma unroll
    for (int i = 0; i < N; ++i) {
      float s = 0.f;
#pragma unroll
      for (int j = 0; j < N; ++j) s += H_res[i * N + j];
      const float inv = reciprocal(s);
#pragma unroll
      for (int j = 0; j < N; ++j) H_res[i * N + j] *= inv;
      if (sums) sums[(2 * it + 1) * N + i] = s;
    }
  }
  lane_gates<N>(u + R, r, b + R, p, H_pre, H_post);
  return r;
}

// g_z from the gradients on the coefficients, back through the half steps as in
// token_stage_kernel.  g and H are used up.
template <int N>
__device__ __forceinline__ void sk_token_bwd(float *g, const float *gH_pre, const float *gH_post,
                                             const float *a, float *H, const float *H_pre,
                                             const float *H_post, const float *sums, int sk_iters,
                                             float *g_z) {
  constexpr int R = N * N;
  // the divisors of an iteration (private memory: rows, then columns) are fetched one iteration ahead
  float row[N], col[N], row_next[N], col_next[N];
  auto fetch = [&](int it, float (&rows)[N], float (&cols)[N]) {
#pragma unroll
    for (int i = 0; i < N; ++i) {
      cols[i] = sums[(2 * it) * N + i];
      rows[i] = sums[(2 * it + 1) * N + i];
    }
  };
  fetch(sk_iters - 1, row, col);
  for (int it = sk_iters - 1; it >= 0; --it) {
    fetch(it > 0 ? it - 1 : 0, row_next, col_next);
#pragma unroll
    for (int i = 0; i < N; ++i) {
      const float inv = reciprocal(row[i]);
      float d = 0.f;
#pragma unroll
      for (int j = 0; j < N; ++j) d += g[i * N + j] * H[i * N + j];
#pragma unroll
      for (int j = 0; j < N; ++j) {
        g[i * N + j] = (g[i * N + j] - d) * inv;
        H[i * N + j] *= row[i];
      }
    }
#pragma unroll
    for (int j = 0; j < N; ++j) {
      const float inv = reciprocal(col[j]);
      float d = 0.f;
#pragma unroll
      for (int i = 0; i < N; ++i) d += g[i * N + j] * H[i * N + j];
#pragma unroll
      for (int i = 0; i < N; ++i) {
        g[i * N + j] = (g[i * N + j] - d) * inv;
        H[i * N + j] *= col[j];
      }
    }
#pragma unroll
    for (int i = 0; i < N; ++i) { row[i] = row_next[i]; col[i] = col_next[i]; }
  }
#pragma unroll
  for (int e = 0; e < R; ++e) g_z[e] = g[e] * a[e];
#pragma unroll
  for (int j = 0; j < N; ++j) {
    g_z[R + j] = gH_pre[j] * H_pre[j] * (1.f - H_pre[j]);
    g_z[R + N + j] = gH_post[j] * H_post[j] * (1.f - 0.5f * H_post[j]);
  }
}

// the slices of token t's logits and sum of squares, added in order; returns the latter
template <int M>
__device__ __forceinline__ float lane_logits(const TokenIn &in, int64_t t, float (&u)[M]) {
  float ssq = in.sumsq[t];
#pragma unroll
  for (int m = 0; m < M; ++m) u[m] = in.u_raw[t * M + m];
  for (int pt = 1; pt < in.parts; ++pt) {
    ssq += in.sumsq[pt * in.T + t];
#pragma unroll
    for (int m = 0; m < M; ++m) u[m] += in.u_raw[(pt * in.T + t) * M + m];
  }
  return ssq;
}

// (blocks of 256: 64 and 128 leave some compute units with a wave more than others, 36 / 44 / 43 us for
// mhcl_coeffs at n = 4, C = 64, 114688 tokens, 32 iterations)
constexpr int kLaneThreads = 256;
template <int N, int MODE>
__global__ __launch_bounds__(kLaneThreads) void lane_coeffs_kernel(TokenIn in, TokenOut out) {
  constexpr int R = Dims<N, MODE>::R, M = Dims<N, MODE>::M, NN = N * N;
  const int64_t t = static_cast<int64_t>(blockIdx.x) * kLaneThreads + threadIdx.x;
  if (t >= in.T) return;
  float u[M], a[R], H[NN], Hp[N], Hq[N];
  const float ssq = lane_logits(in, t, u);
  const LaneParams p{in.alpha[0], in.alpha[1], in.alpha[2], in.eps, in.nC, in.sk_iters};
  if constexpr (MODE == MHCL_RES_LITE)
    lite_token<N>(u, ssq, in.b, p, H, Hp, Hq, a, std::make_integer_sequence<int, R>{});
  else
    sk_token<N>(u, ssq, in.b, p, H, Hp, Hq, a, nullptr);
#pragma unroll
  for (int e = 0; e < NN; ++e) out.H_res[t * NN + e] = H[e];
#pragma unroll
  for (int j = 0; j < N; ++j) { out.H_pre[t * N + j] = Hp[j]; out.H_post[t * N + j] = Hq[j]; }
}

// Outputs as token_stage_kernel<kOutFast>, for one slice of the dot products; one wave per block, the
// sums over its 64 tokens by a butterfly.
template <int N>
__global__ __launch_bounds__(64) void sk_bwd_kernel(TokenIn in, TokenOut out) {
  constexpr int R = N * N, M = R + 2 * N;
  constexpr int MP32 = (M + 31) / 32 * 32, MP16 = (M + 15) / 16 * 16;
  constexpr bool F16ROWS = N == 5;
  const int64_t t = static_cast<int64_t>(blockIdx.x) * 64 + threadIdx.x;   // up to the next multiple of 64
  const int64_t blk = t >> 5;
  const int tin = static_cast<int>(t & 31);
  const bool live = t < in.T;
  const int64_t tl = live ? t : in.T - 1;   // (padding lanes go over the last token again and drop it)
  float u[M], a[R], H[R], Hp[N], Hq[N], gz[M + 3], gr[R], gp[N], gq[N];
  float sums[2 * kMaxSkIters * N];
  const float ssq = lane_logits(in, tl, u);
#pragma unroll
  for (int e = 0; e < R; ++e) gr[e] = in.gH_res[tl * R + e];
#pragma unroll
  for (int j = 0; j < N; ++j) { gp[j] = in.gH_pre[tl * N + j]; gq[j] = in.gH_post[tl * N + j]; }
  const LaneParams p{in.alpha[0], in.alpha[1], in.alpha[2], in.eps, in.nC, in.sk_iters};
  const float r = sk_token<N>(u, ssq, in.b, p, H, Hp, Hq, a, sums);
  float *rec = out.rec + t * out.rec_ld;
  if (live) {
#pragma unroll
    for (int e = 0; e < R; ++e) rec[e] = H[e];
#pragma unroll
    for (int j = 0; j < N; ++j) { rec[R + j] = Hp[j]; rec[R + N + j] = Hq[j]; }
  }
  sk_token_bwd<N>(gr, gp, gq, a, H, Hp, Hq, sums, in.sk_iters, gz);
  auto alpha_of = [&](int m) { return m < R ? p.alpha_res : (m < R + N ? p.alpha_pre : p.alpha_post); };
  float inv_s = 1.f;
  if constexpr (F16ROWS) {
    float vmax = 0.f;
#pragma unroll
    for (int m = 0; m < M; ++m) vmax = fmaxf(vmax, fabsf(r * alpha_of(m) * (live ? gz[m] : 0.f)));
    const float sc = vmax > 0.f ? vmax : 1.f;
    inv_s = 1.f / sc;
    if (live) rec[R + 2 * N + 1] = sc;
  }
  float ga[3] = {0.f, 0.f, 0.f}, dot = 0.f;
  u32x4 rows_hi[MP32 / 8], rows_lo[MP32 / 8];   // the token's vr row, eight 16-bit parts per vector
#pragma unroll
  for (int v8 = 0; v8 < MP32 / 8; ++v8) {
    float v[8], vs[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int m = 8 * v8 + e;
      v[e] = 0.f;
      if (m < M) {
        if (!live) gz[m] = 0.f;
        v[e] = r * alpha_of(m) * gz[m];
        ga[m < R ? 0 : (m < R + N ? 1 : 2)] += live ? gz[m] * (r * u[m]) : 0.f;
        dot += v[e] * u[m];
        if (!live) v[e] = 0.f;
      }
      vs[e] = v[e] * inv_s;
    }
    u32x4 hi, lo;
    split8(v, std::false_type{}, hi, lo);
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int m = 8 * v8 + e;
      if (m < MP16) {
        out.vrT_hi[(blk * MP16 + m) * 32 + tin] = static_cast<uint16_t>(hi[e >> 1] >> (16 * (e & 1)));
        out.vrT_lo[(blk * MP16 + m) * 32 + tin] = static_cast<uint16_t>(lo[e >> 1] >> (16 * (e & 1)));
      }
    }
    if constexpr (F16ROWS) split8(vs, std::true_type{}, hi, lo);
    rows_hi[v8] = hi;
    rows_lo[v8] = lo;
  }
#pragma unroll
  for (int v8 = 0; v8 < MP32 / 8; ++v8) {
    reinterpret_cast<u32x4 *>(out.vr_hi + t * MP32)[v8] = rows_hi[v8];
    reinterpret_cast<u32x4 *>(out.vr_lo + t * MP32)[v8] = rows_lo[v8];
  }
  if (live) rec[R + 2 * N] = (r * r / static_cast<float>(in.nC)) * dot;
#pragma unroll
  for (int g = 0; g < 3; ++g) gz[M + g] = ga[g];
#pragma unroll
  for (int m = 0; m < M + 3; ++m) {
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) gz[m] += __shfl_xor(gz[m], off, 64);
  }
  if (threadIdx.x == 0) {
#pragma unroll
    for (int m = 0; m < M + 3; ++m) out.gz_sums[static_cast<int64_t>(blockIdx.x) * (M + 3) + m] = gz[m];
  }
}

hipError_t launch_token_pre(const mhcl_desc &d, const TokenIn &in, const TokenOut &out, const void *x, void *h,
                            hipStream_t s) {
  const bool many = token_stage_many(d, false);
  const int64_t blocks64 = (d.T + 63) / 64;
  auto go = [&](auto nn, auto mm) {
    constexpr int N = decltype(nn)::value, MODE = decltype(mm)::value;
    constexpr int LF = N <= 4 ? 16 : 8;
    auto with = [&](auto ll, auto io) {
      constexpr int L = decltype(ll)::value;
      const PreArgs p{x, h, static_cast<unsigned>(many ? blocks64 : 2 * blocks64), d.C};
      hipLaunchKernelGGL((token_pre_kernel<N, MODE, L, decltype(io)>),
                         dim3(p.first + pre_blocks(d, kTokThreads<L>)), dim3(kTokThreads<L>), 0, s, in, out, p);
      return hipGetLastError();
    };
    return dispatch_io(d.io_dtype, [&](auto io) {
      if constexpr (N <= 4)
        if (many) return with(std::integral_constant<int, 4>{}, io);
      return with(std::integral_constant<int, LF>{}, io);
    });
  };
  using L = std::integral_constant<int, MHCL_RES_LITE>;
  using S = std::integral_constant<int, MHCL_RES_SK>;
  const bool lite = d.res_mode == MHCL_RES_LITE;
  switch (d.n) {
    case 1: return lite ? go(std::integral_constant<int, 1>{}, L{}) : go(std::integral_constant<int, 1>{}, S{});
    case 2: return lite ? go(std::integral_constant<int, 2>{}, L{}) : go(std::integral_constant<int, 2>{}, S{});
    case 3: return lite ? go(std::integral_constant<int, 3>{}, L{}) : go(std::integral_constant<int, 3>{}, S{});
    case 4: return lite ? go(std::integral_constant<int, 4>{}, L{}) : go(std::integral_constant<int, 4>{}, S{});
    case 5: return lite ? hipErrorInvalidValue : go(std::integral_constant<int, 5>{}, S{});
  }
  return hipErrorInvalidValue;
}

hipError_t launch_lane_coeffs(const mhcl_desc &d, const TokenIn &in, const TokenOut &out, hipStream_t s) {
  auto go = [&](auto nn, auto mm) {
    hipLaunchKernelGGL((lane_coeffs_kernel<decltype(nn)::value, decltype(mm)::value>),
                       dim3(static_cast<unsigned>((d.T + kLaneThreads - 1) / kLaneThreads)),
                       dim3(kLaneThreads), 0, s, in, out);
    return hipGetLastError();
  };
  using L = std::integral_constant<int, MHCL_RES_LITE>;
  using S = std::integral_constant<int, MHCL_RES_SK>;
  const bool lite = d.res_mode == MHCL_RES_LITE;
  switch (d.n) {
    case 1: return lite ? go(std::integral_constant<int, 1>{}, L{}) : go(std::integral_constant<int, 1>{}, S{});
    case 2: return lite ? go(std::integral_constant<int, 2>{}, L{}) : go(std::integral_constant<int, 2>{}, S{});
    case 3: return lite ? go(std::integral_constant<int, 3>{}, L{}) : go(std::integral_constant<int, 3>{}, S{});
    case 4: return lite ? go(std::integral_constant<int, 4>{}, L{}) : go(std::integral_constant<int, 4>{}, S{});
    case 5: return lite ? hipErrorInvalidValue : go(std::integral_constant<int, 5>{}, S{});
  }
  return hipErrorInvalidValue;
}

hipError_t launch_sk_bwd(const mhcl_desc &d, const TokenIn &in, const TokenOut &out, hipStream_t s) {
  auto go = [&](auto nn) {
    hipLaunchKernelGGL(sk_bwd_kernel<decltype(nn)::value>, dim3(static_cast<unsigned>((d.T + 63) / 64)),
                       dim3(64), 0, s, in, out);
    return hipGetLastError();
  };
  switch (d.n) {
    case 1: return go(std::integral_constant<int, 1>{});
    case 2: return go(std::integral_constant<int, 2>{});
    case 3: return go(std::integral_constant<int, 3>{});
    case 4: return go(std::integral_constant<int, 4>{});
    case 5: return go(std::integral_constant<int, 5>{});
  }
  return hipErrorInvalidValue;
}

TokenIn token_in(const mhcl_desc &d, const RawSums &raw, const float *b, const float *alpha) {
  TokenIn in{};
  in.u_raw = raw.u_raw; in.sumsq = raw.sumsq; in.parts = raw.parts; in.wide = raw.wide;
  in.b = b; in.alpha = alpha;
  in.nC = d.n * d.C; in.eps = d.eps; in.sk_iters = d.sk_iters; in.T = d.T;
  return in;
}

}  // namespace

// Four lanes per token against sixteen, measured (n = 4, the calls at C = 64 where this stage
// dominates): forward 25.4 / 23.2 us at 512 tokens, 23.5 / 25.5 at 16384, 46 / 48 at 65536; backward
// 32.0 / 29.7, 38.3 / 38.8, 91.5 / 95.2.  The Sinkhorn-Knopp backward is a chain of 4 sk_iters sums
// per token, which sixteen lanes walk faster at every count (65.8 against 69.3 us at 32768 tokens).
bool token_stage_many(const mhcl_desc &d, bool backward) {
  return d.n <= 4 && d.T >= 16384 && !(backward && d.res_mode == MHCL_RES_SK);
}

// One token per lane from so many token-iterations on (eight iterations' worth is the rest of the stage).
// Group of lanes / one lane, us per call at C = 64, 20 iterations: mhcl_coeffs n = 4 23.3 / 26.8 at
// 65536 tokens, 41.2 / 32.4 at 131072; n = 1 13.6 / 16.3 and 18.3 / 13.2; n = 5 18.3 / 22.1 at 16384,
// 84 / 45 at 131072.  mhcl_bwd_fused n = 1 29.0 / 24.7 at 16384, 103 / 58 at 131072; n = 2 45.8 /
// 46.4 at 32768, 120 / 85 at 131072; n = 3 70.1 / 72.5 at 49152, 144 / 128 at 131072; n = 4 101 / 109 at
// 65536, 274 / 263 at 196608; n = 5 112 / 114 at 32768, 344 / 297 at 131072 (with 32 iterations 513 / 329).
// Permutation form, forward, 2^20 tokens of C = 64, the stage alone: n = 1 18.7 / 7.9 us, n = 4 93 / 68 (equal near 200000).
bool token_per_lane(const mhcl_desc &d, bool backward) {
  constexpr int64_t kForward[] = {0, 1800000, 1500000, 1900000, 2200000, 800000};
  constexpr int64_t kBackward[] = {0, 450000, 1100000, 1750000, 5500000, 950000};
  if (d.n < 1 || d.n > 5) return false;
  if (d.res_mode == MHCL_RES_LITE) return d.n <= 4 && !backward && d.T >= 200000;
  if (d.res_mode != MHCL_RES_SK) return false;
  return d.T * (d.sk_iters + 8) >= (backward ? kBackward : kForward)[d.n];
}

// one per block: the blocks cover tokens up to the next multiple of 64, as the readers of vr do
int64_t gz_rows(const mhcl_desc &d, bool fast) {
  const int64_t blocks64 = (d.T + 63) / 64;
  if (coeffs_group_ok(d) || token_stage_many(d, true) || (fast && token_per_lane(d, true))) return blocks64;
  return 2 * blocks64;
}

int64_t gz_rows_reserved(const mhcl_desc &d) {
  const int64_t blocks64 = (d.T + 63) / 64;
  return coeffs_group_ok(d) ? blocks64 : 2 * blocks64;
}

hipError_t launch_token_coeffs(const mhcl_desc &d, const RawSums &raw, const float *b,
                               const float *alpha, float *H_res, float *H_pre, float *H_post,
                               hipStream_t s) {
  TokenOut out{};
  out.H_res = H_res; out.H_pre = H_pre; out.H_post = H_post;
  const TokenIn in = token_in(d, raw, b, alpha);
  // (a lane reads its slices one after the other, in fp32)
  if (raw.parts < 8 && !raw.wide && token_per_lane(d, false)) return launch_lane_coeffs(d, in, out, s);
  return launch_token_stage<kOutForward>(d, in, out, s);
}

// Two launches / one, us for mhcl_fwd_coeffs_pre, by the 16-byte chunks of h.  Permutation form, n = 4: C = 1024, 3000 tokens 18.1 /
// 16.5, 5120 (655 thousand chunks) 23.5 / 22.6, 7000 28.2 / 27.9, 8000 (a million) 30.6 / 30.7, C = 768, 8192 tokens (786 thousand)
// 25.8 / 26.4 (C = 4096 still gains there: 1500 tokens 28.5 / 26.8); fp64 slices, bf16, C = 1000, 5300 tokens (662 thousand) 50.7 / 50.3,
// 6000 51.9 / 52.7; n = 3, f32, C = 1024, 2600 tokens (666 thousand) 21.9 / 21.4, 3000 23.1 / 23.2, 6000 36.7 / 38.7.  f32 at n = 4,
// whose projection is the longer: C = 768, 4096 tokens (786 thousand) 34.8 / 33.2, 8000 60.1 / 59.6, C = 4096, 3000 tokens (3 million)
// 109 / 107, C = 2048, 8000 tokens (4 million) 144 / 148.  n = 2, C = 512, 9000 tokens 23.3 / 23.8 (both forward calls); four lanes per token, C = 64,
// 16384 tokens (131 thousand) 19.2 / 16.5, 65536 tokens 36.8 / 37.6.  Sinkhorn-Knopp, whose stage is the longer, C = 768: 3001
// tokens 25.3 / 23.5, 65536 344 / 340.
bool token_coeffs_pre_ok(const mhcl_desc &d, const RawSums &raw) {
  if (coeffs_group_ok(d) || (raw.parts < 8 && !raw.wide && token_per_lane(d, false))) return false;
  const int64_t chunks = pre_chunks(d);
  if (d.res_mode == MHCL_RES_SK) return chunks <= (1 << 23);
  if (token_stage_many(d, false) || d.n <= 2) return chunks <= (1 << 18);
  return chunks <= (raw.wide && d.io_dtype == MHCL_F32 && d.n == 4 ? 3 << 20 : 5 << 17);
}
hipError_t launch_token_coeffs_pre(const mhcl_desc &d, const RawSums &raw, const float *b, const float *alpha,
                                   const void *x, float *H_res, float *H_pre, float *H_post, void *h,
                                   hipStream_t s) {
  TokenOut out{};
  out.H_res = H_res; out.H_pre = H_pre; out.H_post = H_post;
  return launch_token_pre(d, token_in(d, raw, b, alpha), out, x, h, s);
}

bool token_logits_ok(const mhcl_desc &d, const RawSums &raw) {
  return !coeffs_group_ok(d) && !(raw.parts < 8 && !raw.wide && token_per_lane(d, false));
}
hipError_t launch_token_coeffs_logits(const mhcl_desc &d, const RawSums &raw, const float *b,
                                      const float *alpha, float *H_res, float *H_pre, float *H_post,
                                      float *z, float *spread, hipStream_t s) {
  TokenOut out{};
  out.H_res = H_res; out.H_pre = H_pre; out.H_post = H_post; out.z = z; out.spread = spread;
  return launch_token_stage<kOutLogits>(d, token_in(d, raw, b, alpha), out, s);
}

// Where the launches of several layers are shared: the forms whose per-token stage writes the logits, and whose
// projection takes W as it is.
bool joint_layers_ok(const mhcl_desc &d) {
  if (d.T == 0 || coeffs_group_ok(d) || token_per_lane(d, false)) return false;
  return proj_fullprec_used(d) || proj_mfma_direct(d);
}
hipError_t launch_token_layers(const mhcl_desc &d, const RawSums &raw, const JointLayers &layers, int count, float *H_res,
                               float *z, float *spread, hipStream_t s) {
  const TokenIn in = token_in(d, raw, nullptr, nullptr);
  TokenOut out{};
  out.H_res = H_res; out.z = z; out.spread = spread;
  // Four lanes per token from the tokens of all layers on where sums over rows and columns are all that lanes share
  // (six layers of 8192 tokens, sixteen / four, us: n = 4 16.5 / 12.4, n = 3, four layers 11.1 / 7.4; n = 2, six of 4000 8.9 / 6.8).
  // Not over fp64 slices, and not in the permutation form, whose weights would be summed in another order.
  const bool many = token_stage_many(d, false) ||
                    (d.res_mode == MHCL_RES_SK && d.n <= 4 && !raw.wide && d.T * count >= 16384);
  const int64_t blocks64 = (d.T + 63) / 64;
  const dim3 grid(static_cast<unsigned>(many ? blocks64 : 2 * blocks64), count);
  auto go = [&](auto nn, auto mm) {
    constexpr int N = decltype(nn)::value, MODE = decltype(mm)::value, LF = N <= 4 ? 16 : 8;
    auto kern = token_layers_kernel<N, MODE, LF>;
    int threads = kTokThreads<LF>;
    if constexpr (N <= 4) {
      if (many) {
        kern = token_layers_kernel<N, MODE, 4>;
        threads = kTokThreads<4>;
      }
    }
    hipLaunchKernelGGL(kern, grid, dim3(threads), 0, s, in, out, layers);
    return hipGetLastError();
  };
  using LI = std::integral_constant<int, MHCL_RES_LITE>;
  using SK = std::integral_constant<int, MHCL_RES_SK>;
  const bool lite = d.res_mode == MHCL_RES_LITE;
  switch (d.n) {
    case 1: return lite ? go(std::integral_constant<int, 1>{}, LI{}) : go(std::integral_constant<int, 1>{}, SK{});
    case 2: return lite ? go(std::integral_constant<int, 2>{}, LI{}) : go(std::integral_constant<int, 2>{}, SK{});
    case 3: return lite ? go(std::integral_constant<int, 3>{}, LI{}) : go(std::integral_constant<int, 3>{}, SK{});
    case 4: return lite ? go(std::integral_constant<int, 4>{}, LI{}) : go(std::integral_constant<int, 4>{}, SK{});
    case 5: return lite ? hipErrorInvalidValue : go(std::integral_constant<int, 5>{}, SK{});
  }
  return hipErrorInvalidValue;
}

hipError_t launch_token_bwd_fast(const mhcl_desc &d, const float *b, const float *alpha,
                                 const FastBwdWs &w, hipStream_t s) {
  // what the kernels fix at compile time against what pass 2 reads: row lengths, and fp16 rows with
  // their scale at n = 5 exactly where bwd_out_w16_kernel takes them
  const int M = res_logits(d) + 2 * d.n, record = d.n * d.n + 2 * d.n + (d.n == 5 ? 2 : 1);
  if (w.MP32 != (M + 31) / 32 * 32 || w.MP16 != (M + 15) / 16 * 16 || w.CP < record ||
      (d.n == 5) != fast_bwd_whi(d))
    return hipErrorInvalidValue;
  TokenIn in = token_in(d, w.raw(), b, alpha);
  in.gH_res = w.gH_res; in.gH_pre = w.gH_pre; in.gH_post = w.gH_post; in.gparts = w.gparts;
  TokenOut out{};
  out.rec = w.cpk; out.rec_ld = w.CP;
  out.vr_hi = w.vr_hi; out.vr_lo = w.vr_lo; out.vrT_hi = w.vrT_hi; out.vrT_lo = w.vrT_lo;
  out.gz_sums = w.gz;
  if (token_per_lane(d, true)) {
    if (w.gparts != 1 || w.wide_sums) return hipErrorInvalidValue;   // (more only up to 8192 tokens)
    return launch_sk_bwd(d, in, out, s);
  }
  return launch_token_stage<kOutFast>(d, in, out, s);
}

hipError_t launch_token_bwd_full(const mhcl_desc &d, const RawSums &raw, const float *b,
                                 const float *alpha, const float *g_H_res, const float *g_H_pre,
                                 const float *g_H_post, const BwdTokenBufs &o, hipStream_t s) {
  TokenIn in = token_in(d, raw, b, alpha);
  in.gH_res = g_H_res; in.gH_pre = g_H_pre; in.gH_post = g_H_post; in.gparts = 1;
  TokenOut out{};
  out.rec = o.rec; out.rec_ld = token_rec_floats(d.n); out.vr = o.vr; out.gz_sums = o.gz;
  return launch_token_stage<kOutFull>(d, in, out, s);
}

}  // namespace mhcl
