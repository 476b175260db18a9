// Per-token coefficients of the table forms: a = softmax over K logits,
// H_res = sum_k a_k P_k over the K permutations of a table [K][n] (Sec. 5, the
// paragraph on larger n: a run-time subset, n up to 8, K up to 128; also the
// full form at n = 5, whose 120 permutations make the unrolled compile-time
// sums too large for the registers); gates as in Sec. 3.2.
// Eight lanes per token: forward coefficients and the stage of the backward between the
// reductions over C and the stream outputs.
#include "mhcl_common.h"
#include "mhcl_internal.h"
#include "mhcl_mfma.h"
#include "mhcl_pre.h"

namespace mhcl {

namespace {

// ---------------------------------------------------------------------------
// Block = 64 tokens, 512 threads (one token per lane leaves a single wave per CU walking K-long
// dependent loops over strided global loads).  The block first stages its tokens' logits, summed over the
// K-split slices, with contiguous loads into LDS; lane l of a token then owns
// the logits k = l, l + 8, ... (softmax, g_a, g_z).  Bound by a chain of short phases with one block per compute unit; of
// 91 thousand cycles at n = 5, backward, 14 were the rows of H_res (matrix cores now), 32 vr read eight logits or tokens
// at a time with bank conflicts, divisions and a factor per element (vr stands in LDS now, rows an odd number of 16-byte
// pieces long).  Steps, us before / now: n = 5, C = 512, 16 tokens 112 / 98, 3000 tokens 179 / 164, C = 2560, 16384 tokens 1255 /
// 1239; n = 8, K = 64, C = 1024, 16384 tokens 805 / 799; forward n = 5, C = 512, 4000 tokens 52.8 / 48.7.
//   kGroupForward: H_res, H_pre, H_post
//   kGroupFast   : for the bf16 backward, in the layouts its MFMAs read:
//     cpk  [T][CP] f32 : H_res (N*N) | H_pre (N) | H_post (N) | coefx
//     vr   [Tpad][MP32] bf16 hi, lo : vr = r alpha g_z, row per token
//     vrT  [Tpad/32][MP16][32] bf16 hi, lo : the same, tokens innermost
//     gzs  [Tpad/64][M+3] f32 : per 64 tokens, the sums of g_z and of the per-group g_z u
//          (what g_b and g_alpha are summed from), added pairwise
//     Tokens T..Tpad-1 get zero vr so that padded tiles add nothing to g_W.
//     F16ROWS (the single-kernel wide pass 2): the vr ROWS hold fp16 hi, lo parts of vr / s with
//     s = max_m |vr_m| of the token (1 if that is 0), so that any gradient scale fits fp16; s
//     goes to cpk[N*N + 2N + 1].  vrT stays bf16 in either case.
//   kGroupFull   : for the full-precision backward: cpk, gzs and vr as fp32 rows [T][MP16]
// The table comes from device memory (`sigma`) or, if `use_tab`, by value.
struct TableArg {
  int8_t s[kMaxPerm * kMaxNSubset];
};
constexpr int kGTok = 64, kGThreads = 512;
enum { kGroupForward, kGroupFast, kGroupFull };

__device__ __forceinline__ float group_sum(float v) {
  v = lane_add(v, __shfl_xor(v, 1, 64));
  v = lane_add(v, __shfl_xor(v, 2, 64));
  v = lane_add(v, __shfl_xor(v, 4, 64));
  return v;
}
__device__ __forceinline__ float group_max(float v) {
  v = fmaxf(v, __shfl_xor(v, 1, 64));
  v = fmaxf(v, __shfl_xor(v, 2, 64));
  v = fmaxf(v, __shfl_xor(v, 4, 64));
  return v;
}

// row length of the LDS arrays of M logits: whole 16-byte pieces, an odd number of them
__host__ __device__ constexpr int group_ld(int M) { return 4 * (((M + 3) / 4) | 1); }

// dynamic LDS the kernel needs, eight table bytes per permutation among it
inline size_t group_lds_bytes(int N, int K, bool bwd) {
  size_t fl = 2 * static_cast<size_t>(kGTok) * group_ld(K + 2 * N) + kGTok;
  if (bwd) fl += static_cast<size_t>(kGTok) * (N * N + 1) + 4 * kGTok;
  return fl * sizeof(float) + static_cast<size_t>(K) * 8;
}

// dst[tok][0..W) = the sums over the slices of src [slices][T][W] for the block's 64 tokens (past the
// last one: some valid element again), slices in order.  Nine elements per thread and three more
// slices of each are on their way together: with one slice of four elements at a time the
// block, alone on its CU, spent 20 us in round trips at n = 5.
template <typename F>
__device__ __forceinline__ void stage_run(const F *__restrict__ src, int slices, int64_t T,
                                          int64_t t0, int W, float *dst, int ld) {
  constexpr int E = 9, S = sizeof(F) == 4 ? 3 : 1;
  const unsigned per = 0xffffffffu / static_cast<unsigned>(W) + 1;   // e / W is the high word of e per
  const int64_t stride = T * W, base = t0 * W;
  for (int e0 = threadIdx.x; e0 < kGTok * W; e0 += E * kGThreads) {
    F s[E];
    int64_t at[E];
#pragma unroll
    for (int v = 0; v < E; ++v) {
      const int e = e0 + v * kGThreads;
      at[v] = base + (e < kGTok * W ? e : kGTok * W - 1);
      if (at[v] > stride - 1) at[v] = stride - 1;
      s[v] = src[at[v]];
    }
    for (int p0 = 1; p0 < slices; p0 += S) {
      F w[S][E];
#pragma unroll
      for (int k = 0; k < S; ++k) {
        const F *slice = src + (p0 + k < slices ? p0 + k : slices - 1) * stride;
#pragma unroll
        for (int v = 0; v < E; ++v) w[k][v] = slice[at[v]];
      }
#pragma unroll
      for (int k = 0; k < S; ++k)
#pragma unroll
        for (int v = 0; v < E; ++v)
          if (p0 + k < slices) s[v] += w[k][v];
    }
#pragma unroll
    for (int v = 0; v < E; ++v) {
      const int e = e0 + v * kGThreads;
      const int row = W == 1 ? e : static_cast<int>(__umulhi(static_cast<unsigned>(e), per));
      if (e < kGTok * W) dst[row * ld + e - row * W] = static_cast<float>(s[v]);
    }
  }
}

// OWN: residual logits per lane, 8 OWN >= K
template <int N, int OUT, bool F16ROWS, int OWN>
__device__ __forceinline__ void coeffs_group(
    const float *__restrict__ u_raw, const float *__restrict__ sumsq, int parts, int wide,
    const float *__restrict__ b, const float *__restrict__ alpha,
    const float *__restrict__ gH_res, const float *__restrict__ gH_pre,
    const float *__restrict__ gH_post, int gparts, int nC, float eps, int64_t T, int K,
    const int8_t *__restrict__ sigma, const TableArg &tab, int use_tab,
    float *__restrict__ H_res, float *__restrict__ H_pre, float *__restrict__ H_post, int CP,
    int MP32, int MP16, float *__restrict__ cpk, uint16_t *__restrict__ vr_hi,
    uint16_t *__restrict__ vr_lo, uint16_t *__restrict__ vrT_hi, uint16_t *__restrict__ vrT_lo,
    float *__restrict__ vr32, float *__restrict__ gz_sums) {
  constexpr bool BWD = OUT != kGroupForward;
  extern __shared__ __align__(16) float smem[];
  const int M = K + 2 * N, ld = group_ld(M);
  constexpr int NN = N * N, gld = NN + 1;
  float *u_s = smem;                              // [64][ld]  raw logits, later vr
  float *a_s = u_s + kGTok * ld;                  // [64][ld]  softmax weights, later g_z
  float *g_s = a_s + kGTok * ld;                  // [64][gld] g_H_res            (BWD)
  float *r_s = g_s + (BWD ? kGTok * gld : 0);     // [64]      RMSNorm scale
  float *t_s = r_s + kGTok;                       // [64][4]   sums of g_z u per group, row scale (BWD)
  int8_t *sig = reinterpret_cast<int8_t *>(t_s + (BWD ? 4 * kGTok : 0));   // [K][8], N of them used
  const int tid = threadIdx.x;
  const int64_t t0 = static_cast<int64_t>(blockIdx.x) * kGTok;

  // stage: table (entries clamped to 0..N-1), logits, scale, g_H_res
  for (int i = tid; i < K * 8; i += kGThreads) {
    const int at = (i >> 3) * N + ((i & 7) < N ? i & 7 : 0);
    int v = use_tab ? tab.s[at] : sigma[at];
    v = v < 0 ? 0 : (v > N - 1 ? N - 1 : v);
    sig[i] = static_cast<int8_t>(v);
  }
  const int tok = tid >> 3, l = tid & 7;
  // Every lane takes OWN logits; past the last one it repeats that (same loads on every path, all
  // requested together: under a condition each was a round trip of its own) and drops the result.
  auto kc = [&](int kk) { return l + 8 * kk < K ? l + 8 * kk : K - 1; };
  auto owns = [&](int kk) { return l + 8 * kk < K; };
  float bk[OWN];
#pragma unroll
  for (int kk = 0; kk < OWN; ++kk) bk[kk] = b[kc(kk)];
  if (wide)
    stage_run(reinterpret_cast<const double *>(u_raw), parts, T, t0, M, u_s, ld);
  else
    stage_run(u_raw, parts, T, t0, M, u_s, ld);
  if (tid < kGTok) {
    int64_t tt = t0 + tid;
    if (tt > T - 1) tt = T - 1;
    const float ssq = slice_sum(sumsq, parts, wide, T, tt);
    r_s[tid] = rms_factor(ssq, nC, eps);
  }
  if constexpr (BWD) stage_run(gH_res, gparts, T, t0, NN, g_s, gld);
  __syncthreads();

  const int64_t t = t0 + tok;
  const bool live = t < T;
  const int64_t tl = live ? t : T - 1;
  const float r = r_s[tok];
  const float a0 = alpha[0], a1 = alpha[1], a2 = alpha[2];
  float *ut = u_s + tok * ld;
  float *at = a_s + tok * ld;

  // softmax over the K residual logits; own[] = this lane's weights
  float own[OWN];
  float zmax = -INFINITY;
#pragma unroll
  for (int kk = 0; kk < OWN; ++kk) {
    const float z = logit_of(a0, r, ut[kc(kk)], bk[kk]);
    own[kk] = owns(kk) ? z : -INFINITY;
    zmax = fmaxf(zmax, own[kk]);
  }
  zmax = group_max(zmax);
  float sum = 0.f;
#pragma unroll
  for (int kk = 0; kk < OWN; ++kk) {
    own[kk] = owns(kk) ? expf(own[kk] - zmax) : 0.f;
    sum += own[kk];
  }
  sum = group_sum(sum);
#pragma unroll
  for (int kk = 0; kk < OWN; ++kk) {
    own[kk] = own[kk] / sum;
    if (owns(kk)) at[l + 8 * kk] = own[kk];
  }
  __syncthreads();

  // H_res = sum_k a_k P_k: the weights of 16 tokens times the 0/1 matrix of the table, in fp32 on the matrix cores (a
  // lane per row that walked the K permutations took 14 thousand cycles of 90 at n = 5)
  {
    constexpr int CT = (NN + 15) / 16;   // tiles of 16 entries
    const int lane = tid & 63, rr = lane & 15, q = lane >> 4;
    for (int tile = tid >> 6; tile < kGTok / 16 * CT; tile += kGThreads / 64) {
      const int tk0 = 16 * (tile / CT), cell = 16 * (tile % CT) + rr;
      const int ci = cell < NN ? cell / N : 0, cj = cell < NN ? cell % N : -1;
      const float *aw = a_s + (tk0 + rr) * ld;
      f32x4 h = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 4
      for (int k0 = 0; k0 < K; k0 += 4) {
        const int k = k0 + q < K ? k0 + q : K - 1;
        const float w = k0 + q < K ? aw[k] : 0.f;
        h = mfma_f32(w, sig[k * 8 + ci] == cj ? 1.f : 0.f, h);
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int64_t tt = t0 + tk0 + 4 * q + i;
        if (tt < T && cell < NN) (BWD ? cpk + tt * CP : H_res + tt * NN)[cell] = h[i];
      }
    }
  }

  if constexpr (!BWD) {
    if (l < N && live) {
      H_pre[t * N + l] = sigmoidf(logit_of(a1, r, ut[K + l], b[K + l]));
      H_post[t * N + l] = 2.f * sigmoidf(logit_of(a2, r, ut[K + N + l], b[K + N + l]));
    }
    return;
  } else {
    // g_a[k] = sum_i g_H_res[i][sigma_k(i)], g_z = a (g_a - <a, g_a>)
    const float *gt = g_s + tok * gld;
    float gown[OWN];
    float meanp = 0.f;
#pragma unroll
    for (int kk = 0; kk < OWN; ++kk) {
      const u32x2 row = *reinterpret_cast<const u32x2 *>(sig + kc(kk) * 8);
      float sg = 0.f;
#pragma unroll
      for (int i = 0; i < N; ++i) sg += gt[i * N + ((row[i >> 2] >> (8 * (i & 3))) & 0xffu)];
      gown[kk] = sg;
      meanp += owns(kk) ? own[kk] * sg : 0.f;
    }
    const float mean = group_sum(meanp);
    __syncthreads();   // the weights in a_s are no longer needed: it now takes g_z
    float dotp = 0.f, gap[3] = {0.f, 0.f, 0.f}, vmaxp = 0.f;
#pragma unroll
    for (int kk = 0; kk < OWN; ++kk) {
      const bool ok = live && owns(kk);
      const float g = ok ? own[kk] * (gown[kk] - mean) : 0.f;
      const float uk = ut[kc(kk)];
      const float v = ok ? r * a0 * g : 0.f;
      if (owns(kk)) {   // (a lane that has no logit kk re-reads the last one's place, and drops it)
        at[l + 8 * kk] = g;
        ut[l + 8 * kk] = v;
      }
      gap[0] += ok ? g * (r * uk) : 0.f;   // (selected: uk may be infinite where there is no logit or token)
      dotp += ok ? v * uk : 0.f;
      vmaxp = fmaxf(vmaxp, fabsf(v));
    }
    if (l < N) {
      const float up = ut[K + l], uq = ut[K + N + l];
      const float hp = sigmoidf(logit_of(a1, r, up, b[K + l]));
      const float hq = 2.f * sigmoidf(logit_of(a2, r, uq, b[K + N + l]));
      float dp = gH_pre[tl * N + l], dq = gH_post[tl * N + l];
#pragma unroll 4
      for (int pt = 1; pt < gparts; ++pt) {
        dp += gH_pre[(pt * T + tl) * N + l];
        dq += gH_post[(pt * T + tl) * N + l];
      }
      float gp = dp * hp * (1.f - hp);
      float gq = dq * hq * (1.f - 0.5f * hq);
      if (live) {
        cpk[t * CP + NN + l] = hp;
        cpk[t * CP + NN + N + l] = hq;
      } else {
        gp = 0.f;
        gq = 0.f;
      }
      at[K + l] = gp;
      at[K + N + l] = gq;
      const float vp = live ? r * a1 * gp : 0.f, vq = live ? r * a2 * gq : 0.f;
      ut[K + l] = vp;
      ut[K + N + l] = vq;
      gap[1] = live ? gp * (r * up) : 0.f;
      gap[2] = live ? gq * (r * uq) : 0.f;
      dotp += live ? vp * up + vq * uq : 0.f;
      vmaxp = fmaxf(vmaxp, fmaxf(fabsf(vp), fabsf(vq)));
    }
    const float dot = group_sum(dotp);
    const float vmax = group_max(vmaxp);
#pragma unroll
    for (int g = 0; g < 3; ++g) gap[g] = group_sum(gap[g]);
    if (l == 0) {
      const float sc = (F16ROWS && vmax > 0.f) ? vmax : 1.f;
      t_s[tok * 4 + 0] = gap[0];
      t_s[tok * 4 + 1] = gap[1];
      t_s[tok * 4 + 2] = gap[2];
      t_s[tok * 4 + 3] = 1.f / sc;
      if (live) {
        cpk[t * CP + NN + 2 * N] = (r * r / static_cast<float>(nC)) * dot;
        if constexpr (F16ROWS) cpk[t * CP + NN + 2 * N + 1] = sc;
      }
    }
    __syncthreads();

    // vr = r alpha_g g_z, zero past the last logit
    if constexpr (OUT == kGroupFull) {
      if (live)
        for (int m = l; m < MP16; m += 8) vr32[t * MP16 + m] = m < M ? ut[m] : 0.f;
    } else {
    // rows [Tpad][MP32]: eight consecutive logits at a time, by the token's lanes
    const float inv = F16ROWS ? t_s[tok * 4 + 3] : 1.f;
    for (int v8 = l; v8 < MP32 / 8; v8 += 8) {
      const f32x4 lo4 = *reinterpret_cast<const f32x4 *>(ut + 8 * v8);   // (past the row: another one's, not used)
      const f32x4 hi4 = *reinterpret_cast<const f32x4 *>(ut + 8 * v8 + 4);
      float v[8];
      u32x4 hi, lo;
#pragma unroll
      for (int i = 0; i < 8; ++i) v[i] = 8 * v8 + i < M ? (i < 4 ? lo4[i] : hi4[i - 4]) * inv : 0.f;
      split8(v, std::bool_constant<F16ROWS>{}, hi, lo);
      const size_t off = static_cast<size_t>(t) * MP32 + 8 * v8;
      *reinterpret_cast<u32x4 *>(vr_hi + off) = hi;
      *reinterpret_cast<u32x4 *>(vr_lo + off) = lo;
    }
    // tokens innermost [Tpad/32][MP16][32]: eight consecutive tokens of one logit per thread
    const int64_t blk0 = t0 >> 5;
    for (int e = tid; e < 8 * MP16; e += kGThreads) {
      const int m = e >> 3, half = (e >> 2) & 1, tg = e & 3;
      const float *src = u_s + (half * 32 + tg * 8) * ld + (m < M ? m : M - 1);
      float v[8];
      u32x4 hi, lo;
#pragma unroll
      for (int i = 0; i < 8; ++i) v[i] = m < M ? src[i * ld] : 0.f;
      split8(v, std::false_type{}, hi, lo);
      const size_t off = (static_cast<size_t>(blk0 + half) * MP16 + m) * 32 + tg * 8;
      *reinterpret_cast<u32x4 *>(vrT_hi + off) = hi;
      *reinterpret_cast<u32x4 *>(vrT_lo + off) = lo;
    }
    }
    // sums over the block's 64 tokens, pairwise: four lanes per column, 16 tokens each (one lane
    // for all 64 keeps too many loads in flight: 8 us more of 1288 for the n = 5 step)
    for (int e = tid; e < 4 * (M + 3); e += kGThreads) {
      const int m = e >> 2, tk0 = 16 * (e & 3);
      const float *src = m < M ? a_s + tk0 * ld + m : t_s + tk0 * 4 + (m - M);
      const int step = m < M ? ld : 4;
      float s = pairwise_sum<16>([&](int tk) { return src[tk * step]; });
      s += __shfl_xor(s, 1, 64);
      s += __shfl_xor(s, 2, 64);
      if ((e & 3) == 0) gz_sums[static_cast<int64_t>(blockIdx.x) * (M + 3) + m] = s;
    }
  }
}

template <int N, int OUT, bool F16ROWS, int OWN>
__global__ __launch_bounds__(kGThreads) void coeffs_group_kernel(
    const float *__restrict__ u_raw, const float *__restrict__ sumsq, int parts, int wide,
    const float *__restrict__ b, const float *__restrict__ alpha,
    const float *__restrict__ gH_res, const float *__restrict__ gH_pre,
    const float *__restrict__ gH_post, int gparts, int nC, float eps, int64_t T, int K,
    const int8_t *__restrict__ sigma, const TableArg tab, int use_tab,
    float *__restrict__ H_res, float *__restrict__ H_pre, float *__restrict__ H_post, int CP,
    int MP32, int MP16, float *__restrict__ cpk, uint16_t *__restrict__ vr_hi,
    uint16_t *__restrict__ vr_lo, uint16_t *__restrict__ vrT_hi, uint16_t *__restrict__ vrT_lo,
    float *__restrict__ vr32, float *__restrict__ gz_sums) {
  coeffs_group<N, OUT, F16ROWS, OWN>(
      u_raw, sumsq, parts, wide, b, alpha, gH_res, gH_pre, gH_post, gparts, nC, eps, T, K, sigma, tab, use_tab, H_res, H_pre, H_post, CP, MP32, MP16, cpk, vr_hi, vr_lo, vrT_hi, vrT_lo, vr32, gz_sums);
}
// the forward's coefficients, and from block p.first on the pre-aggregate
template <int N, int OWN, typename IO>
__global__ __launch_bounds__(kGThreads) void coeffs_group_pre_kernel(
    const float *__restrict__ u_raw, const float *__restrict__ sumsq, int parts, int wide,
    const float *__restrict__ b, const float *__restrict__ alpha, float eps, int64_t T, int K,
    const int8_t *__restrict__ sigma, const TableArg tab, int use_tab, float *__restrict__ H_res,
    float *__restrict__ H_pre, float *__restrict__ H_post, PreArgs p) {
  if (blockIdx.x < p.first)
    coeffs_group<N, kGroupForward, false, OWN>(u_raw, sumsq, parts, wide, b, alpha, nullptr, nullptr, nullptr, 1,
                                               N * p.C, eps, T, K, sigma, tab, use_tab, H_res, H_pre, H_post, 0, 0,
                                               0, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr);
  else
    pre_from_slices<IO, N, kGThreads>(p, blockIdx.x - p.first, u_raw, sumsq, parts, wide, b, alpha, eps, T, K);
}

// table of the launch: the caller's subset, or all 120 permutations of n = 5 in
// lexicographic order (full form), passed by value
struct GroupTable {
  int K = 0, use_tab = 0;
  const int8_t *sigma = nullptr;
  TableArg tab{};
};
bool group_table(const mhcl_desc &d, GroupTable &g) {
  if (d.res_mode == MHCL_RES_SUBSET) {
    if (d.n_perm < 1 || d.n_perm > kMaxPerm || !d.perm) return false;
    g.K = d.n_perm;
    g.sigma = d.perm;
    return true;
  }
  if (d.res_mode == MHCL_RES_LITE && d.n == 5) {
    g.K = factorial(5);
    g.use_tab = 1;
    for (int k = 0; k < g.K; ++k)
      for (int i = 0; i < 5; ++i) g.tab.s[k * 5 + i] = Perm<5>::tab.s[k][i];
    return true;
  }
  return false;
}

// lds: this call's need, most: the kernel's (the limit is the kernel's, also for other threads' calls)
template <typename Kern>
hipError_t allow_lds(Kern kern, size_t lds, size_t most) {
  if (lds <= 64 * 1024) return hipSuccess;
  return hipFuncSetAttribute(reinterpret_cast<const void *>(kern),
                             hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(most));
}

// Slices that are added by a launch of their own: a block here takes 64 tokens and would read 16 slices of
// 64 x 130 fp64 logits through its one compute unit.  mhcl_coeffs, f32, inside / before (n = 5, C = 1024: 16 parts at
// 16 tokens 42.5 / 30.3 us, 512 tokens 63.3 / 52.0; two parts, C = 256, 4096 tokens 52.7 / 55.6).
bool add_first(const RawSums &raw) { return raw.wide && raw.parts > 2; }

}  // namespace

bool coeffs_group_ok(const mhcl_desc &d) {
  return d.res_mode == MHCL_RES_SUBSET || (d.res_mode == MHCL_RES_LITE && d.n == 5);
}

hipError_t launch_coeffs_group(const mhcl_desc &d, const RawSums &raw, const float *b,
                               const float *alpha, float *H_res, float *H_pre, float *H_post,
                               hipStream_t s) {
  GroupTable g;
  if (!group_table(d, g)) return hipErrorInvalidValue;
  RawSums r = raw;
  if (add_first(r)) {
    hipError_t e = add_wide_slices(d, r, s);
    if (e != hipSuccess) return e;
  }
  return dispatch_n(d.n, [&](auto nn) {
    constexpr int N = decltype(nn)::value;
    auto kern = g.K <= 64 ? coeffs_group_kernel<N, kGroupForward, false, 8>
                          : coeffs_group_kernel<N, kGroupForward, false, 16>;
    const size_t lds = group_lds_bytes(N, g.K, false);
    hipError_t e = allow_lds(kern, lds, group_lds_bytes(N, kMaxPerm, false));
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kern, dim3(static_cast<unsigned>((d.T + kGTok - 1) / kGTok)),
                       dim3(kGThreads), lds, s, r.u_raw, r.sumsq, r.parts, r.wide, b, alpha, nullptr, nullptr,
                       nullptr, 1, d.n * d.C, d.eps, d.T, g.K, g.sigma, g.tab, g.use_tab, H_res, H_pre,
                       H_post, 0, 0, 0, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr);
    return hipGetLastError();
  });
}

// Up to 64 permutations (eight residual logits per lane) the kernel has 110 registers and at most 64 KB of LDS, so two of its
// blocks stream on a compute unit; with more it has 133, and one does, which is too few for many tokens.  Two launches /
// one, us for mhcl_fwd_coeffs_pre.  n = 8, K = 64, C = 1024, 4000 tokens 51.8 / 46.1, 16384 (2.1 million 16-byte chunks of h) 121 / 116,
// 32768 261 / 254, 65536 498 / 490; n = 6, K = 40, 65536 tokens 394 / 381; n = 5, K = 30, 32768 tokens 146.9 / 147.7, 65536 315 /
// 312.  n = 8, K = 66, C = 1024, 4000 tokens 53.4 / 46.9, 8000 (1 million) 76.5 / 73.4, 16384 125 / 137, C = 256, 16384 tokens 50.6 /
// 58.6; n = 6, K = 128, C = 1024, 16384 tokens 115 / 125; n = 5, full form, C = 2560, 1500 tokens (480 thousand) 67.8 / 61.7, C = 1024, 6000 tokens
// 68.4 / 67.7, C = 320, 8000 tokens 44.3 / 40.9, 12000 tokens 52.7 / 53.1.
bool group_coeffs_pre_ok(const mhcl_desc &d) {
  if (!coeffs_group_ok(d)) return false;
  return res_logits(d) <= 64 ? pre_chunks(d) <= (1 << 23) : pre_chunks(d) <= (1 << 19) && d.T <= 128 * kGTok;
}
hipError_t launch_coeffs_pre_group(const mhcl_desc &d, const RawSums &raw, const float *b, const float *alpha,
                                   const void *x, float *H_res, float *H_pre, float *H_post, void *h,
                                   hipStream_t s) {
  GroupTable g;
  if (!group_table(d, g)) return hipErrorInvalidValue;
  const PreArgs p{x, h, static_cast<unsigned>((d.T + kGTok - 1) / kGTok), d.C};
  RawSums r = raw;
  if (add_first(r)) {
    hipError_t e = add_wide_slices(d, r, s);
    if (e != hipSuccess) return e;
  }
  return dispatch_io(d.io_dtype, [&](auto io) {
    return dispatch_n(d.n, [&](auto nn) {
      constexpr int N = decltype(nn)::value;
      using IO = decltype(io);
      auto kern = g.K <= 64 ? coeffs_group_pre_kernel<N, 8, IO> : coeffs_group_pre_kernel<N, 16, IO>;
      const size_t lds = group_lds_bytes(N, g.K, false);
      // (with the static arrays it may pass 64 KiB before it does by itself)
      hipError_t e = allow_lds(kern, lds + sizeof(float) * (kGThreads + 1) * N + sizeof(double) * kGThreads,
                                group_lds_bytes(N, kMaxPerm, false));
      if (e != hipSuccess) return e;
      hipLaunchKernelGGL(kern, dim3(p.first + pre_blocks(d, kGThreads)), dim3(kGThreads), lds, s, r.u_raw, r.sumsq,
                         r.parts, r.wide, b, alpha, d.eps, d.T, g.K, g.sigma, g.tab, g.use_tab, H_res, H_pre, H_post, p);
      return hipGetLastError();
    });
  });
}

hipError_t launch_coeffs_bwd_group(const mhcl_desc &d, const RawSums &raw, const float *b,
                                   const float *alpha, const float *g_H_res, const float *g_H_pre,
                                   const float *g_H_post, const BwdTokenBufs &o, hipStream_t s) {
  GroupTable g;
  if (!group_table(d, g)) return hipErrorInvalidValue;
  RawSums r = raw;
  if (add_first(r)) {
    hipError_t e = add_wide_slices(d, r, s);
    if (e != hipSuccess) return e;
  }
  const int M = g.K + 2 * d.n;
  return dispatch_n(d.n, [&](auto nn) {
    constexpr int N = decltype(nn)::value;
    auto kern = g.K <= 64 ? coeffs_group_kernel<N, kGroupFull, false, 8>
                          : coeffs_group_kernel<N, kGroupFull, false, 16>;
    const size_t lds = group_lds_bytes(N, g.K, true);
    hipError_t e = allow_lds(kern, lds, group_lds_bytes(N, kMaxPerm, true));
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kern, dim3(static_cast<unsigned>((d.T + kGTok - 1) / kGTok)),
                       dim3(kGThreads), lds, s, r.u_raw, r.sumsq, r.parts, r.wide, b, alpha, g_H_res, g_H_pre,
                       g_H_post, 1, d.n * d.C, d.eps, d.T, g.K, g.sigma, g.tab, g.use_tab, nullptr, nullptr,
                       nullptr, token_rec<N>(), 0, (M + 15) / 16 * 16, o.rec, nullptr, nullptr, nullptr,
                       nullptr, o.vr, o.gz);
    return hipGetLastError();
  });
}

hipError_t launch_bwd_epilogue_group(const mhcl_desc &d, const float *b, const float *alpha,
                                     const FastBwdWs &w, hipStream_t s) {
  GroupTable g;
  if (!group_table(d, g)) return hipErrorInvalidValue;
  const int64_t Tpad = (d.T + 63) / 64 * 64;
  const int M = g.K + 2 * d.n;
  if (w.MP32 != (M + 31) / 32 * 32 || w.MP16 != (M + 15) / 16 * 16) return hipErrorInvalidValue;
  const bool f16 = fast_bwd_whi(d);   // rows for bwd_out_w16_kernel
  if (f16 && w.CP < d.n * d.n + 2 * d.n + 2) return hipErrorInvalidValue;
  RawSums r = w.raw();
  if (add_first(r)) {
    hipError_t e = add_wide_slices(d, r, s);
    if (e != hipSuccess) return e;
  }
  return dispatch_n(d.n, [&](auto nn) {
    constexpr int N = decltype(nn)::value;
    auto launch = [&](auto kern) {
      const size_t lds = group_lds_bytes(N, g.K, true);
      hipError_t e = allow_lds(kern, lds, group_lds_bytes(N, kMaxPerm, true));
      if (e != hipSuccess) return e;
      hipLaunchKernelGGL(kern, dim3(static_cast<unsigned>(Tpad / kGTok)), dim3(kGThreads), lds, s,
                         r.u_raw, r.sumsq, r.parts, r.wide, b, alpha, w.gH_res, w.gH_pre, w.gH_post,
                         w.gparts, d.n * d.C, d.eps, d.T, g.K, g.sigma, g.tab, g.use_tab, nullptr, nullptr,
                         nullptr, w.CP, w.MP32, w.MP16, w.cpk, w.vr_hi, w.vr_lo, w.vrT_hi, w.vrT_lo,
                         nullptr, w.gz);
      return hipGetLastError();
    };
    if constexpr (N >= 5) {
      if (f16)
        return launch(g.K <= 64 ? coeffs_group_kernel<N, kGroupFast, true, 8>
                                : coeffs_group_kernel<N, kGroupFast, true, 16>);
    }
    return launch(g.K <= 64 ? coeffs_group_kernel<N, kGroupFast, false, 8>
                            : coeffs_group_kernel<N, kGroupFast, false, 16>);
  });
}

}  // namespace mhcl
