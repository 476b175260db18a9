// Thin products at full precision on the matrix cores: f32 streams, bf16 streams whose C is no
// multiple of 64, the separable entry points, and the projection of few tokens.  Operands enter as
// they are (x widened, W and the per-token vectors in fp32); the projection sums in fp64
// (v_mfma_f64_16x16x4_f64), the others in fp32 (v_mfma_f32_16x16x4_f32), so nothing is split or
// rounded on the way.
#include "mhcl_common.h"
#include "mhcl_internal.h"
#include "mhcl_mfma.h"

namespace mhcl {

namespace {

// logit tiles of 16: 1 ... 9
template <typename F>
hipError_t dispatch_tiles(int NT, F &&f) {
  switch (NT) {
    case 1: return f(std::integral_constant<int, 1>{});
    case 2: return f(std::integral_constant<int, 2>{});
    case 3: return f(std::integral_constant<int, 3>{});
    case 4: return f(std::integral_constant<int, 4>{});
    case 5: return f(std::integral_constant<int, 5>{});
    case 6: return f(std::integral_constant<int, 6>{});
    case 7: return f(std::integral_constant<int, 7>{});
    case 8: return f(std::integral_constant<int, 8>{});
    case 9: return f(std::integral_constant<int, 9>{});
  }
  return hipErrorInvalidValue;
}

// V consecutive stream elements, as they lie in memory and widened
template <typename IO, int V>
struct Piece;
template <>
struct Piece<BF16, 8> {
  u32x4 w;
  __device__ __forceinline__ void load(const void *p, size_t elem) {
    w = *reinterpret_cast<const u32x4 *>(static_cast<const uint16_t *>(p) + elem);
  }
  __device__ __forceinline__ float at(int e) const { return (e & 1) ? bf16hi(w[e >> 1]) : bf16lo(w[e >> 1]); }
  __device__ __forceinline__ void clear() { w = u32x4{0, 0, 0, 0}; }
};
template <>
struct Piece<BF16, 4> {
  u32x2 w;
  __device__ __forceinline__ void load(const void *p, size_t elem) {
    w = *reinterpret_cast<const u32x2 *>(static_cast<const uint16_t *>(p) + elem);
  }
  __device__ __forceinline__ float at(int e) const { return (e & 1) ? bf16hi(w[e >> 1]) : bf16lo(w[e >> 1]); }
  __device__ __forceinline__ void clear() { w = u32x2{0, 0}; }
};
template <>
struct Piece<F32, 4> {
  f32x4 w;
  __device__ __forceinline__ void load(const void *p, size_t elem) {
    w = *reinterpret_cast<const f32x4 *>(static_cast<const float *>(p) + elem);
  }
  __device__ __forceinline__ float at(int e) const { return w[e]; }
  __device__ __forceinline__ void clear() { w = f32x4{0.f, 0.f, 0.f, 0.f}; }
};

// ---------------------------------------------------------------------------
// u_raw[t][m] = sum_k x_hat[t][k] W[k][m] and sumsq[t] = sum_k x_hat[t][k]^2 (the two reductions
// over nC behind RMSNorm and the linear maps of Sec. 3.2), with exact products and fp64 sums
// (v_mfma_f64_16x16x4_f64): f32 streams keep their logits to fp32 rounding at any width.
// A block takes 16 tokens, its eight waves every eighth step of 4 V columns of the block's part of
// the row (gridDim.y parts; the consumer adds the parts' slices in order).  Lane (r, q) reads V
// consecutive columns of token r; element e is the left operand of the MFMAs whose contraction
// index q stands for column k0 + V q + e, the right operand comes straight from W (fp32, as
// it is; all blocks read the same rows, so these are L2 hits).
// Bound by the fp64 matrix rate (67 TFLOP/s: 12 us for f32 n = 4, C = 768, 4096 tokens; it takes
// 23; one thread per logit and eighth of the row, fp64 on the vector units, took 145).
constexpr int kProjWaves = 8;

// WAVES == 1: rows of one or two steps, whose other waves would only take part in the sums (n = 2, C = 8,
// K = 126, bf16, 131072 tokens: 261 us for mhcl_coeffs with eight waves, 97 with one).
// Block bx of `part`, of parts (fp64 slices if more than one).
template <typename IO, int NT, int WAVES>
__device__ __forceinline__ void proj_fullprec(
    const void *__restrict__ x, const float *__restrict__ W, int nC, int M, int64_t T,
    int steps_per_part, float *__restrict__ u_raw, float *__restrict__ sumsq, int bx, int part, int parts) {
  constexpr int V = IO::kVec;
  __shared__ double red[2][WAVES][4][64];
  __shared__ double red_ss[WAVES][16];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int r = lane & 15, q = lane >> 4;
  const int64_t t0 = static_cast<int64_t>(bx) * 16;
  const int64_t tl = t0 + r < T ? t0 + r : T - 1;
  const size_t row = static_cast<size_t>(tl) * nC;
  const int nsteps = (nC + 4 * V - 1) / (4 * V);
  const int s0 = part * steps_per_part;
  const int s1 = s0 + steps_per_part < nsteps ? s0 + steps_per_part : nsteps;
  int mj[NT];   // this lane's logit of tile j (past the last one: the last again, not stored)
#pragma unroll
  for (int j = 0; j < NT; ++j) mj[j] = 16 * j + r < M ? 16 * j + r : M - 1;

  f64x4 acc[NT];
  double ss = 0.0;
#pragma unroll
  for (int j = 0; j < NT; ++j) acc[j] = f64x4{0.0, 0.0, 0.0, 0.0};
  struct In {
    Piece<IO, V> x;
    float w[V][NT];
  };
  auto load = [&](In &in, int s) {
    const int k = s * 4 * V + V * q;
    const int kc = k < nC ? k : nC - V;   // (only the row's last step can reach past it)
    in.x.load(x, row + kc);
#pragma unroll
    for (int e = 0; e < V; ++e)
#pragma unroll
      for (int j = 0; j < NT; ++j) in.w[e][j] = W[static_cast<size_t>(kc + e) * M + mj[j]];
  };
  auto compute = [&](In &in, int s) {
    if (s * 4 * V + V * q >= nC) {
      in.x.clear();
#pragma unroll
      for (int e = 0; e < V; ++e)
#pragma unroll
        for (int j = 0; j < NT; ++j) in.w[e][j] = 0.f;
    }
#pragma unroll
    for (int e = 0; e < V; ++e) {
      const double xv = in.x.at(e);
      ss += xv * xv;
#pragma unroll
      for (int j = 0; j < NT; ++j) acc[j] = mfma_f64(xv, static_cast<double>(in.w[e][j]), acc[j]);
    }
  };
  {
    In a, b;
    int s = s0 + wave;
    load(a, s < s1 ? s : s1 - 1);
    for (; s + WAVES < s1; s += 2 * WAVES) {
      load(b, s + WAVES);
      __builtin_amdgcn_sched_barrier(0);
      compute(a, s);
      load(a, s + 2 * WAVES < s1 ? s + 2 * WAVES : s1 - 1);
      __builtin_amdgcn_sched_barrier(0);
      compute(b, s + WAVES);
    }
    if (s < s1) compute(a, s);
  }

  ss += __shfl_xor(ss, 16, 64);   // the four lanes of a token
  ss += __shfl_xor(ss, 32, 64);
  if constexpr (WAVES == 1) {   // (one part)
    if (q == 0 && t0 + r < T) sumsq[t0 + r] = static_cast<float>(ss);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int64_t t = t0 + 4 * i + q;   // (fp64 tiles hold rows 4 i + q)
#pragma unroll
      for (int j = 0; j < NT; ++j)
        if (t < T && 16 * j + r < M) u_raw[t * M + 16 * j + r] = static_cast<float>(acc[j][i]);
    }
    return;
  }
  // A row's one part is rounded to fp32 here; parts stay in fp64 and are rounded when they are added.
  // (Relative error of H_pre against 64 bits, f32, n = 4, C = 4096, 16 tokens: 5.7e-8 with fp32 slices, 4.0e-8.)
  auto put = [&](float *dst, int64_t at, double v) {
    if (parts > 1)
      reinterpret_cast<double *>(dst)[at] = v;
    else
      dst[at] = static_cast<float>(v);
  };
  if (q == 0) red_ss[wave][r] = ss;
  // the waves' sums, two logit tiles at a time, in wave order
#pragma unroll
  for (int base = 0; base < NT; base += 2) {
    __syncthreads();
#pragma unroll
    for (int j = 0; j < 2; ++j)
      if (base + j < NT) {
#pragma unroll
        for (int i = 0; i < 4; ++i) red[j][wave][i][lane] = acc[base + j][i];
      }
    __syncthreads();
    const int j = threadIdx.x >> 8, i = (threadIdx.x >> 6) & 3;
    if (base + j < NT) {
      double sum = red[j][0][i][lane];
#pragma unroll
      for (int w = 1; w < WAVES; ++w) sum += red[j][w][i][lane];
      // fp64 tiles hold rows 4 i + q: token 4 i + q, logit 16 (base + j) + r
      const int64_t t = t0 + 4 * i + q;
      const int m = 16 * (base + j) + r;
      if (t < T && m < M) put(u_raw, (part * T + t) * M + m, sum);
    }
  }
  if (threadIdx.x < 16 && t0 + threadIdx.x < T) {   // (red_ss was complete at the barriers above)
    double sum = red_ss[0][threadIdx.x];
#pragma unroll
    for (int w = 1; w < WAVES; ++w) sum += red_ss[w][threadIdx.x];
    put(sumsq, part * T + t0 + threadIdx.x, sum);
  }
}

template <typename IO, int NT, int WAVES>
__global__ __launch_bounds__(64 * WAVES, 1) void proj_fullprec_kernel(
    const void *__restrict__ x, const float *__restrict__ W, int nC, int M, int64_t T,
    int steps_per_part, float *__restrict__ u_raw, float *__restrict__ sumsq) {
  proj_fullprec<IO, NT, WAVES>(x, W, nC, M, T, steps_per_part, u_raw, sumsq, blockIdx.x, blockIdx.y, gridDim.y);
}

// gridDim.z layers of a stack side by side
template <typename IO, int NT>
__global__ __launch_bounds__(64 * kProjWaves, 1) void proj_fullprec_layers_kernel(
    JointLayers layers, int nC, int M, int64_t T, int steps_per_part, float *__restrict__ u_raw,
    float *__restrict__ sumsq) {
  const int l = blockIdx.z;
  proj_fullprec<IO, NT, kProjWaves>(layers.x[l], layers.W[l], nC, M, T, steps_per_part, u_raw + l * layers.stride,
                                    sumsq + l * layers.stride, blockIdx.x, blockIdx.y, gridDim.y);
}

// The n^2 + 2n reductions over C of the backward, as bwd_dots_kernel has them: `waves` waves per token, the block's
// eight take 8 / waves tokens.  They need nothing of the projection, so one launch has blocks of both: the
// products run at the fp64 rate and these at that of HBM, and x comes from the caches the second time.
struct DotsArgs {
  const void *y, *g_xout, *g_h;
  float *g_H_res, *g_H_post, *g_H_pre;
  int C, waves;
};
template <typename IO, int N>
__device__ __forceinline__ void dots_of_tokens(const DotsArgs &p, const void *__restrict__ x, int64_t T, int block) {
  constexpr int V = IO::kVec, D = N * N + 2 * N;
  __shared__ float red[kProjWaves][D];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, W = p.waves, C = p.C;
  const int per_block = kProjWaves / W, sub = wave / W;
  const int64_t t = static_cast<int64_t>(block) * per_block + sub;
  float dots[D];
#pragma unroll
  for (int e = 0; e < D; ++e) dots[e] = 0.f;
  if (sub < per_block && t < T) {
    for (int c = ((wave - sub * W) * 64 + lane) * V; c < C; c += 64 * W * V) {
      float xv[N][V], gv[N][V], yv[V], gh[V];
#pragma unroll
      for (int j = 0; j < N; ++j) {
        IO::load(x, (t * N + j) * C + c, xv[j]);
        IO::load(p.g_xout, (t * N + j) * C + c, gv[j]);
      }
      IO::load(p.y, t * C + c, yv);
      IO::load(p.g_h, t * C + c, gh);
#pragma unroll
      for (int i = 0; i < N; ++i) {
#pragma unroll
        for (int e = 0; e < V; ++e) {
          dots[N * N + i] += gv[i][e] * yv[e];
          dots[N * N + N + i] += gh[e] * xv[i][e];
        }
#pragma unroll
        for (int j = 0; j < N; ++j)
#pragma unroll
          for (int e = 0; e < V; ++e) dots[i * N + j] += gv[i][e] * xv[j][e];
      }
    }
#pragma unroll
    for (int e = 0; e < D; ++e) {
      const float s = wave_sum(dots[e]);
      if (lane == 0) red[wave][e] = s;
    }
  }
  __syncthreads();
  for (int i = threadIdx.x; i < per_block * D; i += 64 * kProjWaves) {
    const int k = i / D, e = i - k * D;
    const int64_t tt = static_cast<int64_t>(block) * per_block + k;
    if (tt >= T) continue;
    float s = red[k * W][e];
    for (int w = 1; w < W; ++w) s += red[k * W + w][e];
    if (e < N * N) p.g_H_res[tt * N * N + e] = s;
    else if (e < N * N + N) p.g_H_post[tt * N + e - N * N] = s;
    else p.g_H_pre[tt * N + e - N * N - N] = s;
  }
}

template <typename IO, int N, int NT>
__global__ __launch_bounds__(64 * kProjWaves, 1) void proj_dots_kernel(
    const void *__restrict__ x, const float *__restrict__ W, int nC, int M, int64_t T, int steps_per_part,
    float *__restrict__ u_raw, float *__restrict__ sumsq, int groups, int parts, DotsArgs p) {
  const int b = static_cast<int>(blockIdx.x);
  if (b < groups * parts)
    proj_fullprec<IO, NT, kProjWaves>(x, W, nC, M, T, steps_per_part, u_raw, sumsq, b % groups, b / groups, parts);
  else
    dots_of_tokens<IO, N>(p, x, T, b - groups * parts);
}

// Element e of [u_raw | sumsq] in fp64 slices: its sum over the slices, left in the first one.  For the stages
// whose blocks take 64 tokens or whose threads add serially (measured there).
template <int S>
__global__ __launch_bounds__(256) void add_slices_kernel(double *__restrict__ u_raw, double *__restrict__ sumsq,
                                                         int64_t n_u, int64_t T) {
  int64_t e = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
  if (e >= n_u + T) return;
  double *p = u_raw;
  int64_t stride = n_u;
  if (e >= n_u) { p = sumsq; stride = T; e -= n_u; }
  double v[S], s;
#pragma unroll
  for (int k = 0; k < S; ++k) v[k] = p[k * stride + e];
  s = v[0];
#pragma unroll
  for (int k = 1; k < S; ++k) s += v[k];
  p[e] = s;
}

// ---------------------------------------------------------------------------
// g_W[k][m] = sum_t x_hat[t][k] vr[t][m], the one reduction over tokens.
// A wave owns 16 V columns and takes four tokens per step: lane (r, q) reads V consecutive
// columns of token q, which are the left operands of V MFMAs (tile v: rows are columns
// k0 + V r + v), and the right operand is vr of the same four tokens, 16 logits at a time
// (L2 hits: all column blocks read the same rows).  The eight waves of a block share the
// columns and take every eighth group of four tokens; their sums meet in LDS, so a block
// leaves one partial result for its chunk of tokens.
// Bound by the fp32 matrix rate (152 TFLOP/s here) and HBM about equally at 32 logits.  It
// replaced a kernel of one (column, logit) pair per thread that walked the tokens serially:
// 572 -> 18.5 us for bf16 n = 4, C = 1024, 5003 tokens, 301 -> 14.8 us for f32 C = 768, 4096 tokens.
constexpr int kGwWaves = 8;

// columns per lane: 16-byte pieces, 8-byte ones where the accumulators of a 16-byte bf16
// piece (8 NT x 4 registers) no longer fit
template <typename IO, int NT>
constexpr int gw_piece() { return IO::kVec == 8 && NT <= 3 ? 8 : 4; }

constexpr int kGwLds = 8 * kGwWaves * 64 * sizeof(f32x4);
extern __shared__ f32x4 fullprec_lds[];   // of either role

template <typename IO, int NT, int V>
__device__ __forceinline__ void gw_fullprec(
    const void *__restrict__ x, const float *__restrict__ vr, int nC, int M, int64_t T,
    int64_t chunk, float *__restrict__ out, int bx, int by) {
  constexpr int U = NT <= 3 ? 4 : 2;   // groups per step (registers: 4 V NT are accumulators)
  constexpr int TILES = V * NT;
  f32x4(*red)[kGwWaves][64] = reinterpret_cast<f32x4(*)[kGwWaves][64]>(fullprec_lds);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int r = lane & 15, q = lane >> 4;
  const int k0 = bx * 16 * V;
  const int kr = k0 + V * r < nC ? k0 + V * r : nC - V;   // (lanes past the row re-read its end)
  const int64_t tb = static_cast<int64_t>(by) * chunk;
  const int64_t te = tb + chunk < T ? tb + chunk : T;
  f32x4 acc[V][NT];
#pragma unroll
  for (int v = 0; v < V; ++v)
#pragma unroll
    for (int j = 0; j < NT; ++j) acc[v][j] = f32x4{0.f, 0.f, 0.f, 0.f};

  struct In {
    Piece<IO, V> x[U];
    float b[U][NT];
  };
  auto load = [&](In &in, int64_t t0) {   // the wave's U groups of the block's step at t0
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int64_t t = t0 + (u * kGwWaves + wave) * 4 + q;
      const int64_t tl = t < te ? t : te - 1;
      in.x[u].load(x, static_cast<size_t>(tl) * nC + kr);
#pragma unroll
      for (int j = 0; j < NT; ++j) in.b[u][j] = vr[tl * (16 * NT) + 16 * j + r];
    }
  };
  auto compute = [&](In &in, int64_t t0) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (t0 + (u * kGwWaves + wave) * 4 + q >= te) {   // past the chunk: adds nothing
        in.x[u].clear();
#pragma unroll
        for (int j = 0; j < NT; ++j) in.b[u][j] = 0.f;
      }
#pragma unroll
      for (int v = 0; v < V; ++v)
#pragma unroll
        for (int j = 0; j < NT; ++j) acc[v][j] = mfma_f32(in.x[u].at(v), in.b[u][j], acc[v][j]);
    }
  };
  constexpr int kStep = 4 * U * kGwWaves;
  if (tb < te) {
    In a, b;
    load(a, tb);
    int64_t t0 = tb;
    for (; t0 + kStep < te; t0 += 2 * kStep) {
      load(b, t0 + kStep);
      __builtin_amdgcn_sched_barrier(0);
      compute(a, t0);
      load(a, t0 + 2 * kStep);   // (clamped to the chunk's last token when past its end)
      __builtin_amdgcn_sched_barrier(0);
      compute(b, t0 + kStep);
    }
    if (t0 < te) compute(a, t0);
  }

  // the waves' sums, eight tiles at a time: wave w adds tile w over the waves, in order
  float *dst = out + static_cast<size_t>(by) * nC * M;
#pragma unroll
  for (int base = 0; base < TILES; base += 8) {
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 8; ++i)
      if (base + i < TILES) red[i][wave][lane] = acc[(base + i) / NT][(base + i) % NT];
    __syncthreads();
    const int tile = base + wave;
    if (tile < TILES) {
      f32x4 s = red[wave][0][lane];
#pragma unroll
      for (int w = 1; w < kGwWaves; ++w) s += red[wave][w][lane];
      const int v = tile / NT, m = 16 * (tile % NT) + r;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int k = k0 + V * (4 * q + i) + v;
        if (k < nC && m < M) dst[static_cast<size_t>(k) * M + m] = s[i];
      }
    }
  }
}

template <typename IO, int NT, int V>
__global__ __launch_bounds__(64 * kGwWaves, 1) void gw_fullprec_kernel(
    const void *__restrict__ x, const float *__restrict__ vr, int nC, int M, int64_t T,
    int64_t chunk, float *__restrict__ out) {
  gw_fullprec<IO, NT, V>(x, vr, nC, M, T, chunk, out, blockIdx.x, blockIdx.y);
}

// ---------------------------------------------------------------------------
// Gradient on x.  With vr = r alpha g_z and coefx = (r^2/nC) <vr, u_raw>, the RMSNorm +
// projection part is  W vr - x_hat coefx.
//   FUSED: g_x = H_res^T g_xout + H_pre g_h + (that part), rounded once;
//          g_y = sum_i H_post[i] g_xout[i]
//   else : g_x += (that part)
// W vr is a product of W (left operand) and the vr of 16 tokens: a wave owns a window of 4 V
// columns of every stream, the rows of tile h are arranged so that lane (token, q) receives the V
// columns 4 q ... it reads and writes of the streams (row 4 q + i of tile h = column V q + 4 h + i).
// Four steps of the contraction are taken from one 16-byte read of W (LDS) and of vr: step i of
// group s covers the logits 16 s + 4 q + i.  The block's slice of W sits in LDS for its whole
// walk down the tokens; `win` of the eight waves take adjacent windows (so that a row visit covers
// win x 64 contiguous bytes), the others the next tokens.
// Bound by HBM (by itself, bf16, n = 4, C = 1024, 5003 tokens: 123 MB in 40 us; f32, C = 768, 4096 tokens,
// FUSED: 176 MB in 45 us; together with g_W: see gx_gw_kernel).  A block per token, every thread re-reading its rows of W from L2
// for each token, took 340 and 218 us.
constexpr int kGxWaves = 8;

struct GxArgs {
  const void *x;
  const float *W;
  const void *g_xout, *g_h;
  const float *rec, *vr;
  int M, S, C;
  int64_t T;
  int win, tokens_per_block;
  void *g_x, *g_y;
};

template <typename IO, int N, int SC, bool FUSED>   // SC: the groups of 16 logits, 0: as S says
__device__ __forceinline__ void gx_fullprec(
    const void *__restrict__ x, const float *__restrict__ W, const void *__restrict__ g_xout,
    const void *__restrict__ g_h, const float *__restrict__ rec, const float *__restrict__ vr, int M,
    int S, int C, int64_t T, int win, int tokens_per_block, void *__restrict__ g_x,
    void *__restrict__ g_y, int bx, int by) {
  constexpr int V = IO::kVec, TL = V / 4, CP = token_rec<N>();
  f32x4 *wl_all = fullprec_lds;   // [window][stream][tile][group of 16 logits][lane]
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int r = lane & 15, q = lane >> 4;
  const int per_win = N * TL * S * 64;
  for (int e = threadIdx.x; e < win * per_win; e += 64 * kGxWaves) {
    const int ln = e & 63, lr = ln & 15, lq = ln >> 4;
    int idx = e >> 6;
    const int s = idx % S; idx /= S;
    const int h = idx % TL; idx /= TL;
    const int j = idx % N, w = idx / N;
    const int col = (bx * win + w) * (4 * V) + V * (lr >> 2) + 4 * h + (lr & 3);
    const int m = 16 * s + 4 * lq;
    f32x4 v = f32x4{0.f, 0.f, 0.f, 0.f};
    if (col < C) {
      const float *row = W + (static_cast<size_t>(j) * C + col) * M;
      if (M % 4 == 0) {
        if (m < M) v = *reinterpret_cast<const f32x4 *>(row + m);
      } else {
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (m + i < M) v[i] = row[m + i];
      }
    }
    wl_all[e] = v;
  }
  __syncthreads();
  const int wi = wave % win, sub = wave / win, subs = kGxWaves / win;
  const f32x4 *wl = wl_all + wi * per_win + lane;
  const int c0 = (bx * win + wi) * (4 * V) + V * q;
  const bool col_ok = c0 < C;
  const int cl = col_ok ? c0 : C - V;
  const int64_t tb = static_cast<int64_t>(by) * tokens_per_block;
  const int64_t te = tb + tokens_per_block < T ? tb + tokens_per_block : T;
  // g: g_xout (FUSED) or the g_x so far
  struct In {
    Piece<IO, V> x[N], g[N], h;
    f32x4 rc[CP / 4], b[SC > 0 ? SC : 1];
  };
  auto load = [&](In &in, int64_t t0) {
    const int64_t tl = t0 + r < te ? t0 + r : te - 1;
    // (vr ahead of the streams: loads return in order, and W vr is done while these are on their way)
#pragma unroll
    for (int s = 0; s < SC; ++s) in.b[s] = *reinterpret_cast<const f32x4 *>(vr + tl * (16 * S) + 16 * s + 4 * q);
    if constexpr (SC > 0) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int j = 0; j < N; ++j) {
      in.x[j].load(x, (static_cast<size_t>(tl) * N + j) * C + cl);
      in.g[j].load(FUSED ? g_xout : g_x, (static_cast<size_t>(tl) * N + j) * C + cl);
    }
    if constexpr (FUSED) in.h.load(g_h, static_cast<size_t>(tl) * C + cl);
#pragma unroll
    for (int e = 0; e < CP / 4; ++e)
      if (FUSED || e == (N * N + 2 * N) / 4)
        in.rc[e] = *reinterpret_cast<const f32x4 *>(rec + tl * CP + 4 * e);
  };
  auto compute = [&](const In &in, int64_t t0) {
    const int64_t t = t0 + r;
    const bool live = t < te && col_ok;
    auto cf = [&](int e) { return in.rc[e >> 2][e & 3]; };
    const float cx = cf(N * N + 2 * N);
    f32x4 acc[N][TL];
#pragma unroll
    for (int j = 0; j < N; ++j)
#pragma unroll
      for (int h = 0; h < TL; ++h) acc[j][h] = f32x4{0.f, 0.f, 0.f, 0.f};
    auto group = [&](int s, const f32x4 &b) {
#pragma unroll
      for (int j = 0; j < N; ++j)
#pragma unroll
        for (int h = 0; h < TL; ++h) {
          const f32x4 a = wl[((j * TL + h) * S + s) * 64];
#pragma unroll
          for (int i = 0; i < 4; ++i) acc[j][h] = mfma_f32(a[i], b[i], acc[j][h]);
        }
    };
    if constexpr (SC > 0) {
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int s = 0; s < SC; ++s) group(s, in.b[s]);
      __builtin_amdgcn_sched_barrier(0);
    } else {
      const float *vrow = vr + (t < te ? t : te - 1) * (16 * S) + 4 * q;
      for (int s = 0; s < S; ++s) group(s, *reinterpret_cast<const f32x4 *>(vrow + 16 * s));
    }
    if constexpr (FUSED) {
      if (g_y != nullptr && live) {   // (optional output)
        float gy[V];
#pragma unroll
        for (int e = 0; e < V; ++e) {
          gy[e] = 0.f;
#pragma unroll
          for (int i = 0; i < N; ++i) gy[e] += cf(N * N + N + i) * in.g[i].at(e);
        }
        IO::store(g_y, t * C + c0, gy);
      }
    }
#pragma unroll
    for (int j = 0; j < N; ++j) {
      float o[V];
#pragma unroll
      for (int e = 0; e < V; ++e) {
        o[e] = acc[j][e >> 2][e & 3] - in.x[j].at(e) * cx;
        if constexpr (FUSED) {
#pragma unroll
          for (int i = 0; i < N; ++i) o[e] += cf(i * N + j) * in.g[i].at(e);
          o[e] += cf(N * N + j) * in.h.at(e);
        } else {
          o[e] += in.g[j].at(e);
        }
      }
      if (live) IO::store(g_x, (t * N + j) * C + c0, o);
    }
  };
  const int64_t step = 16 * subs;
  int64_t t0 = tb + 16 * sub;
  // (the next tokens' loads ahead of these tokens' work: 2 us slower at n = 4, C = 1024, bf16 and f32)
  for (; t0 < te; t0 += step) {
    In in;
    load(in, t0);
    compute(in, t0);
  }
}

template <typename IO, int N, bool FUSED>
__global__ __launch_bounds__(64 * kGxWaves, 1) void gx_fullprec_kernel(GxArgs p) {
  gx_fullprec<IO, N, 0, FUSED>(p.x, p.W, p.g_xout, p.g_h, p.rec, p.vr, p.M, p.S, p.C, p.T, p.win, p.tokens_per_block,
                               p.g_x, p.g_y, blockIdx.x, blockIdx.y);
}

// What is left of a backward once vr is there, in one launch: g_W (blocks [0, gw_blocks)), the columns of the g_z
// sums (g_b and g_alpha, one block each) and g_x, g_y.  None needs another's result, and all but the columns read x.
// With launch_proj_dots, steps in us, five launches / two or three: f32, n = 4, C = 64, 256 tokens 41.2 / 29.7; C = 768, 33
// tokens 44.1 / 34.0, 4096 tokens 166 / 150; bf16, n = 3, C = 200, 2000 tokens 41.4 / 34.5, n = 4, 10000 tokens 136 / 113;
// separable calls n = 4, C = 1024, 300 tokens 68 / 59, 5003 tokens 168 / 157.  By itself, the fused backward, two launches and the
// sums / one: n = 5, bf16, C = 1000, 300 tokens 63.6 / 51.2, 8000 342 / 337, 30000 1197 / 1169; n = 5, f32, 30000 tokens 1491 / 1482;
// n = 4, bf16, C = 1000, 80000 tokens 1800 / 1768, f32, C = 768, 40000 1030 / 1002, 80000 2000 / 2022; separable calls n = 4, C = 1024,
// 60000 tokens 1714 / 1673.
struct GwArgs {
  int64_t chunk;
  float *out;
  int xblocks, blocks;
};
template <typename IO, int N, int NT, bool FUSED>
__global__ __launch_bounds__(64 * kGxWaves, 1) void gx_gw_kernel(GxArgs p, GwArgs w, ColumnArgs z, int gx_xblocks) {
  static_assert(kGxWaves == kGwWaves, "one block size");
  int b = static_cast<int>(blockIdx.x);
  if (b < w.blocks) {
    gw_fullprec<IO, NT, gw_piece<IO, NT>()>(p.x, p.vr, N * p.C, p.M, p.T, w.chunk, w.out, b % w.xblocks,
                                            b / w.xblocks);
    return;
  }
  b -= w.blocks;
  if (b < p.M + 3) {
    column_sum(z, p.M + 3, b, p.M, reinterpret_cast<float *>(fullprec_lds));
    return;
  }
  b -= p.M + 3;
  gx_fullprec<IO, N, NT, FUSED>(p.x, p.W, p.g_xout, p.g_h, p.rec, p.vr, p.M, NT, p.C, p.T, p.win, p.tokens_per_block,
                            p.g_x, p.g_y, b % gx_xblocks, b / gx_xblocks);
}

// columns per wave
int gw_columns(const mhcl_desc &d, int M) {
  return d.io_dtype == MHCL_BF16 && logit_tiles(M) <= 3 ? 128 : 64;
}

}  // namespace

// Where the bf16 MFMA projection applies too, this one is used for few tokens: it spreads over the
// chip by splitting rows into more parts, but runs at the fp64 rate, so its time grows with the
// tokens and tiles where the other's is flat until its blocks fill the chip.  Both sides, mhcl_coeffs:
// n = 4, C = 1024, 256 tokens 10.5 / 14.7 us, 1024 tokens 13.6 / 15.1, 2048 tokens 18.7 / 15.2; C = 4096,
// 64 tokens 13.5 / 37.8, 1024 tokens 29.6 / 39.2, 1500 tokens 40.9 / 39.2; n = 3, C = 1024, 2000 tokens
// 12.3 / 12.7; n = 5, C = 2560 (nine tiles, where the other one packs W first), 500 tokens 83 / 106.
int64_t few_tokens(const mhcl_desc &d) {
  const int tiles = logit_tiles(res_logits(d) + 2 * d.n);
  return (tiles <= 4 ? 2500 : 5000) / tiles;
}
bool proj_fullprec_used(const mhcl_desc &d) { return !fast_path_ok(d) || d.T <= few_tokens(d); }

// Parts of a row: enough blocks for two per compute unit, each wave with at least one step, at most
// 16 (the coefficient stages add the slices; 4 instead of 16 for n = 5, C = 2560, 256 tokens: 105 us for mhcl_coeffs
// against 57), or 32 for a block or two of tokens with many products: forward, us, 16 / 32 parts at 16 tokens: n = 4, C = 4096
// 17.1 / 16.4, n = 5, C = 2048 36.6 / 32.9, n = 8, K = 64, C = 2048 34.9 / 29.6; but n = 3, C = 4096 15.8 / 16.4, n = 4, C = 2048
// 15.9 / 16.2, and for 256 tokens at n = 4, C = 4096 2 us more; f32 step at n = 4, C = 4096 41.3 / 42.6.
// Eight or nine tiles: 448 blocks are enough, so that the fp64 slices of any T fit in
// MHCL_STATIC_SCRATCH_BYTES (14304 slice-tokens of 143 logits and a sum of squares).
static int64_t enough_blocks(const mhcl_desc &d) {
  return logit_tiles(res_logits(d) + 2 * d.n) >= 8 ? 448 : 512;
}
int proj_fullprec_parts(const mhcl_desc &d) {
  const int V = d.io_dtype == MHCL_BF16 ? BF16::kVec : F32::kVec;
  const int nsteps = (d.n * d.C + 4 * V - 1) / (4 * V);
  const int64_t groups = (d.T + 15) / 16;
  // 32 where 16 leave a wave with 64 products or more of 32 tokens or fewer (128 for f32 streams)
  const int products = nsteps / (16 * kProjWaves) * V * logit_tiles(res_logits(d) + 2 * d.n);
  const int most = groups <= 2 && products >= (d.io_dtype == MHCL_BF16 ? 64 : 128) ? 32 : 16;
  int parts = 1;
  while (parts < most && groups * parts < enough_blocks(d) && nsteps >= 2 * parts * kProjWaves) parts *= 2;
  return parts;
}

RawSums projected(const mhcl_desc &d, const float *u_raw, const float *sumsq) {
  const int parts = proj_ksplit(d);
  return {u_raw, sumsq, parts, proj_fullprec_used(d) && parts > 1};
}

hipError_t add_wide_slices(const mhcl_desc &d, RawSums &raw, hipStream_t s) {
  if (!raw.wide) return hipErrorInvalidValue;
  const int64_t n_u = d.T * (res_logits(d) + 2 * d.n);
  auto go = [&](auto kern) {
    hipLaunchKernelGGL(kern, dim3(static_cast<unsigned>((n_u + d.T + 255) / 256)), dim3(256), 0, s,
                       reinterpret_cast<double *>(const_cast<float *>(raw.u_raw)),
                       reinterpret_cast<double *>(const_cast<float *>(raw.sumsq)), n_u, d.T);
    return hipGetLastError();
  };
  const int parts = raw.parts;
  raw.parts = 1;
  switch (parts) {
    case 2: return go(add_slices_kernel<2>);
    case 4: return go(add_slices_kernel<4>);
    case 8: return go(add_slices_kernel<8>);
    case 16: return go(add_slices_kernel<16>);
    case 32: return go(add_slices_kernel<32>);
  }
  return hipErrorInvalidValue;
}

// (p > 1 parts only up to 16 (2 enough_blocks / p - 1) tokens, see above)
int64_t proj_fullprec_slice_floats(const mhcl_desc &d) {
  mhcl_desc one = d;
  one.T = 1;
  int64_t T = d.T;
  if (fast_path_ok(d)) {   // above few_tokens the bf16 projection runs
    const int64_t few = few_tokens(d);
    if (T > few) T = few;
  }
  const int parts = proj_fullprec_parts(one);
  if (parts == 1) return T;
  const int64_t slices = slice_tokens(T, 2 * (parts < 16 ? parts : 16), 2 * 16 * 2 * enough_blocks(d));
  const int64_t first = 2 * parts * (T < 32 ? T : 32);   // (32 parts: of 32 tokens or fewer)
  return slices > first ? slices : first;
}

hipError_t launch_proj_fullprec(const mhcl_desc &d, int M, const void *x, const float *W,
                                float *u_raw, float *sumsq, hipStream_t s) {
  const int V = d.io_dtype == MHCL_BF16 ? BF16::kVec : F32::kVec;
  const int nC = d.n * d.C, parts = proj_fullprec_parts(d);
  const int nsteps = (nC + 4 * V - 1) / (4 * V), spp = (nsteps + parts - 1) / parts;
  const dim3 grid(static_cast<unsigned>((d.T + 15) / 16), parts);
  return dispatch_io(d.io_dtype, [&](auto io) {
    return dispatch_tiles(logit_tiles(M), [&](auto nt) {
      constexpr int NT = decltype(nt)::value;
      auto kern = proj_fullprec_kernel<decltype(io), NT, kProjWaves>;
      int waves = kProjWaves;
      if constexpr (NT >= 4) {   // (with fewer tiles the sums are short)
        if (nsteps <= 2) {
          kern = proj_fullprec_kernel<decltype(io), NT, 1>;
          waves = 1;
        }
      }
      hipLaunchKernelGGL(kern, grid, dim3(64 * waves), 0, s, x, W, nC, M, d.T, spp, u_raw, sumsq);
      return hipGetLastError();
    });
  });
}

hipError_t launch_proj_fullprec_layers(const mhcl_desc &d, int M, const JointLayers &layers, int L, float *u_raw,
                                       float *sumsq, hipStream_t s) {
  const int V = d.io_dtype == MHCL_BF16 ? BF16::kVec : F32::kVec;
  const int nC = d.n * d.C, parts = proj_fullprec_parts(d);
  const int nsteps = (nC + 4 * V - 1) / (4 * V), spp = (nsteps + parts - 1) / parts;
  const dim3 grid(static_cast<unsigned>((d.T + 15) / 16), parts, L);
  auto go = [&](auto nt) {
    return dispatch_io(d.io_dtype, [&](auto io) {
      hipLaunchKernelGGL((proj_fullprec_layers_kernel<decltype(io), decltype(nt)::value>), grid, dim3(64 * kProjWaves), 0,
                         s, layers, nC, M, d.T, spp, u_raw, sumsq);
      return hipGetLastError();
    });
  };
  switch (logit_tiles(M)) {   // (those of the forms of joint_layers_ok)
    case 1: return go(std::integral_constant<int, 1>{});
    case 2: return go(std::integral_constant<int, 2>{});
    case 3: return go(std::integral_constant<int, 3>{});
  }
  return hipErrorInvalidValue;
}

// Token chunks: one round of blocks on the 256 compute units, and no more than one per 256 tokens (two
// steps of its loop to run ahead in, four above three logit tiles).
int gw_chunks_fullprec(const mhcl_desc &d) {
  const int M = res_logits(d) + 2 * d.n, cols = gw_columns(d, M);
  const int64_t xblocks = (static_cast<int64_t>(d.n) * d.C + cols - 1) / cols;
  int64_t c = 256 / xblocks;
  if (c > (d.T + 255) / 256) c = (d.T + 255) / 256;
  return c < 1 ? 1 : static_cast<int>(c);
}

// (n, logit tiles) of the forms whose two roles are built as one launch: the full permutation form up to n = 4 and
// Sinkhorn-Knopp; at more tiles the products' registers would leave the other role short of waves
template <typename F>
static hipError_t dispatch_joint(const mhcl_desc &d, F &&f) {
  const int NT = logit_tiles(res_logits(d) + 2 * d.n);
  auto go = [&](auto nn, auto nt) { return NT == decltype(nt)::value ? f(nn, nt) : hipErrorInvalidValue; };
  using std::integral_constant;
  switch (d.n) {
    case 1: return go(integral_constant<int, 1>{}, integral_constant<int, 1>{});
    case 2: return go(integral_constant<int, 2>{}, integral_constant<int, 1>{});
    case 3: return go(integral_constant<int, 3>{}, integral_constant<int, 1>{});
    case 4: return go(integral_constant<int, 4>{}, integral_constant<int, 2>{});
    case 5: return go(integral_constant<int, 5>{}, integral_constant<int, 3>{});
  }
  return hipErrorInvalidValue;
}
// (the bound keeps the joint grid below 2^32 threads)
bool joint_fullprec_ok(const mhcl_desc &d) { return !coeffs_group_ok(d) && d.T <= (1 << 22); }

// Up to so many tokens: the dot products' blocks have eight waves and the registers of the projection's role, so with many tokens
// fewer waves stream than bwd_dots_kernel has on a compute unit (n = 5, bf16: 8 against 12).  The fused backward,
// us, two launches / one: n = 5, bf16, C = 1000, 400 tokens 56.1 / 51.6, 800 74.0 / 73.6, 1000 76.8 / 79.2, 8000 304 / 337, C = 200,
// 50000 533 / 631; n = 5, f32, C = 1000, 14000 tokens 704 / 699, 30000 1460 / 1482; n = 4, f32, C = 768, 4096 tokens 115 / 98 with
// gx_gw_kernel, 10000 255 / 245, 16000 380 / 391, bf16, C = 1000, 10000 238 / 226, 20000 448 / 454 (C = 4096 and C = 200 still gain
// there, 3 %); n = 3, f32, C = 768, 9000 tokens 148 / 144, 12000 195 / 197, bf16, C = 1000 122 / 116 and 155 / 158; n = 2, C = 768, 50000 tokens
// 648 / 629, C = 128, 150000 tokens 370 / 374; n = 1 likewise.
bool joint_proj_dots_ok(const mhcl_desc &d) {
  constexpr int64_t kMost[] = {0, 1 << 17, 1 << 17, 10240, 10240, 16384};
  return joint_fullprec_ok(d) && d.T <= (d.n == 5 && d.io_dtype == MHCL_BF16 ? 800 : kMost[d.n]);
}

hipError_t launch_proj_dots(const mhcl_desc &d, int M, const void *x, const float *W, const void *y,
                            const void *g_xout, const void *g_h, float *u_raw, float *sumsq, float *g_H_res,
                            float *g_H_post, float *g_H_pre, hipStream_t s) {
  const int V = d.io_dtype == MHCL_BF16 ? BF16::kVec : F32::kVec;
  const int nC = d.n * d.C, parts = proj_fullprec_parts(d);
  const int nsteps = (nC + 4 * V - 1) / (4 * V), spp = (nsteps + parts - 1) / parts;
  const int groups = static_cast<int>((d.T + 15) / 16);
  const DotsArgs p{y, g_xout, g_h, g_H_res, g_H_post, g_H_pre, d.C, waves_that_fit(d.C, V)};
  const int per_block = kProjWaves / p.waves;
  const int64_t blocks = groups * static_cast<int64_t>(parts) + (d.T + per_block - 1) / per_block;
  return dispatch_io(d.io_dtype, [&](auto io) {
    return dispatch_joint(d, [&](auto nn, auto nt) {
      hipLaunchKernelGGL((proj_dots_kernel<decltype(io), decltype(nn)::value, decltype(nt)::value>),
                         dim3(static_cast<unsigned>(blocks)), dim3(64 * kProjWaves), 0, s, x, W, nC, M, d.T, spp,
                         u_raw, sumsq, groups, parts, p);
      return hipGetLastError();
    });
  });
}

hipError_t launch_gw_fullprec(const mhcl_desc &d, int M, const void *x, const float *vr,
                              float *partials, float *g_W, hipStream_t s) {
  const int chunks = gw_chunks_fullprec(d), cols = gw_columns(d, M), nC = d.n * d.C;
  const int64_t chunk = (d.T + chunks - 1) / chunks;
  float *dst = chunks == 1 ? g_W : partials;
  const dim3 grid((nC + cols - 1) / cols, chunks);
  return dispatch_io(d.io_dtype, [&](auto io) {   // (the chunks are added by launch_bwd_finish)
    return dispatch_tiles(logit_tiles(M), [&](auto nt) {
      using IO = decltype(io);
      constexpr int NT = decltype(nt)::value;
      hipLaunchKernelGGL((gw_fullprec_kernel<IO, NT, gw_piece<IO, NT>()>), grid, dim3(64 * kGwWaves), kGwLds, s, x,
                         vr, nC, M, d.T, chunk, dst);
      return hipGetLastError();
    });
  });
}

// Windows of W per block, blocks along C and tokens per block: one round of resident blocks, two per compute unit.  In one launch
// with g_W, whose up to 256 blocks come first, half as many (whole step or separable calls, two per compute unit / one: f32, n = 4, C = 768,
// 4096 tokens 153 / 150 us; bf16, C = 1024, 5003 tokens 162 / 156, C = 200, 10000 tokens 123 / 113).  Up to n = 3, and at n = 4
// in f32, the registers let a block of either role stand on a compute unit at once; elsewhere (148 to 224 registers) g_x follows
// as the blocks of g_W end.
struct GxShape {
  int win, lds, xblocks, tokens_per_block, chunks;
};
static GxShape gx_shape(const mhcl_desc &d, int S, bool joint) {
  const int V = d.io_dtype == MHCL_BF16 ? BF16::kVec : F32::kVec;
  const int per_win = d.n * (V / 4) * S * 1024;   // bytes of W in LDS per window (144 KiB at most)
  const int windows = (d.C + 4 * V - 1) / (4 * V);
  GxShape g;
  g.win = kGxWaves;   // adjacent windows per block: two blocks per compute unit where possible
  while (g.win > 1 && (g.win * per_win > 64 * 1024 || g.win > windows)) g.win /= 2;
  g.lds = g.win * per_win;
  g.xblocks = (windows + g.win - 1) / g.win;
  const int64_t step = 16 * (kGxWaves / g.win);     // tokens of one round of the block's waves
  int64_t chunks = (!joint && g.lds <= 80 * 1024 ? 512 : 256) / g.xblocks;
  if (chunks < 1) chunks = 1;
  g.tokens_per_block = static_cast<int>(((d.T + chunks - 1) / chunks + step - 1) / step * step);
  g.chunks = static_cast<int>((d.T + g.tokens_per_block - 1) / g.tokens_per_block);
  return g;
}

hipError_t launch_gx_gw_fullprec(const mhcl_desc &d, int M, bool fused, const void *x, const float *W,
                                 const void *g_xout, const void *g_h, const BwdTokenBufs &o, void *g_x, void *g_y,
                                 float *partials, float *g_W, int64_t gz_count, float *g_b, float *g_alpha,
                                 hipStream_t s) {
  const GxShape g = gx_shape(d, logit_tiles(M), true);
  const int cols = gw_columns(d, M), chunks = gw_chunks_fullprec(d);
  GwArgs w;
  w.chunk = (d.T + chunks - 1) / chunks;
  w.out = chunks == 1 ? g_W : partials;
  w.xblocks = (d.n * d.C + cols - 1) / cols;
  w.blocks = w.xblocks * chunks;
  const ColumnArgs z{o.gz, gz_count, g_b, g_alpha};
  const GxArgs p{x, W, g_xout, g_h, o.rec, o.vr, M, logit_tiles(M), d.C, d.T, g.win, g.tokens_per_block, g_x, g_y};
  const unsigned blocks = w.blocks + M + 3 + g.xblocks * g.chunks;
  return dispatch_io(d.io_dtype, [&](auto io) {
    return dispatch_joint(d, [&](auto nn, auto nt) {
      using IO = decltype(io);
      constexpr int N = decltype(nn)::value, NT = decltype(nt)::value;
      auto kern = fused ? gx_gw_kernel<IO, N, NT, true> : gx_gw_kernel<IO, N, NT, false>;
      // (up to three tiles a window of W is at most 64 KiB)
      hipLaunchKernelGGL(kern, dim3(blocks), dim3(64 * kGxWaves), g.lds > kGwLds ? g.lds : kGwLds, s, p, w, z,
                         g.xblocks);
      return hipGetLastError();
    });
  });
}

hipError_t launch_gx_fullprec(const mhcl_desc &d, int M, bool fused, const void *x, const float *W,
                              const void *g_xout, const void *g_h, const BwdTokenBufs &o, void *g_x,
                              void *g_y, hipStream_t s) {
  const int S = logit_tiles(M);
  const GxShape g = gx_shape(d, S, false);
  const GxArgs p{x, W, g_xout, g_h, o.rec, o.vr, M, S, d.C, d.T, g.win, g.tokens_per_block, g_x, g_y};
  const dim3 grid(g.xblocks, g.chunks);
  return dispatch_io(d.io_dtype, [&](auto io) {
    return dispatch_n(d.n, [&](auto nn) {
      using IO = decltype(io);
      constexpr int N = decltype(nn)::value;
      auto kern = fused ? gx_fullprec_kernel<IO, N, true> : gx_fullprec_kernel<IO, N, false>;
      if (g.lds > 64 * 1024) {   // (one window then; the limit of the kernel, whatever thread launches it with how many logits)
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kern),
                                           hipFuncAttributeMaxDynamicSharedMemorySize,
                                           N * (IO::kVec / 4) * 9 * 1024);
        if (e != hipSuccess) return e;
      }
      hipLaunchKernelGGL(kern, grid, dim3(64 * kGxWaves), g.lds, s, p);
      return hipGetLastError();
    });
  });
}

}  // namespace mhcl
