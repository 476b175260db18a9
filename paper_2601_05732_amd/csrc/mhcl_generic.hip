// Stream kernels of libmhcl: plain fp32 arithmetic on bf16 or f32 streams, any n in 1..8 and any C.
// They are bound by HBM.  Every reduction runs in a fixed order, so results are bitwise
// reproducible.
#include "mhcl_common.h"
#include "mhcl_internal.h"
#include "mhcl_mfma.h"

namespace mhcl {

namespace {

constexpr int kBlock = 256;

// Sum over the block of CNT per-thread values; the totals land in red[0..CNT).  Fixed order:
// butterfly inside each wave, then the waves in order.
template <int WAVES, int CNT>
__device__ __forceinline__ void block_sum(float (&v)[CNT], float *red /* [WAVES * CNT] */) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
  for (int i = 0; i < CNT; ++i) {
    const float s = wave_sum(v[i]);
    if (lane == 0) red[wave * CNT + i] = s;
  }
  __syncthreads();
  for (int i = threadIdx.x; i < CNT; i += 64 * WAVES) {
    float s = red[i];
#pragma unroll
    for (int w = 1; w < WAVES; ++w) s += red[w * CNT + i];
    red[i] = s;
  }
  __syncthreads();
}

// The kernels that take one block per token, W: the wave counts a kernel is built for
template <int... W, typename F>
hipError_t dispatch_waves(std::integer_sequence<int, W...>, int waves, F &&f) {
  hipError_t e = hipErrorInvalidValue;
  ((waves == W ? (void)(e = f(std::integral_constant<int, W>{})) : (void)0), ...);
  return e;
}
// post_bwd_kernel: waves that fit, against four always (idle waves take registers and wait at the sums;
// us per call, four / as many as fit): n = 4, C = 64, 4096 tokens 30.1 / 11.6, C = 1024, 32768 tokens 233 /
// 165, n = 8, f32, C = 768 759 / 584.  Four where all blocks are resident at once anyway (n = 8, C = 64,
// 512 tokens 20.3 / 22.4, n = 5 10.3 / 11.3), and where HBM bounds the kernel and smaller blocks only
// spread its rows (n = 2, C = 1024, 65536 tokens 182 / 193; n = 5, f32, C = 768, 32768 tokens 313 / 340).
int post_bwd_waves(const mhcl_desc &d, int vec) {
  const int fit = waves_that_fit(d.C, vec);
  const int64_t resident = 256 * (d.n >= 7 ? 2 : (d.n >= 5 ? 3 : 4));
  if (d.T <= resident ||
      (fit == 2 && d.n <= (vec == 4 ? 3 : 2) && d.T > 16384) ||
      (fit == 3 && vec == 4 && d.n <= 5)) return 4;
  return fit;
}
// pre_bwd_kernel: one wave likewise (n = 4, C = 64, 32768 tokens 60.4 / 24.1; n = 8, 1280 tokens 7.3 / 8.2),
// two for bf16 rows while the streams stay in cache (n = 8, C = 768, 2048 tokens 17.7 / 14.2; n = 4, C = 768,
// 65536 tokens 228 / 246), three never (n = 2, f32, C = 768, 16384 tokens 43.9 / 45.2)
int pre_bwd_waves(const mhcl_desc &d, int vec) {
  const int fit = waves_that_fit(d.C, vec);
  if (d.T <= 1536) return 4;
  return fit == 1 || (fit == 2 && vec == 8 && d.T <= 16384) ? fit : 4;
}

// ------------------------------------------------------------ stream mixing
// h = H_pre x   (Eq. 1, argument of f): one thread per 16-byte chunk of h.
template <typename IO, int N>
__global__ __launch_bounds__(kBlock) void pre_kernel(const void *__restrict__ x,
                                                     const float *__restrict__ H_pre,
                                                     void *__restrict__ h, int C, int64_t T) {
  constexpr int V = IO::kVec;
  const int vpr = C / V;
  const int64_t idx = static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x;
  if (idx >= T * vpr) return;
  const int64_t t = idx / vpr;
  const int c = static_cast<int>(idx % vpr) * V;
  float acc[V];
#pragma unroll
  for (int e = 0; e < V; ++e) acc[e] = 0.f;
#pragma unroll
  for (int j = 0; j < N; ++j) {
    float v[V];
    IO::load(x, (t * N + j) * C + c, v);
    const float w = H_pre[t * N + j];
#pragma unroll
    for (int e = 0; e < V; ++e) acc[e] = fmaf(w, v[e], acc[e]);
  }
  IO::store(h, t * C + c, acc);
}

// The ends of a stack, one thread per 16-byte chunk of a row of C.  Bound by HBM or the memory-side cache: n = 4, C = 1024,
// 2048 tokens, bf16, us a call, torch's copy and sum / these: in 16.0 / 6.1 (21 MB), out 7.5 / 4.3.
template <typename IO, int N>
__global__ __launch_bounds__(kBlock) void streams_in_kernel(const u32x4 *__restrict__ x0, u32x4 *__restrict__ x, int C,
                                                            int64_t T) {
  const int vpr = C / IO::kVec;
  const int64_t idx = static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x;
  if (idx >= T * vpr) return;
  const int64_t t = idx / vpr, c = idx - t * vpr;
  const u32x4 v = x0[idx];
#pragma unroll
  for (int j = 0; j < N; ++j) x[(t * N + j) * vpr + c] = v;
}
template <typename IO, int N>
__global__ __launch_bounds__(kBlock) void streams_out_kernel(const void *__restrict__ x, void *__restrict__ out, int C,
                                                             int64_t T) {
  constexpr int V = IO::kVec;
  const int vpr = C / V;
  const int64_t idx = static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x;
  if (idx >= T * vpr) return;
  const int64_t t = idx / vpr;
  const int c = static_cast<int>(idx % vpr) * V;
  float acc[V], v[N][V];
#pragma unroll
  for (int j = 0; j < N; ++j) IO::load(x, (t * N + j) * C + c, v[j]);
#pragma unroll
  for (int e = 0; e < V; ++e) {
    acc[e] = v[0][e];
#pragma unroll
    for (int j = 1; j < N; ++j) acc[e] += v[j][e];
  }
  IO::store(out, t * C + c, acc);
}

// x_out = H_res x + H_post^T y   (Eq. 1). Bound by memory: one pass over x, y and x_out. Stores past the caches leave x, which
// the backward reads again, in the last-level cache; the rule and its figures stand at launch_post.
enum class Past { kNone, kStores, kAll };   // which accesses go past the caches
template <typename IO, int N, Past PAST>
__global__ __launch_bounds__(kBlock) void post_kernel(const void *__restrict__ x,
                                                      const void *__restrict__ y,
                                                      const float *__restrict__ H_res,
                                                      const float *__restrict__ H_post,
                                                      void *__restrict__ x_out, int C, int64_t T) {
  constexpr int V = IO::kVec;
  const int vpr = C / V;
  const int64_t idx = static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x;
  if (idx >= T * vpr) return;
  const int64_t t = idx / vpr;
  const int c = static_cast<int>(idx % vpr) * V;
  float xv[N][V], yv[V];
#pragma unroll
  for (int j = 0; j < N; ++j) {
    if constexpr (PAST == Past::kAll)
      IO::load_once(x, (t * N + j) * C + c, xv[j]);
    else
      IO::load(x, (t * N + j) * C + c, xv[j]);
  }
  if constexpr (PAST == Past::kAll)
    IO::load_once(y, t * C + c, yv);
  else
    IO::load(y, t * C + c, yv);
#pragma unroll
  for (int i = 0; i < N; ++i) {
    float acc[V];
#pragma unroll
    for (int e = 0; e < V; ++e) acc[e] = 0.f;
#pragma unroll
    for (int j = 0; j < N; ++j) {
      const float w = H_res[(t * N + i) * N + j];
#pragma unroll
      for (int e = 0; e < V; ++e) acc[e] += w * xv[j][e];
    }
    const float wp = H_post[t * N + i];
#pragma unroll
    for (int e = 0; e < V; ++e) acc[e] += wp * yv[e];
    if constexpr (PAST != Past::kNone)
      IO::store_once(x_out, (t * N + i) * C + c, acc);
    else
      IO::store(x_out, (t * N + i) * C + c, acc);
  }
}

// Backward of post: one block per token.
//   g_y = sum_i H_post[i] g_xout[i];  g_x[j] = sum_i H_res[i][j] g_xout[i]
//   g_H_post[i] = <g_xout[i], y>;     g_H_res[i][j] = <g_xout[i], x[j]>
template <typename IO, int N, int WAVES>
__global__ __launch_bounds__(64 * WAVES) void post_bwd_kernel(
    const void *__restrict__ x, const void *__restrict__ y, const float *__restrict__ H_res,
    const float *__restrict__ H_post, const void *__restrict__ g_xout, void *__restrict__ g_x,
    void *__restrict__ g_y, float *__restrict__ g_H_res, float *__restrict__ g_H_post, int C) {
  constexpr int V = IO::kVec;
  constexpr int D = N * N + N;
  __shared__ float red[WAVES * D];
  const int64_t t = blockIdx.x;
  float Hr[N * N], Hq[N], dots[D];
#pragma unroll
  for (int e = 0; e < N * N; ++e) Hr[e] = H_res[t * N * N + e];
#pragma unroll
  for (int i = 0; i < N; ++i) Hq[i] = H_post[t * N + i];
#pragma unroll
  for (int e = 0; e < D; ++e) dots[e] = 0.f;
  for (int c = threadIdx.x * V; c < C; c += 64 * WAVES * V) {
    float xv[N][V], gv[N][V], yv[V];
#pragma unroll
    for (int j = 0; j < N; ++j) {
      IO::load(x, (t * N + j) * C + c, xv[j]);
      IO::load(g_xout, (t * N + j) * C + c, gv[j]);
    }
    IO::load(y, t * C + c, yv);
    float gy[V];
#pragma unroll
    for (int e = 0; e < V; ++e) gy[e] = 0.f;
#pragma unroll
    for (int i = 0; i < N; ++i) {
#pragma unroll
      for (int e = 0; e < V; ++e) {
        gy[e] += Hq[i] * gv[i][e];
        dots[N * N + i] += gv[i][e] * yv[e];
      }
#pragma unroll
      for (int j = 0; j < N; ++j)
#pragma unroll
        for (int e = 0; e < V; ++e) dots[i * N + j] += gv[i][e] * xv[j][e];
    }
    IO::store(g_y, t * C + c, gy);
#pragma unroll
    for (int j = 0; j < N; ++j) {
      float gx[V];
#pragma unroll
      for (int e = 0; e < V; ++e) gx[e] = 0.f;
#pragma unroll
      for (int i = 0; i < N; ++i)
#pragma unroll
        for (int e = 0; e < V; ++e) gx[e] += Hr[i * N + j] * gv[i][e];
      IO::store(g_x, (t * N + j) * C + c, gx);
    }
  }
  block_sum<WAVES, D>(dots, red);
  for (int e = threadIdx.x; e < N * N; e += 64 * WAVES) g_H_res[t * N * N + e] = red[e];
  if (threadIdx.x < N) g_H_post[t * N + threadIdx.x] = red[N * N + threadIdx.x];
}

// Backward of pre: g_x[j] += H_pre[j] g_h ; g_H_pre[j] = <g_h, x[j]>
template <typename IO, int N, int WAVES>
__global__ __launch_bounds__(64 * WAVES) void pre_bwd_kernel(const void *__restrict__ x,
                                                         const float *__restrict__ H_pre,
                                                         const void *__restrict__ g_h,
                                                         void *__restrict__ g_x,
                                                         float *__restrict__ g_H_pre, int C) {
  constexpr int V = IO::kVec;
  __shared__ float red[WAVES * N];
  const int64_t t = blockIdx.x;
  float Hp[N], dots[N];
#pragma unroll
  for (int j = 0; j < N; ++j) { Hp[j] = H_pre[t * N + j]; dots[j] = 0.f; }
  for (int c = threadIdx.x * V; c < C; c += 64 * WAVES * V) {
    float gh[V];
    IO::load(g_h, t * C + c, gh);
#pragma unroll
    for (int j = 0; j < N; ++j) {
      float xv[V], gx[V];
      IO::load(x, (t * N + j) * C + c, xv);
      IO::load(g_x, (t * N + j) * C + c, gx);
#pragma unroll
      for (int e = 0; e < V; ++e) {
        dots[j] += gh[e] * xv[e];
        gx[e] += Hp[j] * gh[e];
      }
      IO::store(g_x, (t * N + j) * C + c, gx);
    }
  }
  block_sum<WAVES, N>(dots, red);
  if (threadIdx.x < N) g_H_pre[t * N + threadIdx.x] = red[threadIdx.x];
}

// The n^2 + 2n reductions over C that the backward needs, without outputs.
template <typename IO, int N, int WAVES>
__global__ __launch_bounds__(64 * WAVES) void bwd_dots_kernel(
    const void *__restrict__ x, const void *__restrict__ y, const void *__restrict__ g_xout,
    const void *__restrict__ g_h, float *__restrict__ g_H_res, float *__restrict__ g_H_post,
    float *__restrict__ g_H_pre, int C) {
  constexpr int V = IO::kVec;
  constexpr int D = N * N + 2 * N;
  __shared__ float red[WAVES * D];
  const int64_t t = blockIdx.x;
  float dots[D];
#pragma unroll
  for (int e = 0; e < D; ++e) dots[e] = 0.f;
  for (int c = threadIdx.x * V; c < C; c += 64 * WAVES * V) {
    float xv[N][V], gv[N][V], yv[V], gh[V];
#pragma unroll
    for (int j = 0; j < N; ++j) {
      IO::load(x, (t * N + j) * C + c, xv[j]);
      IO::load(g_xout, (t * N + j) * C + c, gv[j]);
    }
    IO::load(y, t * C + c, yv);
    IO::load(g_h, t * C + c, gh);
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
  block_sum<WAVES, D>(dots, red);
  for (int e = threadIdx.x; e < N * N; e += 64 * WAVES) g_H_res[t * N * N + e] = red[e];
  if (threadIdx.x < N) {
    g_H_post[t * N + threadIdx.x] = red[N * N + threadIdx.x];
    g_H_pre[t * N + threadIdx.x] = red[N * N + N + threadIdx.x];
  }
}

// The end of a backward in one launch.  Blocks [0, nbW): g_W = sum over the token chunks' partial
// sums, in a fixed association: the GR groups of threads of a block each add every GR-th chunk for
// the same 256 / GR elements (eight independent loads in flight), then the groups' sums in order.
// Many chunks of few elements take more groups, or a thread would walk down them one round trip after
// another (256 chunks of n = 3, C = 64: 11 -> 6 us with 16 groups instead of 4); with blocks enough for the
// chip they do not, since a group's loads are then 64 bytes long instead of 256 (64 chunks of n = 4, C = 512:
// 8.2 us with 16 groups, 4.3 with 4).
// Block nbW + c: column c of the [rows, ld] matrix of g_z sums per 32 or 64 tokens (none if its launch has had them).
// V: elements of a thread, four where that leaves blocks for the chip (steps, us, one / four: n = 5, C = 2560, 16384 tokens
// 1239 / 1232, C = 2048, 100 tokens 146.7 / 142.6; n = 7, K = 100 755 / 751; n = 4, C = 2048, 4000 tokens 154.9 / 154.0).
template <int GR, int V>
__global__ __launch_bounds__(kBlock) void bwd_finish_kernel(const float *__restrict__ part,
                                                            size_t size, int chunks, int nbW,
                                                            float *__restrict__ out, ColumnArgs columns, int M) {
  using Vec = float __attribute__((ext_vector_type(V)));
  constexpr int EB = kBlock / GR;
  __shared__ Vec red[kBlock];
  if (static_cast<int>(blockIdx.x) < nbW) {
    const int el = threadIdx.x % EB, grp = threadIdx.x / EB;
    const size_t i = (static_cast<size_t>(blockIdx.x) * EB + el) * V;   // (size is a multiple of V)
    Vec s = 0.f;
    if (i < size) {
#pragma unroll 8
      for (int c = grp; c < chunks; c += GR) s += *reinterpret_cast<const Vec *>(part + c * size + i);
    }
    red[threadIdx.x] = s;
    __syncthreads();
    if (grp == 0 && i < size) {
#pragma unroll
      for (int w = 1; w < GR; ++w) s += red[w * EB + el];
      *reinterpret_cast<Vec *>(out + i) = s;
    }
    return;
  }
  column_sum(columns, M + 3, static_cast<int>(blockIdx.x) - nbW, M, reinterpret_cast<float *>(red));
}

__global__ __launch_bounds__(kBlock) void fill_zero_kernel(float *__restrict__ p, size_t count) {
  const size_t i = static_cast<size_t>(blockIdx.x) * kBlock + threadIdx.x;
  if (i < count) p[i] = 0.f;
}

// 16 bytes per thread and iteration, grid-stride
__global__ __launch_bounds__(kBlock) void copy_kernel(uint4 *__restrict__ dst,
                                                      const uint4 *__restrict__ src, size_t n16) {
  for (size_t i = static_cast<size_t>(blockIdx.x) * kBlock + threadIdx.x; i < n16;
       i += static_cast<size_t>(gridDim.x) * kBlock)
    dst[i] = src[i];
}

inline unsigned blocks_for(int64_t items, int per) {
  return static_cast<unsigned>((items + per - 1) / per);
}

}  // namespace

// ================================================================ launchers
hipError_t launch_pre(const mhcl_desc &d, const void *x, const float *H_pre, void *h, hipStream_t s) {
  return dispatch_io(d.io_dtype, [&](auto io) {
    return dispatch_n(d.n, [&](auto nn) {
      using IO = decltype(io);
      constexpr int N = decltype(nn)::value;
      hipLaunchKernelGGL((pre_kernel<IO, N>), dim3(blocks_for(d.T * (d.C / IO::kVec), kBlock)),
                         dim3(kBlock), 0, s, x, H_pre, h, d.C, d.T);
      return hipGetLastError();
    });
  });
}

hipError_t launch_streams_in(const mhcl_desc &d, const void *x0, void *x, hipStream_t s) {
  return dispatch_io(d.io_dtype, [&](auto io) {
    return dispatch_n(d.n, [&](auto nn) {
      using IO = decltype(io);
      hipLaunchKernelGGL((streams_in_kernel<IO, decltype(nn)::value>), dim3(blocks_for(d.T * (d.C / IO::kVec), kBlock)),
                         dim3(kBlock), 0, s, static_cast<const u32x4 *>(x0), static_cast<u32x4 *>(x), d.C, d.T);
      return hipGetLastError();
    });
  });
}
hipError_t launch_streams_out(const mhcl_desc &d, const void *x, void *out, hipStream_t s) {
  return dispatch_io(d.io_dtype, [&](auto io) {
    return dispatch_n(d.n, [&](auto nn) {
      using IO = decltype(io);
      hipLaunchKernelGGL((streams_out_kernel<IO, decltype(nn)::value>), dim3(blocks_for(d.T * (d.C / IO::kVec), kBlock)),
                         dim3(kBlock), 0, s, x, out, d.C, d.T);
      return hipGetLastError();
    });
  });
}

hipError_t launch_post(const mhcl_desc &d, const void *x, const void *y, const float *H_res,
                       const float *H_post, void *x_out, hipStream_t s) {
  return dispatch_io(d.io_dtype, [&](auto io) {
    return dispatch_n(d.n, [&](auto nn) {
      using IO = decltype(io);
      constexpr int N = decltype(nn)::value;
      const int64_t x_bytes = d.T * N * d.C * (16 / IO::kVec);
      auto go = [&](auto past) {
        hipLaunchKernelGGL((post_kernel<IO, N, decltype(past)::value>), dim3(blocks_for(d.T * (d.C / IO::kVec), kBlock)),
                           dim3(kBlock), 0, s, x, y, H_res, H_post, x_out, d.C, d.T);
        return hipGetLastError();
      };
      // Figures: us a layer of four (three above 256 MiB) in a row, x_out being the next one's x; f forward, t forward and backward.
      // x that exceeds the last-level cache has left it before any later reader comes, and is then read past it as well, with y
      // (stores alone / both: n = 3, C = 1024, 45000 tokens f 236 / 219, t 697 / 680; n = 4, C = 4096, 8400 tokens f 223 / 210, t 687 / 674;
      // n = 8, C = 1024, 64 permutations, 17000 tokens f 266 / 263, t 932 / 932; f32, none / both, n = 4, C = 1024, 17000 tokens f 304 / 293,
      // t 871 / 855). The same layer step after step on the same inputs loses up to 1.7 % with both between 256 and 330 MiB (n = 8, 17000
      // tokens 889 / 904) and gains above; up to 256 MiB its backward may still find x there (n = 8, 16384 tokens 795 / 826).
      if (x_bytes > kLastLevelCache) return go(std::integral_constant<Past, Past::kAll>{});
      // bf16, none / stores: n = 4, C = 1024, 2048 tokens f 24.5 / 23.6, t 74.1 / 73.6, 8192 tokens f 68.3 / 66.0, t 184.5 / 183.7; Sinkhorn-Knopp,
      // C = 768, 3001 tokens f 25.4 / 25.1, t 79.3 / 77.9; n = 2, C = 1024, 32768 tokens f 142 / 132, t 389 / 376. What loses: x of 24 to 32 MiB,
      // forward only (n = 4, C = 1024, 3000 tokens f 28.8 / 29.5, t 89.3 / 89.5). Below 4 MiB x_out stays in the L2s for the next layer
      // (n = 4, C = 4096, 64 tokens f 19.6 / 19.8, C = 512, 700 tokens f 16.6 / 16.8; at 4 MiB, C = 2048, 256 tokens f 18.33 / 18.26). More than
      // 64 logits, whose projection walks x in another form: n = 5, C = 1024, 4096 tokens, M = 64 f 51.8 / 51.6, M = 66 f 52.9 / 54.9,
      // t 178 / 181, M = 130 f 72.2 / 74.2; 7000 tokens f 104.7 / 104.4, C = 2560, 3000 tokens (73 MiB) f 140.7 / 142.9, 4096 tokens f 178 / 176, t 523 / 517.
      // f32 gains 0 to 2 % and loses 2 to 3 % where a step's tensors just fill that cache (C = 768, 3500 tokens 142.3 / 146.6).
      if constexpr (IO::kVec == BF16::kVec) {
        if (x_bytes >= (res_logits(d) + 2 * N > 64 ? int64_t{80} << 20 : int64_t{4} << 20))
          return go(std::integral_constant<Past, Past::kStores>{});
      }
      return go(std::integral_constant<Past, Past::kNone>{});
    });
  });
}

hipError_t launch_post_bwd(const mhcl_desc &d, const void *x, const void *y, const float *H_res,
                           const float *H_post, const void *g_xout, void *g_x, void *g_y,
                           float *g_H_res, float *g_H_post, hipStream_t s) {
  return dispatch_io(d.io_dtype, [&](auto io) {
    return dispatch_n(d.n, [&](auto nn) {
      using IO = decltype(io);
      constexpr int N = decltype(nn)::value;
      using Waves = std::conditional_t<(IO::kVec == 4 && N <= 5), std::integer_sequence<int, 1, 2, 4>,
                                       std::integer_sequence<int, 1, 2, 3, 4>>;
      return dispatch_waves(Waves{}, post_bwd_waves(d, IO::kVec), [&](auto ww) {
        constexpr int W = decltype(ww)::value;
        hipLaunchKernelGGL((post_bwd_kernel<IO, N, W>), dim3(static_cast<unsigned>(d.T)), dim3(64 * W), 0, s,
                           x, y, H_res, H_post, g_xout, g_x, g_y, g_H_res, g_H_post, d.C);
        return hipGetLastError();
      });
    });
  });
}

hipError_t launch_pre_bwd(const mhcl_desc &d, const void *x, const float *H_pre, const void *g_h,
                          void *g_x, float *g_H_pre, hipStream_t s) {
  return dispatch_io(d.io_dtype, [&](auto io) {
    return dispatch_n(d.n, [&](auto nn) {
      using IO = decltype(io);
      constexpr int N = decltype(nn)::value;
      using Waves = std::conditional_t<IO::kVec == 8, std::integer_sequence<int, 1, 2, 4>,
                                       std::integer_sequence<int, 1, 4>>;
      return dispatch_waves(Waves{}, pre_bwd_waves(d, IO::kVec), [&](auto ww) {
        constexpr int W = decltype(ww)::value;
        hipLaunchKernelGGL((pre_bwd_kernel<IO, N, W>), dim3(static_cast<unsigned>(d.T)), dim3(64 * W), 0, s,
                           x, H_pre, g_h, g_x, g_H_pre, d.C);
        return hipGetLastError();
      });
    });
  });
}

hipError_t launch_bwd_dots(const mhcl_desc &d, const void *x, const void *y, const void *g_xout,
                           const void *g_h, float *g_H_res, float *g_H_post, float *g_H_pre,
                           hipStream_t s) {
  return dispatch_io(d.io_dtype, [&](auto io) {
    return dispatch_n(d.n, [&](auto nn) {
      using IO = decltype(io);
      constexpr int N = decltype(nn)::value;
      return dispatch_waves(std::integer_sequence<int, 1, 2, 3, 4>{}, waves_that_fit(d.C, IO::kVec), [&](auto ww) {
        constexpr int W = decltype(ww)::value;
        hipLaunchKernelGGL((bwd_dots_kernel<IO, N, W>), dim3(static_cast<unsigned>(d.T)), dim3(64 * W), 0, s,
                           x, y, g_xout, g_h, g_H_res, g_H_post, g_H_pre, d.C);
        return hipGetLastError();
      });
    });
  });
}

hipError_t launch_bwd_finish(const float *partials, size_t size, int chunks, float *g_W,
                             const float *gz_rows, int64_t rows, int M, float *g_b, float *g_alpha,
                             hipStream_t s) {
  auto go = [&](auto gr, auto vv) {
    constexpr int GR = decltype(gr)::value, V = decltype(vv)::value;
    const int nbW = chunks > 1 ? static_cast<int>(blocks_for(size, kBlock / GR * V)) : 0;
    hipLaunchKernelGGL((bwd_finish_kernel<GR, V>), dim3(nbW + (rows > 0 ? M + 3 : 0)), dim3(kBlock), 0, s, partials,
                       size, chunks, nbW, g_W, ColumnArgs{gz_rows, rows, g_b, g_alpha}, M);
    return hipGetLastError();
  };
  using One = std::integral_constant<int, 1>;
  using Four = std::integral_constant<int, 4>;
  if (size % 4 == 0 && size >= (1 << 17)) return go(Four{}, Four{});
  return chunks > 32 && size < 64 * 256 ? go(std::integral_constant<int, 16>{}, One{}) : go(Four{}, One{});
}

hipError_t launch_copy(void *dst, const void *src, size_t bytes, hipStream_t s) {
  const size_t n16 = bytes / 16;
  if (n16 == 0) return hipSuccess;
  size_t blocks = (n16 + kBlock - 1) / kBlock;
  if (blocks > 256 * 32) blocks = 256 * 32;
  hipLaunchKernelGGL(copy_kernel, dim3(static_cast<unsigned>(blocks)), dim3(kBlock), 0, s,
                     static_cast<uint4 *>(dst), static_cast<const uint4 *>(src), n16);
  return hipGetLastError();
}

hipError_t launch_fill_zero(float *p, size_t count, hipStream_t s) {
  if (count == 0) return hipSuccess;
  hipLaunchKernelGGL(fill_zero_kernel, dim3(blocks_for(count, kBlock)), dim3(kBlock), 0, s, p, count);
  return hipGetLastError();
}

}  // namespace mhcl
