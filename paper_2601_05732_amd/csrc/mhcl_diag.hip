// Diagnostics kernels of libmhcl: the logits of a layer with the relative
// range of the Sinkhorn-Knopp input (Sec. 3.1, Eq. 3), and column sums / l1
// errors of single residual matrices and of their product over the layers
// (Sec. 3.1, footnote 1; Sec. 4.3).  Plain fp32.
#include "mhcl_common.h"
#include "mhcl_internal.h"

namespace mhcl {

namespace {

// z[t][m] = alpha_g (r u_raw[t][m]) + b[m], the same expression the coefficient
// kernels evaluate; spread[t] = max - min of the residual logits, which is
// log(1/nu) of exp(z_res) (every entry of exp(.) is positive).
// A block takes 256 / LANES tokens, whose logits are one contiguous run of u_raw and of z; the run is
// kept in LDS, where LANES lanes per token look for its extremes.  (One thread per token, each of
// its logits a strided load and store, took 17.5 us for 8192 tokens of 24 logits; eight lanes 6.3.)
constexpr int kLogitThreads = 256;
template <int LANES>
__global__ __launch_bounds__(kLogitThreads) void logits_kernel(
    const float *__restrict__ u_raw, const float *__restrict__ sumsq, int parts, int wide,
    const float *__restrict__ b, const float *__restrict__ alpha, int nC, float eps, int64_t T,
    int M, int R, int n, float *__restrict__ z, float *__restrict__ spread) {
  constexpr int kLogitTok = kLogitThreads / LANES;
  extern __shared__ float z_s[];   // [kLogitTok][M | 1]
  __shared__ float r_s[kLogitTok];
  const int ld = M | 1;
  const int64_t t0 = static_cast<int64_t>(blockIdx.x) * kLogitTok;
  const int live = T - t0 < kLogitTok ? static_cast<int>(T - t0) : kLogitTok;
  if (static_cast<int>(threadIdx.x) < live) {
    const float ssq = slice_sum(sumsq, parts, wide, T, t0 + threadIdx.x);
    r_s[threadIdx.x] = rms_factor(ssq, nC, eps);
  }
  const float a0 = alpha[0], a1 = alpha[1], a2 = alpha[2];
  __syncthreads();
#pragma unroll 4
  for (int e = threadIdx.x; e < live * M; e += kLogitThreads) {
    const int tk = e / M, m = e - tk * M;
    const float u = slice_sum(u_raw, parts, wide, T * M, t0 * M + e);
    const float al = m < R ? a0 : (m < R + n ? a1 : a2);
    const float v = logit_of(al, r_s[tk], u, b[m]);
    if (z) z[t0 * M + e] = v;
    z_s[tk * ld + m] = v;
  }
  if (spread == nullptr) return;
  __syncthreads();
  const int tk = threadIdx.x / LANES, l = threadIdx.x % LANES;
  float zmax = -INFINITY, zmin = INFINITY;
  if (tk < live) {
    for (int m = l; m < R; m += LANES) {
      zmax = fmaxf(zmax, z_s[tk * ld + m]);
      zmin = fminf(zmin, z_s[tk * ld + m]);
    }
  }
#pragma unroll
  for (int off = 1; off < LANES; off <<= 1) {
    zmax = fmaxf(zmax, __shfl_xor(zmax, off, 64));
    zmin = fminf(zmin, __shfl_xor(zmin, off, 64));
  }
  if (l == 0 && tk < live) spread[t0 + tk] = zmax - zmin;
}

template <int N>
__device__ __forceinline__ float l1_error(const float (&Q)[N * N], float (&cs)[N]) {
  float e = 0.f;
#pragma unroll
  for (int i = 0; i < N; ++i) {
    float s = 0.f;
#pragma unroll
    for (int j = 0; j < N; ++j) s += Q[i * N + j];
    e += fabsf(s - 1.f);
  }
#pragma unroll
  for (int j = 0; j < N; ++j) {
    float s = 0.f;
#pragma unroll
    for (int i = 0; i < N; ++i) s += Q[i * N + j];
    cs[j] = s;
    e += fabsf(s - 1.f);
  }
  return e;
}

// Q_l = H_l Q_{l-1}, Q_0 = I: later layers multiply on the left, the order in
// which Eq. 1 applies them.
// (Bound by the chain of loads of few waves: blocks of one wave spread over all compute units, six layers of 8192 tokens, H from the caches, us
// with 128 / 64 threads: n = 4 5.5 / 5.2, n = 8 16.6 / 15.6. AHEAD: a layer's matrix is requested while the one before is multiplied;
// see launch_ds_chain.)
constexpr int kChainThreads = 64;
template <int N, bool AHEAD>
__global__ __launch_bounds__(kChainThreads) void ds_chain_kernel(
    const float *__restrict__ H, int L, int64_t T, float *__restrict__ colsum,
    float *__restrict__ l1, float *__restrict__ prod, float *__restrict__ prod_colsum,
    float *__restrict__ prod_l1) {
  const int64_t t = static_cast<int64_t>(blockIdx.x) * kChainThreads + threadIdx.x;
  if (t >= T) return;
  float Q[N * N], Hl[N * N], Qn[N * N], cs[N];
  [[maybe_unused]] float next[AHEAD ? N * N : 1];
  auto fetch = [&](int l, float *to) {
#pragma unroll
    for (int e = 0; e < N * N; ++e) to[e] = H[(static_cast<int64_t>(l) * T + t) * (N * N) + e];
  };
  if constexpr (AHEAD) fetch(0, next);
#pragma unroll
  for (int e = 0; e < N * N; ++e) Q[e] = (e / N == e % N) ? 1.f : 0.f;
  for (int l = 0; l < L; ++l) {
    const int64_t lt = static_cast<int64_t>(l) * T + t;
    if constexpr (AHEAD) {
#pragma unroll
      for (int e = 0; e < N * N; ++e) Hl[e] = next[e];
      if (l + 1 < L) fetch(l + 1, next);
    } else {
      fetch(l, Hl);
    }
    const float e1 = l1_error<N>(Hl, cs);
    if (l1) l1[lt] = e1;
    if (colsum) {
#pragma unroll
      for (int j = 0; j < N; ++j) colsum[lt * N + j] = cs[j];
    }
#pragma unroll
    for (int i = 0; i < N; ++i)
#pragma unroll
      for (int j = 0; j < N; ++j) {
        float s = 0.f;
#pragma unroll
        for (int k = 0; k < N; ++k) s += Hl[i * N + k] * Q[k * N + j];
        Qn[i * N + j] = s;
      }
#pragma unroll
    for (int e = 0; e < N * N; ++e) Q[e] = Qn[e];
    const float e2 = l1_error<N>(Q, cs);
    if (prod_l1) prod_l1[lt] = e2;
    if (prod_colsum) {
#pragma unroll
      for (int j = 0; j < N; ++j) prod_colsum[lt * N + j] = cs[j];
    }
  }
  if (prod) {
#pragma unroll
    for (int e = 0; e < N * N; ++e) prod[t * N * N + e] = Q[e];
  }
}

}  // namespace

hipError_t launch_logits(const mhcl_desc &d, int M, const RawSums &raw, const float *b,
                         const float *alpha, float *z, float *spread, hipStream_t s) {
  // A thread adds the slices of its logits one after the other; where that is a long chain they are added
  // before (mhcl_logits, f32, C = 1024, n = 4, 128 tokens 28.0 / 15.0 us; 3 logits, n = 1, 10.0 / 12.4).
  RawSums r = raw;
  if (raw.wide && (d.T < 32 ? d.T : 32) * M * raw.parts > 24 * kLogitThreads) {
    hipError_t e = add_wide_slices(d, r, s);
    if (e != hipSuccess) return e;
  }
  auto go = [&](auto lanes) {
    constexpr int L = decltype(lanes)::value, kTok = kLogitThreads / L;
    hipLaunchKernelGGL(logits_kernel<L>, dim3(static_cast<unsigned>((d.T + kTok - 1) / kTok)),
                       dim3(kLogitThreads), kTok * (M | 1) * sizeof(float), s, r.u_raw, r.sumsq, r.parts, r.wide, b,
                       alpha, d.n * d.C, d.eps, d.T, M, M - 2 * d.n, d.n, z, spread);
    return hipGetLastError();
  };
  // few logits of many tokens leave seven of eight lanes idle at the extremes (mhcl_logits at C = 64,
  // eight / one: M = 3, 262144 tokens 22.7 / 17.4 us; M = 15 35.6 / 32.6, 65536 tokens 13.2 / 15.8)
  return M <= 16 && d.T >= 131072 ? go(std::integral_constant<int, 1>{}) : go(std::integral_constant<int, 8>{});
}

hipError_t launch_ds_chain(int n, int L, int64_t T, const float *H, float *colsum, float *l1,
                           float *prod, float *prod_colsum, float *prod_l1, hipStream_t s) {
  auto go = [&](auto nn) {
    constexpr int N = decltype(nn)::value;
    // Up to two waves a compute unit (us without / with, H not from the caches: six layers of 8192 tokens n = 2 6.9 / 6.3, n = 4 9.3 / 8.6, n = 8
    // 24.5 / 23.1, 32768 tokens n = 4 15.2 / 14.8, n = 8 35.6 / 34.2). More waves hide the loads by themselves, and then the second
    // matrix's registers cost: 65536 tokens n = 4 18.7 / 19.0, n = 8 54.9 / 57.4, one layer 20.4 / 22.8.
    const auto kern = T <= 2 * 256 * kChainThreads ? ds_chain_kernel<N, true> : ds_chain_kernel<N, false>;
    hipLaunchKernelGGL(kern, dim3(static_cast<unsigned>((T + kChainThreads - 1) / kChainThreads)), dim3(kChainThreads), 0, s, H, L, T,
                       colsum, l1, prod, prod_colsum, prod_l1);
    return hipGetLastError();
  };
  switch (n) {
    case 1: return go(std::integral_constant<int, 1>{});
    case 2: return go(std::integral_constant<int, 2>{});
    case 3: return go(std::integral_constant<int, 3>{});
    case 4: return go(std::integral_constant<int, 4>{});
    case 5: return go(std::integral_constant<int, 5>{});
    case 6: return go(std::integral_constant<int, 6>{});
    case 7: return go(std::integral_constant<int, 7>{});
    case 8: return go(std::integral_constant<int, 8>{});
  }
  return hipErrorInvalidValue;
}

}  // namespace mhcl
