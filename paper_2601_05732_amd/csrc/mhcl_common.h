// Shared device-side building blocks of libmhcl (gfx950 only).
//
//  * stream element traits (bf16 / f32) and 16-byte vector access
//  * the permutation table of Theorem 3.1, generated at compile time
//  * the logistic function and wave sums
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <utility>

#include "../../include/mhcl.h"

namespace mhcl {

constexpr int kMaxN = 5;          // full permutation form and Sinkhorn-Knopp form
constexpr int kMaxNSubset = 8;    // permutation-subset form
constexpr int kMaxPerm = 128;     // permutations in a subset
constexpr int kMaxSkIters = 32;

// ------------------------------------------------------------------ bf16
__device__ __forceinline__ float bf16_to_f32(uint16_t b) {
  return __uint_as_float(static_cast<uint32_t>(b) << 16);
}
// Round to nearest, ties to even; NaN stays NaN: v_cvt_pk_bf16_f32, the same bits as seven integer instructions a value
// (us with those / this: mhcl_fwd_coeffs_pre with mhcl_post, n = 4, C = 2048, 32768 tokens 375 / 365; the separable step at C = 1024,
// 5003 tokens 155 / 149; the packing of W at n = 4, C = 4096 7.8 / 4.5).
__device__ __forceinline__ uint16_t f32_to_bf16(float f) {
  return __builtin_bit_cast(uint16_t, static_cast<__bf16>(f));
}
__device__ __forceinline__ float bf16lo(uint32_t p) { return __uint_as_float(p << 16); }
__device__ __forceinline__ float bf16hi(uint32_t p) { return __uint_as_float(p & 0xffff0000u); }
__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
  typedef __bf16 pair __attribute__((ext_vector_type(2)));
  return __builtin_bit_cast(uint32_t, pair{static_cast<__bf16>(lo), static_cast<__bf16>(hi)});
}

// w = hi + lo up to 2^-17 of its size
__device__ __forceinline__ void split_bf16(float w, uint16_t &hi, uint16_t &lo) {
  hi = f32_to_bf16(w);
  lo = f32_to_bf16(w - bf16_to_f32(hi));
}

// A 16-byte chunk of a stream tensor held as fp32 lanes. load_once and store_once are for data that is not soon read again:
// the chunk does not displace what is (nt bit of the load or store).
typedef uint32_t chunk16 __attribute__((ext_vector_type(4)));
struct BF16 {
  static constexpr int kVec = 8;      // elements per 16 bytes
  __device__ static __forceinline__ void load(const void *p, size_t elem, float (&v)[8]) {
    const uint4 q = *reinterpret_cast<const uint4 *>(static_cast<const uint16_t *>(p) + elem);
    v[0] = bf16lo(q.x); v[1] = bf16hi(q.x); v[2] = bf16lo(q.y); v[3] = bf16hi(q.y);
    v[4] = bf16lo(q.z); v[5] = bf16hi(q.z); v[6] = bf16lo(q.w); v[7] = bf16hi(q.w);
  }
  __device__ static __forceinline__ void store(void *p, size_t elem, const float (&v)[8]) {
    uint4 q;
    q.x = pack_bf16x2(v[0], v[1]); q.y = pack_bf16x2(v[2], v[3]);
    q.z = pack_bf16x2(v[4], v[5]); q.w = pack_bf16x2(v[6], v[7]);
    *reinterpret_cast<uint4 *>(static_cast<uint16_t *>(p) + elem) = q;
  }
  __device__ static __forceinline__ void load_once(const void *p, size_t elem, float (&v)[8]) {
    const chunk16 q = __builtin_nontemporal_load(reinterpret_cast<const chunk16 *>(static_cast<const uint16_t *>(p) + elem));
    v[0] = bf16lo(q.x); v[1] = bf16hi(q.x); v[2] = bf16lo(q.y); v[3] = bf16hi(q.y);
    v[4] = bf16lo(q.z); v[5] = bf16hi(q.z); v[6] = bf16lo(q.w); v[7] = bf16hi(q.w);
  }
  __device__ static __forceinline__ void store_once(void *p, size_t elem, const float (&v)[8]) {
    const chunk16 q = {pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3]), pack_bf16x2(v[4], v[5]), pack_bf16x2(v[6], v[7])};
    __builtin_nontemporal_store(q, reinterpret_cast<chunk16 *>(static_cast<uint16_t *>(p) + elem));
  }
};
struct F32 {
  static constexpr int kVec = 4;
  __device__ static __forceinline__ void load(const void *p, size_t elem, float (&v)[4]) {
    const float4 q = *reinterpret_cast<const float4 *>(static_cast<const float *>(p) + elem);
    v[0] = q.x; v[1] = q.y; v[2] = q.z; v[3] = q.w;
  }
  __device__ static __forceinline__ void store(void *p, size_t elem, const float (&v)[4]) {
    *reinterpret_cast<float4 *>(static_cast<float *>(p) + elem) = make_float4(v[0], v[1], v[2], v[3]);
  }
  __device__ static __forceinline__ void load_once(const void *p, size_t elem, float (&v)[4]) {
    const chunk16 q = __builtin_nontemporal_load(reinterpret_cast<const chunk16 *>(static_cast<const float *>(p) + elem));
    v[0] = __uint_as_float(q.x); v[1] = __uint_as_float(q.y); v[2] = __uint_as_float(q.z); v[3] = __uint_as_float(q.w);
  }
  __device__ static __forceinline__ void store_once(void *p, size_t elem, const float (&v)[4]) {
    const chunk16 q = {__float_as_uint(v[0]), __float_as_uint(v[1]), __float_as_uint(v[2]), __float_as_uint(v[3])};
    __builtin_nontemporal_store(q, reinterpret_cast<chunk16 *>(static_cast<float *>(p) + elem));
  }
};

// ------------------------------------------------- host: run-time values as types
template <typename F>
inline hipError_t dispatch_n(int n, F &&f) {
  switch (n) {
    case 1: return f(std::integral_constant<int, 1>{});
    case 2: return f(std::integral_constant<int, 2>{});
    case 3: return f(std::integral_constant<int, 3>{});
    case 4: return f(std::integral_constant<int, 4>{});
    case 5: return f(std::integral_constant<int, 5>{});
    case 6: return f(std::integral_constant<int, 6>{});
    case 7: return f(std::integral_constant<int, 7>{});
    case 8: return f(std::integral_constant<int, 8>{});
  }
  return hipErrorInvalidValue;
}
template <typename F>
inline hipError_t dispatch_io(int io, F &&f) {
  if (io == MHCL_BF16) return f(BF16{});
  return f(F32{});
}

// ------------------------------------------------- permutation table
constexpr int factorial(int n) { return n <= 1 ? 1 : n * factorial(n - 1); }

template <int N>
struct PermTab {
  signed char s[factorial(N)][N];
};

// k-th permutation in lexicographic order by unranking k in the factorial
// number system: digit i selects the d-th smallest value not yet used.
template <int N>
constexpr PermTab<N> make_perm_tab() {
  PermTab<N> t{};
  for (int k = 0; k < factorial(N); ++k) {
    bool used[N] = {};
    int rem = k;
    for (int i = 0; i < N; ++i) {
      const int f = factorial(N - 1 - i);
      const int d = rem / f;
      rem %= f;
      int seen = 0;
      for (int j = 0; j < N; ++j) {
        if (used[j]) continue;
        if (seen == d) { t.s[k][i] = static_cast<signed char>(j); used[j] = true; break; }
        ++seen;
      }
    }
  }
  return t;
}

template <int N>
struct Perm {
  static constexpr PermTab<N> tab = make_perm_tab<N>();
};
// ------------------------------------------------- per-token coefficients
template <int N, int MODE>
struct Dims {
  static constexpr int R = (MODE == MHCL_RES_LITE) ? factorial(N) : N * N;   // residual logits
  static constexpr int M = R + 2 * N;                                         // all logits
};

__device__ __forceinline__ float sigmoidf(float t) { return 1.f / (1.f + expf(-t)); }

// RMSNorm's factor of a token and a logit from its projection u.  Several kernels compute the same ones (the gates of
// h are computed apart from those handed out where one launch takes both) and must get the same bits: which product
// is fused with which sum is fixed here and not left to each kernel's compilation.
__device__ __forceinline__ float rms_factor(float sumsq, int nC, float eps) {
  return 1.f / sqrtf(sumsq / static_cast<float>(nC) + eps);
}
__device__ __forceinline__ float logit_of(float alpha, float r, float u, float b) { return fmaf(alpha, r * u, b); }

// ------------------------------------------------- sums in a fixed order
// a + b, of two lanes' values: never fused with a product that a lane's own value is.  (Fused, either lane adds
// its unrounded product to the other's rounded one, and the lanes get different sums.)
__device__ __forceinline__ float lane_add(float a, float b) {
#pragma clang fp contract(off)
  return a + b;
}

// sum of `v` over the 64 lanes of a wave, in every lane
__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}

// at(first) + ... + at(first + CNT - 1), CNT a power of two, added pairwise: log2 CNT roundings per
// term (one after the other, the sum of g_z over a block's tokens had 1.7 times the error)
template <int CNT, typename F>
__device__ __forceinline__ float pairwise_sum(F at, int first = 0) {
  if constexpr (CNT == 1) {
    return at(first);
  } else {
    const float lo = pairwise_sum<CNT / 2>(at, first), hi = pairwise_sum<CNT / 2>(at, first + CNT / 2);
    return lo + hi;
  }
}

// src[at] + src[at + stride] + ..., one element of each slice, in order; in fp64 and rounded once if the
// slices are fp64 (`wide`)
__device__ __forceinline__ float slice_sum(const float *src, int slices, int wide, int64_t stride, int64_t at) {
  if (wide) {
    const double *p = reinterpret_cast<const double *>(src);
    double s = p[at];
#pragma unroll 4
    for (int k = 1; k < slices; ++k) s += p[k * stride + at];
    return static_cast<float>(s);
  }
  float s = src[at];
#pragma unroll 4
  for (int k = 1; k < slices; ++k) s += src[k * stride + at];
  return s;
}

// Columns of the [count, ld] matrix of g_z sums per 32 or 64 tokens, which add up to g_b and g_alpha.
struct ColumnArgs {
  const float *rows;
  int64_t count;
  float *g_b, *g_alpha;
};
// Column c, by a block's first 256 threads in a fixed order (thread i takes rows i, i + 256, ... in turn, then a
// pairwise tree over the threads, in red[256]); columns below M go to g_b, the others to g_alpha.
__device__ __forceinline__ void column_sum(const ColumnArgs &p, int ld, int c, int M, float *red) {
  const int tid = threadIdx.x;
  float s = 0.f;
  if (tid < 256) {
#pragma unroll 4
    for (int64_t r = tid; r < p.count; r += 256) s += p.rows[r * ld + c];
    red[tid] = s;
  }
  __syncthreads();
#pragma unroll
  for (int w = 128; w > 0; w >>= 1) {
    if (tid < w) red[tid] += red[tid + w];
    __syncthreads();
  }
  if (tid == 0) {
    if (c < M) p.g_b[c] = red[0];
    else p.g_alpha[c - M] = red[0];
  }
}

// ------------------------------------------------- host: blocks of one token
// as many waves as a row of C has 16-byte pieces for, at most four
inline int waves_that_fit(int C, int vec) {
  const int pieces = C / vec;
  return pieces <= 64 ? 1 : (pieces <= 128 ? 2 : (pieces <= 192 ? 3 : 4));
}

}  // namespace mhcl
