// The pre-aggregate h = H_pre x as one role of a launch whose other blocks compute the coefficients.
#pragma once
#include "mhcl_common.h"

namespace mhcl {

// What the blocks of the pre-aggregate read besides the projection's slices.
struct PreArgs {
  const void *x;
  void *h;
  unsigned first;   // blocks before this one have the launch's other role
  int C;
};

// Block `block` takes THREADS consecutive 16-byte chunks of h.  H_pre needs N logits and the sum of
// squares of each of the few tokens they lie in, none of the softmax or the iteration behind H_res, so the
// block adds those from the projection's slices itself (in the order of the per-token stage) while its x is
// on its way, and need not wait for the stage.
template <typename IO, int N, int THREADS>
__device__ __forceinline__ void pre_from_slices(const PreArgs &p, unsigned block, const float *u_raw,
                                                const float *sumsq, int parts, int wide, const float *b,
                                                const float *alpha, float eps, int64_t T, int R) {
  constexpr int V = IO::kVec;
  __shared__ float gate_s[(THREADS + 1) * N];   // (a row of C is one chunk at least)
  __shared__ double stage_s[THREADS];
  const int vpr = p.C / V, M = R + 2 * N, nC = N * p.C;
  const int64_t e0 = static_cast<int64_t>(block) * THREADS, t0 = e0 / vpr;
  const int rem = static_cast<int>(e0 - t0 * vpr);
  const unsigned at = static_cast<unsigned>(rem) + threadIdx.x;
  const int tok = static_cast<int>(at / static_cast<unsigned>(vpr));
  const int c = static_cast<int>(at - static_cast<unsigned>(tok) * vpr) * V;
  const bool live = t0 + tok < T;
  const int64_t t = live ? t0 + tok : T - 1;
  int tokens = static_cast<int>((static_cast<unsigned>(rem) + THREADS - 1) / static_cast<unsigned>(vpr)) + 1;
  if (tokens > T - t0) tokens = static_cast<int>(T - t0);
  // (the parameters of a thread's first gate ahead of everything else)
  const float alpha_pre = alpha[1], b_first = b[R + static_cast<int>(threadIdx.x) % N];
  auto gate = [&](int i, float u, float ssq) {
    const float bias = i < THREADS ? b_first : b[R + i % N];
    gate_s[i] = sigmoidf(logit_of(alpha_pre, rms_factor(ssq, nC, eps), u, bias));
  };
  float v[N][V];
  auto load_x = [&]() {
#pragma unroll
    for (int j = 0; j < N; ++j) IO::load(p.x, (t * N + j) * p.C + c, v[j]);
  };
  // [token][slice][gates | sum of squares]: one by each thread, ahead of x (loads return in order); a thread that
  // walks the slices of a gate pays a round trip every few of them (n = 4, C = 2048, 1000 tokens: 7 us)
  const int per = parts * (N + 1), all = tokens * per;
  if (all <= THREADS) {
    const int i = static_cast<int>(threadIdx.x) < all ? threadIdx.x : all - 1;
    const int k = i / per, rest = i - k * per, pt = rest / (N + 1), j = rest - pt * (N + 1);
    const int64_t tt = pt * T + t0 + k;
    const float *src = j < N ? u_raw : sumsq;
    const int64_t from = j < N ? tt * M + R + j : tt;
    double s;
    if (wide) s = reinterpret_cast<const double *>(src)[from];
    else s = src[from];
    load_x();
    __builtin_amdgcn_sched_barrier(0);
    stage_s[threadIdx.x] = s;
    __syncthreads();
    for (int i = threadIdx.x; i < tokens * N; i += THREADS) {
      const double *s = stage_s + (i / N) * per;
      if (wide) {
        double u = s[i % N], ssq = s[N];
        for (int k = 1; k < parts; ++k) { u += s[k * (N + 1) + i % N]; ssq += s[k * (N + 1) + N]; }
        gate(i, static_cast<float>(u), static_cast<float>(ssq));
      } else {
        float u = static_cast<float>(s[i % N]), ssq = static_cast<float>(s[N]);
        for (int k = 1; k < parts; ++k) {
          u += static_cast<float>(s[k * (N + 1) + i % N]);
          ssq += static_cast<float>(s[k * (N + 1) + N]);
        }
        gate(i, u, ssq);
      }
    }
  } else {
    load_x();
    for (int i = threadIdx.x; i < tokens * N; i += THREADS) {
      const int64_t t = t0 + i / N;
      gate(i, slice_sum(u_raw, parts, wide, T * M, t * M + R + i % N), slice_sum(sumsq, parts, wide, T, t));
    }
  }
  __syncthreads();
  if (!live) return;
  float acc[V];
#pragma unroll
  for (int e = 0; e < V; ++e) acc[e] = 0.f;
#pragma unroll
  for (int j = 0; j < N; ++j) {
    const float w = gate_s[tok * N + j];
#pragma unroll
    for (int e = 0; e < V; ++e) acc[e] = fmaf(w, v[j][e], acc[e]);   // (as pre_kernel)
  }
  IO::store(p.h, t * p.C + c, acc);
}

inline int64_t pre_chunks(const mhcl_desc &d) {
  return d.T * (d.C / (d.io_dtype == MHCL_BF16 ? BF16::kVec : F32::kVec));
}
inline unsigned pre_blocks(const mhcl_desc &d, int threads) {
  return static_cast<unsigned>((pre_chunks(d) + threads - 1) / threads);
}

}  // namespace mhcl
