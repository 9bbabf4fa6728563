// InfoNCE over one row of MaxSim scores, by one workgroup: shared by the loss's own kernel and by the
// total loss's, which runs it beside the pooling.
#pragma once

#include "common.h"

namespace hpr {

constexpr int kRowThreads = 256;
constexpr int kRowCache = 8;  // scores per thread kept in registers by infonce_row

// Deterministic 256-thread block reductions (fixed tree: wave butterfly, then waves in order).
__device__ __forceinline__ float block_sum(float v, float* red) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  v = wave_sum(v);
  __syncthreads();
  if (lane == 0) red[wave] = v;
  __syncthreads();
  return (red[0] + red[1]) + (red[2] + red[3]);
}

__device__ __forceinline__ void block_argmax(float& M, int64_t& dM, float* redf, int64_t* redi) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
  for (int m = 32; m >= 1; m >>= 1) {
    const float oM = __shfl_xor(M, m);
    const int64_t od = __shfl_xor(dM, m);
    if (oM > M || (oM == M && od < dM)) {
      M = oM;
      dM = od;
    }
  }
  __syncthreads();
  if (lane == 0) {
    redf[wave] = M;
    redi[wave] = dM;
  }
  __syncthreads();
  M = redf[0];
  dM = redi[0];
  for (int w = 1; w < kRowThreads / kWave; ++w)
    if (redf[w] > M || (redf[w] == M && redi[w] < dM)) {
      M = redf[w];
      dM = redi[w];
    }
}

// One workgroup of kRowThreads threads per query row q: G[q, :] and the row's loss term; the last
// workgroup to finish reduces the terms in query order into the mean.  ctrl[0] = error flag raised
// by earlier kernels of the call, ctrl[1] = completion counter (both zeroed at the start of the
// call).
__device__ __forceinline__ void infonce_row(const float* __restrict__ S, int nq, int64_t n,
                                            const int32_t* pos, float s, float gw, float* G,
                                            float* terms, float* loss, float* scores_out,
                                            int32_t* ctrl, int q) {
  // No FMA contraction in this function: every logit must be the same rounded product s * S.
  // Contracted, M - s * S[pos] becomes fma(-s, S[pos], M), the rounding error of M's own
  // product (up to half an ulp of ~1e3 when s = 50) instead of exactly 0 when the positive
  // holds the maximum -- larger than the whole loss in that regime.
#pragma clang fp contract(off)
  __shared__ float redf[kRowThreads / kWave];
  __shared__ int64_t redi[kRowThreads / kWave];
  __shared__ int last;
  const int tid = threadIdx.x;
  const float* Sq = S + (int64_t)q * n;
  float* Gq = G + (int64_t)q * n;
  const float gscale = gw * s / (float)nq;  // gw: the loss's weight in a weighted sum

  // The row's first kRowCache * kRowThreads scores stay in registers for the three passes
  // (each later pass would otherwise be another round trip to L2); the rest are re-read.
  float sv[kRowCache];
#pragma unroll
  for (int c = 0; c < kRowCache; ++c) {
    const int64_t d = tid + (int64_t)c * kRowThreads;
    sv[c] = d < n ? Sq[d] : 0.f;
  }
  // f(d, S[q, d]) for this thread's d in increasing order (static register indices first)
  auto each = [&](auto f) {
#pragma unroll
    for (int c = 0; c < kRowCache; ++c) {
      const int64_t d = tid + (int64_t)c * kRowThreads;
      if (d < n) f(d, sv[c]);
    }
    for (int64_t d = tid + (int64_t)kRowCache * kRowThreads; d < n; d += kRowThreads) f(d, Sq[d]);
  };
  float M = -__builtin_huge_valf();
  int64_t dM = n;
  each([&](int64_t d, float sd) {
    const float l = (s * sd);
    if (l > M) {
      M = l;
      dM = d;
    }
  });
  block_argmax(M, dM, redf, redi);
  // log-sum-exp = M + log1p(sum over d != dM of exp(l - M)): keeps the loss accurate when one
  // logit dominates (the loss is then ~ the small sum, which log(1 + x) would lose).
  float so = 0.f;
  each([&](int64_t d, float sd) {
    if (d != dM) so += expf((s * sd) - M);
  });
  so = block_sum(so, redf);
  const float l1p = log1pf(so);
  const float lse = M + l1p;
  const int64_t p = pos[q];
  const bool bad = p < 0 || p >= n;
  float term = 0.f;
  if (bad) {
    each([&](int64_t d, float sd) {
      if (scores_out) scores_out[(int64_t)q * n + d] = sd;
      Gq[d] = 0.f;
    });
    if (tid == 0) atomicOr(&ctrl[0], 2);
  } else {
    term = (M - (s * Sq[p])) + l1p;
    // G[q,d] = (s/B) softmax; the positive gets -(s/B) * (sum of the other probabilities),
    // which equals (s/B) (p_pos - 1) without the cancellation of 1 - p_pos in fp32.
    float rest = 0.f;
    each([&](int64_t d, float sd) {
      if (scores_out) scores_out[(int64_t)q * n + d] = sd;
      if (d != p) {
        const float e = expf((s * sd) - lse);
        Gq[d] = gscale * e;
        rest += e;
      }
    });
    rest = block_sum(rest, redf);
    if (tid == 0) Gq[p] = -gscale * rest;
  }
  if (tid == 0) {
    terms[q] = term;
    __threadfence();
    last = atomicAdd(&ctrl[1], 1) == nq - 1;
  }
  __syncthreads();
  if (!last) return;
  __threadfence();
  float acc = 0.f;  // fixed order: thread t sums queries t, t + 256, ...; then a fixed tree
  for (int qq = tid; qq < nq; qq += kRowThreads)
    acc += __hip_atomic_load(&terms[qq], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  acc = block_sum(acc, redf);
  if (tid == 0) {
    *loss = ctrl[0] != 0 ? __builtin_nanf("") : acc / (float)nq;
    ctrl[1] = 0;
  }
}

}  // namespace hpr
