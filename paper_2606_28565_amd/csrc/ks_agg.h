// Per-step request sums, for the kernels that form them.
#pragma once

#include <hip/hip_runtime.h>

#include "ks_internal.h"

namespace ks {

constexpr int kAggLanes = 16;

// Per step j: over its requests r, Q = sum q, KV = sum (h + q),
// PAIRS = sum (q h + q (q + 1) / 2), TILES = sum ceil(q / 128).  A group of
// 16 lanes per step strides over its requests, then a butterfly reduction
// within the group.
// thread: the caller's thread of `threads` (whole waves).
__device__ __forceinline__ void attn_agg(const uint32_t *__restrict__ req_off, const uint32_t *__restrict__ rq,
                                         const uint32_t *__restrict__ rh, int64_t n_steps, int64_t n_req,
                                         uint64_t *__restrict__ agg, uint32_t *err, int64_t thread, int64_t threads) {
  const int sub = (int)(thread & (kAggLanes - 1));
  const int64_t groups = threads / kAggLanes;
  for (int64_t j = thread / kAggLanes; j < n_steps; j += groups) {
    uint32_t r0 = req_off[j], r1 = req_off[j + 1];
    if (r0 > r1 || (int64_t)r1 > n_req) {
      if (sub == 0) atomicOr(err, kErrReq);
      r0 = r1 = 0;
    }
    uint64_t Q = 0, KV = 0, P = 0, T = 0;
    for (uint32_t r = r0 + sub; r < r1; r += kAggLanes) {
      const uint64_t q = rq[r], h = rh[r];
      Q += q;
      KV += h + q;
      P += q * h + ((q * (q + 1)) >> 1);
      T += (q + 127) >> 7;
    }
#pragma unroll
    for (int off = kAggLanes / 2; off > 0; off >>= 1) {
      Q += __shfl_xor(Q, off);
      KV += __shfl_xor(KV, off);
      P += __shfl_xor(P, off);
      T += __shfl_xor(T, off);
    }
    if (sub == 0) {
      agg[j] = Q;
      agg[n_steps + j] = KV;
      agg[2 * n_steps + j] = P;
      agg[3 * n_steps + j] = T;
    }
  }
}

}  // namespace ks
