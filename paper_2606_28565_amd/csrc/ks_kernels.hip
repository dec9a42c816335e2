// HIP kernels of the batched kernel-latency evaluator, written for gfx950
// (CDNA4: wave64, MFMA, 160 KB LDS per CU).
//
// Data flow of one evaluation (all on the caller's stream):
//   k_clear      reset the workspace's bad-data flag and step-range table,
//                then form the per-spec constants (k_spec_prep instead for
//                more than 1024 specs)
//   k_attn_agg   per step: Q, KV, PAIRS, TILES of its request list (Sec. 5.8)
//   k_eval<K>    per wave: 64 records of one family x every spec vector:
//                exact counts (Eq. 1-2 operands), waves and u (Sec. 2.2),
//                t_roof (Eq. 2), features and the family's efficiency head
//                on MFMA (Sec. 5.3), t = max(t_roof eta, t0) (Eq. 2), a
//                wavefront segmented sum of t by step, and each (family,
//                step) record range
//   k_stream     instead of k_eval for every call with no MLP family and
//                no measured grid (eta = 1, the bounded head): the same per
//                256 records and wave, four consecutive records per lane
//   k_finish     per (spec, step): body sum, all-reduce (Eq. 3), assembly (Eq. 4)
// k_prologue is the first two for a call of few steps.  Calls with an MLP head
// and enough head work find their different records first (k_unique, k_join)
// and evaluate those (k_eval's kVarUniq); their sums are k_finish_few's or
// k_finish_list's, their per-pair outputs k_spread's and k_counts'.
#include <hip/hip_runtime.h>

#include <atomic>
#include <utility>

#include "ks_agg.h"
#include "ks_internal.h"

namespace ks {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef short s16x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr uint32_t kNoKey = 0xFFFFFFFFu;

// ------------------------------------------------------------------ helpers
__device__ __forceinline__ float rcpf(float x) { return __builtin_amdgcn_rcpf(x); }
__device__ __forceinline__ float log2f_fast(float x) { return __builtin_amdgcn_logf(x); }

// ceil(x / d) for x + d < 2^52, through a float64 reciprocal and one
// correction step each way (the product's error is below one unit there).
__device__ __forceinline__ uint64_t ceil_div(uint64_t x, uint32_t d, double rcp_d) {
  const uint64_t y = x + d - 1;
  uint64_t q = (uint64_t)((double)y * rcp_d);
  if (q * d > y) q -= 1;
  else if ((q + 1) * d <= y) q += 1;
  return q;
}

// two floats -> packed bfloat16 pair, round to nearest even
__device__ __forceinline__ uint32_t pack_bf16(float lo, float hi) {
  f32x2 v = {lo, hi};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}

// relu on an fp32 value through its bits: a negative float is a negative
// int32 (one integer max, no canonicalization of the input)
__device__ __forceinline__ float relu_f(float x) {
  return __builtin_bit_cast(float, max(__builtin_bit_cast(int, x), 0));
}

// relu on a packed bfloat16 pair: a negative bf16 is a negative int16
__device__ __forceinline__ uint32_t relu_bf16x2(uint32_t v) {
  s16x2 s = __builtin_bit_cast(s16x2, v);
  s16x2 z = {0, 0};
  return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(s, z));
}

__device__ __forceinline__ float bf16_to_f32(uint32_t bits16) {
  return __builtin_bit_cast(float, bits16 << 16);
}

// Exchange lanes 32..63 of `lo` with lanes 0..31 of `hi`.
__device__ __forceinline__ void swap32(uint32_t &lo, uint32_t &hi) {
  auto r = __builtin_amdgcn_permlane32_swap(lo, hi, false, false);
  lo = r[0];
  hi = r[1];
}

// ------------------------------------------------------------ clear / agg
// Reset the flag word and, when step sums are wanted, the per-(family,
// step) range table (an empty range marks a family without that step).
__device__ void spec_prep_one(const ks_spec *__restrict__ specs, int s, SpecC *__restrict__ out, uint32_t *err);

#if KS_HEADS == 0
// With specs (n_specs > 0), the first workgroup also forms their constants
// once the flag word is reset (a bad spec then flags the fresh word).
__global__ void k_clear(uint32_t *err, uint32_t *range, int64_t n_range, const ks_spec *specs, int32_t n_specs,
                        SpecC *specc) {
  const int64_t i0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (blockIdx.x == 0) {
    if (threadIdx.x == 0) err[0] = 0;
    if (n_specs > 0) {
      __syncthreads();
      for (int s = threadIdx.x; s < n_specs; s += blockDim.x) spec_prep_one(specs, s, specc, err);
    }
  }
  for (int64_t i = i0; i < n_range; i += (int64_t)gridDim.x * blockDim.x) range[i] = 0;
}

// Both for a call of few steps, in one workgroup: the flag reset, then the range
// table, the spec constants and the request sums (one launch instead of two,
// 3.0 us instead of 3.6 and a launch for one serving step).
constexpr int kPrologueThreads = 1024;

__global__ __launch_bounds__(kPrologueThreads) void k_prologue(uint32_t *err, uint32_t *range, int64_t n_range,
                                                               const ks_spec *specs, int32_t n_specs, SpecC *specc,
                                                               const uint32_t *req_off, const uint32_t *rq,
                                                               const uint32_t *rh, int64_t n_steps, int64_t n_req,
                                                               uint64_t *agg) {
  if (threadIdx.x == 0) err[0] = 0;
  __syncthreads();
  for (int64_t i = threadIdx.x; i < n_range; i += kPrologueThreads) range[i] = 0;
  for (int s = threadIdx.x; s < n_specs; s += kPrologueThreads) spec_prep_one(specs, s, specc, err);
  attn_agg(req_off, rq, rh, n_steps, n_req, agg, err, threadIdx.x, kPrologueThreads);
}

__global__ void k_attn_agg(const uint32_t *__restrict__ req_off, const uint32_t *__restrict__ rq,
                           const uint32_t *__restrict__ rh, int64_t n_steps, int64_t n_req,
                           uint64_t *__restrict__ agg, uint32_t *err) {
  attn_agg(req_off, rq, rh, n_steps, n_req, agg, err, (int64_t)blockIdx.x * blockDim.x + threadIdx.x,
           (int64_t)gridDim.x * blockDim.x);
}
#endif

// ------------------------------------------------------------ record counts
struct Cnt {
  uint64_t F, Bt, B, M;
};

// Expert row counts a0 .. a0 + n - 1 of a grouped GEMM (in bounds: the
// caller checks), eight loads issued before any is used, so a record's
// experts cost one memory round trip per eight instead of one each: their
// sum, the experts with rows, and the 128-row tiles, accumulated in T.
template <typename T>
__device__ __forceinline__ void expert_sums(const uint32_t *rows, uint32_t a0, uint32_t n, T &ms, T &act,
                                            T &tiles) {
  ms = act = tiles = 0;
  for (uint32_t e0 = 0; e0 < n; e0 += 8) {
    uint32_t me[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) me[u] = e0 + u < n ? rows[a0 + e0 + u] : 0u;
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      ms += (T)me[u];
      act += me[u] > 0 ? 1 : 0;
      tiles += ((T)me[u] + 127) >> 7;
    }
  }
}

// FLOPs F, bytes Bt, thread blocks B and feature row count M of one record.
__device__ __forceinline__ Cnt record_counts(int fam, uint32_t m32, uint32_t n32, uint32_t k32,
                                             uint32_t a32, uint32_t b32, uint32_t step,
                                             const EvalParams &p, uint32_t &bad) {
  const uint64_t dt = p.elem_bytes, M = m32, N = n32, K = k32, A = a32;
  Cnt c{0, 0, 0, M};
  switch (fam) {
    case KS_GEMM:
    case KS_LM_HEAD:
      c.F = 2 * M * N * K;
      c.Bt = dt * (M * K + K * N + M * N);
      c.B = ((M + 127) >> 7) * ((N + 127) >> 7);
      break;
    case KS_GROUPED_GEMM: {
      uint64_t ms = 0, act = 0, tiles = 0;
      if ((uint64_t)b32 + A <= (uint64_t)p.n_expert_rows && A <= 1024) {
        expert_sums(p.expert_rows, b32, a32, ms, act, tiles);
      } else {
        bad |= kErrExpert;
      }
      c.F = 2 * ms * N * K;
      c.Bt = dt * (ms * K + act * K * N + ms * N);
      c.B = tiles * ((N + 127) >> 7);
      c.M = ms;
      break;
    }
    case KS_ATTN_PREFILL:
    case KS_ATTN_DECODE: {
      uint64_t Q = 0, KV = 0, P = 0, T = 0;
      if ((int64_t)step < p.n_steps) {
        Q = p.agg[step];
        KV = p.agg[p.n_steps + step];
        P = p.agg[2 * p.n_steps + step];
        T = p.agg[3 * p.n_steps + step];
      }
      c.F = 4 * N * K * P;
      c.Bt = dt * (2 * N * K * Q + 2 * A * K * KV);
      c.B = N * T;
      c.M = Q;
      break;
    }
    case KS_RMSNORM:
      c.F = 4 * M * N;
      c.Bt = dt * (2 * M * N + N);
      c.B = M;
      break;
    case KS_ROPE:
      c.F = 3 * M * N * K;
      c.Bt = dt * (2 * M * N * K + M * K);
      c.B = M;
      break;
    case KS_SILU_MUL:
      c.F = 5 * M * N;
      c.Bt = 3 * dt * M * N;
      c.B = (M * N + 1023) >> 10;
      break;
    case KS_KV_WRITE:
      c.F = 0;
      c.Bt = 4 * dt * M * N * K;
      c.B = M;
      break;
    default:  // KS_EMBED
      c.F = 0;
      c.Bt = 2 * dt * M * N + 4 * M;
      c.B = M;
      break;
  }
  return c;
}

// The same counts with F and Bt rounded to fp32 as they are formed (each a
// few roundings, within 1e-6 relative of the exact values) and B exact.
// The eta = 1 stream uses it when no per-record count is written: it avoids
// the 64-bit products and 64-bit to float conversions of the exact path.
struct CntF {
  float F, Bt, M;   // M: the row count of feature x10
  uint64_t B;
};

__device__ __forceinline__ float u64_to_f32(uint64_t v) { return (float)v; }

__device__ __forceinline__ CntF record_counts_f(int fam, uint32_t m32, uint32_t n32, uint32_t k32,
                                                uint32_t a32, uint32_t b32, uint32_t step,
                                                const EvalParams &p, uint32_t &bad) {
  const float dt = (float)p.elem_bytes, M = (float)m32, N = (float)n32, K = (float)k32, A = (float)a32;
  CntF c{0.0f, 0.0f, M, 0};
  switch (fam) {
    case KS_GEMM:
    case KS_LM_HEAD:
      c.F = (M * N) * (2.0f * K);
      c.Bt = dt * (M * K + K * N + M * N);
      c.B = (uint64_t)(((m32 + 127u) >> 7) * ((n32 + 127u) >> 7));
      break;
    case KS_GROUPED_GEMM: {
      uint32_t ms = 0, act = 0, tiles = 0;
      if ((uint64_t)b32 + a32 <= (uint64_t)p.n_expert_rows && a32 <= 1024) {
        expert_sums(p.expert_rows, b32, a32, ms, act, tiles);
      } else {
        bad |= kErrExpert;
      }
      const float Ms = (float)ms;
      c.M = Ms;
      c.F = (Ms * N) * (2.0f * K);
      c.Bt = dt * (Ms * K + (float)act * (K * N) + Ms * N);
      c.B = (uint64_t)tiles * ((n32 + 127u) >> 7);
      break;
    }
    case KS_ATTN_PREFILL:
    case KS_ATTN_DECODE: {
      uint64_t Q = 0, KV = 0, P = 0, T = 0;
      if ((int64_t)step < p.n_steps) {
        Q = p.agg[step];
        KV = p.agg[p.n_steps + step];
        P = p.agg[2 * p.n_steps + step];
        T = p.agg[3 * p.n_steps + step];
      }
      const float NK = N * K;   // exact: N, K < 2^12
      c.M = u64_to_f32(Q);
      c.F = (4.0f * NK) * u64_to_f32(P);
      c.Bt = dt * (2.0f * NK * u64_to_f32(Q) + (2.0f * A * K) * u64_to_f32(KV));
      c.B = (uint64_t)n32 * T;
      break;
    }
    case KS_RMSNORM:
      c.F = 4.0f * (M * N);
      c.Bt = dt * (2.0f * (M * N) + N);
      c.B = m32;
      break;
    case KS_ROPE:
      c.F = 3.0f * ((M * N) * K);
      c.Bt = dt * (2.0f * ((M * N) * K) + M * K);
      c.B = m32;
      break;
    case KS_SILU_MUL:
      c.F = 5.0f * (M * N);
      c.Bt = 3.0f * dt * (M * N);
      c.B = ((uint64_t)m32 * n32 + 1023u) >> 10;
      break;
    case KS_KV_WRITE:
      c.F = 0.0f;
      c.Bt = 4.0f * dt * ((M * N) * K);
      c.B = m32;
      break;
    default:  // KS_EMBED
      c.F = 0.0f;
      c.Bt = 2.0f * dt * (M * N) + 4.0f * M;
      c.B = m32;
      break;
  }
  return c;
}

#if KS_HEADS == 0
// ------------------------------------------------------------ spec constants
__device__ void spec_prep_one(const ks_spec *__restrict__ specs, int s, SpecC *__restrict__ out, uint32_t *err) {
  const ks_spec sp = specs[s];
  SpecC c = {};
  const double P = sp.peak_flops, BW = sp.hbm_bw;
  // n_cu outside 1 .. 65535 is clamped and flagged (the wave count relies on
  // 24-bit products of it)
  uint32_t n = sp.n_cu;
  if (n < 1u || n > 65535u) {
    atomicOr(err, kErrSpec);
    n = n < 1u ? 1u : 65535u;
  }
  c.n = n;
  c.rcp_p = (float)(1.0 / P);
  c.rcp_bw = (float)(1.0 / BW);
  c.bw_over_p = (float)(BW / P);
  c.lr = (float)log2(BW / P);
  // t_roof is below 2^80 then (F u below 2^80, Bt below 2^63) and t_comp + t_mem,
  // unless zero, above 2^-101: x1, x6 and x7 are finite and below 2^5 like the others,
  // which come from whole numbers below 2^64 and ratios of them
  c.usual = P >= 1.0 && P <= 0x1p100 && BW >= 1.0 && BW <= 0x1p100 && sp.l2_bytes >= 0.0 ? 1u : 0u;
  c.l2 = (float)sp.l2_bytes;
  c.t0 = (float)sp.t0;
  c.rcp_t0 = (float)(1.0 / fmax(sp.t0, 1e-9));
  c.n_f = (float)n;
  c.rcp_n = (float)(1.0 / (double)n);
  c.rcp_nd = 1.0 / (double)n;
  out[s] = c;
}

__global__ void k_spec_prep(const ks_spec *__restrict__ specs, int32_t n_specs, SpecC *__restrict__ out,
                            uint32_t *err) {
  const int s = blockIdx.x * blockDim.x + threadIdx.x;
  if (s < n_specs) spec_prep_one(specs, s, out, err);
}
#endif

// Spec constants through the scalar cache: they are read-only during the
// evaluation kernel and the index is wave-uniform, so the load goes through
// the constant address space.
// (The host pass of this file only parses device functions; it has no
// constant address space.)
__device__ __forceinline__ SpecC spec_at(const SpecC *base, int i) {
#if defined(__HIP_DEVICE_COMPILE__)
  typedef const __attribute__((address_space(4))) SpecC *SpecCPtr;
  return ((SpecCPtr)base)[__builtin_amdgcn_readfirstlane(i)];
#else
  return base[i];
#endif
}

// spec-independent per-record quantities
struct RowC {
  uint64_t B;
  float Ff, Btf, Bf, rcp_b, rcp_bt1, la, x0, xs[7];  // la = log2(AI); xs = x8 .. x14
};

__device__ __forceinline__ RowC row_consts(uint64_t B, float Ff, float Btf, float Mf, uint32_t n, uint32_t k) {
  RowC r;
  r.B = B;
  r.Ff = Ff;
  r.Btf = Btf;
  r.Bf = (float)B;
  r.rcp_b = rcpf(fmaxf(r.Bf, 1.0f));
  r.rcp_bt1 = rcpf(fmaxf(r.Btf, 1.0f));
  // log2(0) = -inf for F = 0; every use clamps it from below
  r.la = log2f_fast(r.Ff * r.rcp_bt1);
  r.x0 = fmaxf(r.la, -10.0f) * (1.0f / 16);
  r.xs[0] = log2f_fast(1.0f + r.Ff) * (1.0f / 64);
  r.xs[1] = log2f_fast(1.0f + r.Btf) * (1.0f / 48);
  r.xs[2] = log2f_fast(1.0f + Mf) * (1.0f / 24);
  r.xs[3] = log2f_fast(1.0f + (float)n) * (1.0f / 24);
  r.xs[4] = log2f_fast(1.0f + (float)k) * (1.0f / 24);
  r.xs[5] = log2f_fast(1.0f + r.Ff * r.rcp_b) * (1.0f / 48);
  r.xs[6] = log2f_fast(1.0f + r.Btf * r.rcp_b) * (1.0f / 40);
  return r;
}

// Block counts below 2^23 (every record of the workloads): the wave count
// in fp32 with exact integer-valued products.  With B < 2^23, fl(B fl(1/N)) is
// within 1/N of B/N, so its ceiling is exact unless B/N is an integer k,
// where it may come out k + 1; one test of (W - 1) N >= B corrects that.
// W N <= B + N < 2^24, so the products are exact.
constexpr uint32_t kSmallB = 1u << 23;

struct Roof {
  float t_comp, t_mem, t_roof, u, W;
};

// waves, u and t_roof (Sec. 2.2, Eq. 2)
template <bool kSmall>
__device__ __forceinline__ Roof roofline(const RowC &r, const SpecC &s) {
  Roof o;
  if constexpr (kSmall) {
    // in fp32 with selects: W0 N and (W0 - 1) N are integers below 2^24,
    // exact in fp32; for B = 0, W0 = 0 and the test fails
    const float W0 = ceilf(r.Bf * s.rcp_n);
    const float W = (W0 - 1.0f) * s.n_f >= r.Bf ? W0 - 1.0f : W0;
    o.W = W;
    o.u = r.Bf > 0.0f ? W * s.n_f * r.rcp_b : 1.0f;
  } else if (r.B > 0) {
    const uint64_t W = ceil_div(r.B, s.n, s.rcp_nd);
    o.W = (float)W;
    o.u = (float)(W * s.n) * r.rcp_b;
  } else {
    o.W = 0.0f;
    o.u = 1.0f;
  }
  o.t_comp = r.Ff * o.u * s.rcp_p;
  o.t_mem = r.Btf * s.rcp_bw;
  o.t_roof = fmaxf(o.t_comp, o.t_mem);
  return o;
}

// the 16 dimensionless features (x[16 + i] = x[i]^2 for 32 inputs);
// x1 = log2(AI / ridge) = log2(AI) + log2(BW / P), and the last-wave
// occupancy B / (W N) is 1 / u
template <bool RAW = false>
__device__ __forceinline__ float feature(int i, const RowC &r, const SpecC &s, const Roof &o) {
  // the same rounding wherever the features are formed: no product is fused
  // into a sum (t_comp + t_mem of feature 7 would be, in some schedules)
#pragma clang fp contract(off)
  constexpr float k16 = RAW ? 1.0f : 1.0f / 16;
  switch (i) {
    case 0: return r.x0;
    case 1: return fmaxf(r.la + s.lr, -20.0f) * k16;
    case 2: return log2f_fast(fmaf(r.Bf, s.rcp_n, 1.0f)) * k16;
    case 3: return rcpf(o.u);
    case 4: return log2f_fast(1.0f + o.W) * k16;
    case 5: return fminf(1.0f, s.l2 * r.rcp_bt1);
    case 6: return log2f_fast(fmaxf(o.t_roof * s.rcp_t0, 0x1p-20f)) * k16;
    case 7: {
      const float den = o.t_comp + o.t_mem;
      return den > 0.0f ? o.t_comp * rcpf(den) : 0.0f;
    }
    case 8: return r.xs[0];
    case 9: return r.xs[1];
    case 10: return r.xs[2];
    case 11: return r.xs[3];
    case 12: return r.xs[4];
    case 13: return r.xs[5];
    case 14: return r.xs[6];
    default: return 1.0f;
  }
}

template <int IN, bool RAW = false>
__device__ __forceinline__ void features(const RowC &r, const SpecC &s, const Roof &o, float (&x)[IN]) {
#pragma unroll
  for (int i = 0; i < 16; ++i) x[i] = feature<RAW>(i, r, s, o);
  if constexpr (IN == 32) {
#pragma unroll
    for (int i = 0; i < 16; ++i) x[16 + i] = x[i] * x[i];
  }
}

// MFMA group schedules of the bf16 heads (gen_sched.py writes them and
// checks their dependencies): {MFMA kind (0 none, 1 layer 1, 2 layer 2),
// block, chunk, VALU kind (0 none, 1 pack, 2 epilogue), block, pack half or
// first epilogue pair, epilogue pairs}.
struct SchedGrp {
  int mk, mb, kc, vk, vb, vj, vn;
};
#include "ks_sched.inc"

// ------------------------------------------------------------ bounded head
// The bounded analytical head (Sec. 5.3 and its efficiency-factor figure):
// eta = 1 / (gamma - alpha / W'), gamma = sigma(g . x), alpha = gamma sigma(a . x),
// W' = max(W, 1).  Written as (1 + e^-zg) W' (1 + E) / ((W' - 1) + W' E),
// E = e^-za: every term is positive, so nothing cancels when alpha nears
// gamma.  prm: g (16) then a (16), in LDS.
__device__ __forceinline__ float bounded_eta(const float (&x)[16], float W, const float *prm) {
  float zg = 0.0f, za = 0.0f;
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    zg = fmaf(prm[i], x[i], zg);
    za = fmaf(prm[16 + i], x[i], za);
  }
  const float w = fmaxf(W, 1.0f);
  const float eg = __expf(-zg), ea = __expf(-za);
  return (1.0f + eg) * (w * (1.0f + ea)) * rcpf((w - 1.0f) + w * ea);
}

// ------------------------------------------------------------ Tier B grid
// The measured efficiency grid of Sec. 5.5 (Tier B), density-routed: the
// query's three coordinates (features grid_axis[d]) are mapped to node
// units t_d = (c_d - lo_d) (n_d - 1) / (hi_d - lo_d); inside the closed box,
// with all eight corners of the cell measured (not NaN), eta is their
// trilinear interpolation and `routed` is set; elsewhere the caller keeps
// the family's other head.  g: the family's nodes, row-major [n0][n1][n2],
// in LDS.  Every read stays in the family's nodes: the cell index is clamped
// to 0 .. n_d - 2 (a NaN coordinate clamps to 0 and is never routed).
__device__ __forceinline__ float grid_eta(const RowC &r, const SpecC &s, const Roof &o, const EvalParams &p,
                                          const float *g, bool &routed) {
  float fr[3];
  int idx[3];
  bool in = true;
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    const float t = (feature(p.grid_axis[d], r, s, o) - p.grid_lo[d]) * p.grid_scale[d];
    const float top = (float)(p.grid_n[d] - 1);
    in = in && t >= 0.0f && t <= top;
    const float tc = fminf(fmaxf(t, 0.0f), top);
    idx[d] = min((int)tc, p.grid_n[d] - 2);
    fr[d] = tc - (float)idx[d];
  }
  const int s2 = p.grid_n[2], s1 = p.grid_n[1] * s2;
  const float *c = g + (idx[0] * s1 + idx[1] * s2 + idx[2]);
  const float v000 = c[0], v001 = c[1], v010 = c[s2], v011 = c[s2 + 1];
  const float v100 = c[s1], v101 = c[s1 + 1], v110 = c[s1 + s2], v111 = c[s1 + s2 + 1];
  const bool known = !__builtin_isnan(v000) && !__builtin_isnan(v001) && !__builtin_isnan(v010) &&
                     !__builtin_isnan(v011) && !__builtin_isnan(v100) && !__builtin_isnan(v101) &&
                     !__builtin_isnan(v110) && !__builtin_isnan(v111);
  routed = in && known;
  const float a00 = fmaf(fr[2], v001 - v000, v000), a01 = fmaf(fr[2], v011 - v010, v010);
  const float a10 = fmaf(fr[2], v101 - v100, v100), a11 = fmaf(fr[2], v111 - v110, v110);
  const float b0 = fmaf(fr[1], a01 - a00, a00), b1 = fmaf(fr[1], a11 - a10, a10);
  return fmaf(fr[0], b1 - b0, b0);
}

// ------------------------------------------------------------ bf16 MFMA head
// Orientation: hidden units are the MFMA rows (A = weights), the 64 records
// of a wave are the columns (B = activations, two 32-column blocks), so the
// C tile of one layer is already the B operand of the next one once the
// hidden units are renumbered; the renumbering is folded into the order in
// which W2's columns are staged in LDS.
//
// v_mfma_f32_32x32x16_bf16 lane layout (l = lane, g = l / 32):
//   A[i][k]: lane l holds row l % 32, k = 8 g .. 8 g + 7
//   B[k][j]: lane l holds col l % 32, k = 8 g .. 8 g + 7
//   C[i][j]: lane l holds col l % 32, rows 8 jj + 4 g + ii, register 4 jj + ii
template <int IN, int HID>
struct HeadBF16 {
  static constexpr int MB = HID / 32;   // 32-row blocks of every layer
  static constexpr int KC1 = IN / 16;   // K chunks of layer 1
  static constexpr int KC2 = HID / 16;  // K chunks of layer 2
  static constexpr int W1_DW = MB * KC1 * 64 * 4;
  static constexpr int W2_DW = MB * KC2 * 64 * 4;
  static constexpr int B2_DW = MB * 2 * 16;
  static constexpr int W3_DW = MB * 2 * 16;
  static constexpr int OFF_W2 = W1_DW;
  static constexpr int OFF_B2 = OFF_W2 + W2_DW;
  static constexpr int OFF_W3 = OFF_B2 + B2_DW;
  static constexpr int OFF_B3 = OFF_W3 + W3_DW;
  static constexpr int LDS_DW = OFF_B3 + 4;
  static constexpr bool kMlp = true;

  // layer-2 K slot s (0..15) of chunk kc -> hidden unit of layer 1's C tile
  __device__ static __forceinline__ int hid_of(int kc, int s) {
    const int g = s >> 3, t = s & 7;
    return (kc >> 1) * 32 + 8 * (2 * (kc & 1) + (t >> 2)) + 4 * g + (t & 3);
  }
  // C-tile register r of row-block mb, lane group g -> output unit
  __device__ static __forceinline__ int out_of(int mb, int g, int r) {
    return mb * 32 + 8 * (r >> 2) + 4 * g + (r & 3);
  }

  // The head takes the raw features (x1, x2, x4 and x6 without their 1/16,
  // the squares of 32-input heads without 1/256) and W1's columns carry the
  // scale instead.  Both are powers of two: bf16 rounding commutes with
  // them and the MFMA's products are exact, so every product and sum is the
  // same bit for bit, and the spec loop saves four multiplies per record.
  static constexpr bool kRaw = true;
  // W1 column k times the scale its feature drops in the raw form
  __device__ static __forceinline__ uint32_t raw_scaled(uint16_t w, int k) {
    const int b = k & 15;
    if (b != 1 && b != 2 && b != 4 && b != 6) return w;
    const float f = bf16_to_f32(w) * (k < 16 ? 1.0f / 16 : 1.0f / 256);
    return __builtin_bit_cast(uint32_t, f) >> 16;
  }
  __device__ static void stage(uint32_t *lds, int fam, const EvalParams &p) {
    // The two-wave heads (hidden 64 and 128, 256 registers) take the thread
    // index through an opaque copy, so that the per-thread addresses of
    // these loops are formed here, when a family is staged, rather than
    // hoisted out of the work loop and kept live across it (the 16-128 head
    // spilled them to scratch); the one-wave heads keep the hoisted form
    // (the opaque copy there made their scalar spills to VGPR lanes grow).
    int tid = (int)threadIdx.x;
    if constexpr (HID <= 128) asm volatile("" : "+v"(tid));
    const uint16_t *w1 = (const uint16_t *)p.w1 + (size_t)fam * HID * IN;
    const uint16_t *w2 = (const uint16_t *)p.w2 + (size_t)fam * HID * HID;
    const uint16_t *b2 = (const uint16_t *)p.b2 + (size_t)fam * HID;
    const uint16_t *w3 = (const uint16_t *)p.w3 + (size_t)fam * HID;
    const uint16_t *b3 = (const uint16_t *)p.b3 + fam;
#pragma unroll
    for (int i = 0; i < W1_DW / kWgThreads; ++i) {
      const int d = tid + i * kWgThreads;
      const int q = d & 3, lane = (d >> 2) & 63, frag = d >> 8;
      const int kc = frag % KC1, mb = frag / KC1;
      const int row = mb * 32 + (lane & 31);
      const int k0 = kc * 16 + (lane >> 5) * 8 + 2 * q;
      lds[d] = raw_scaled(w1[row * IN + k0], k0) | (raw_scaled(w1[row * IN + k0 + 1], k0 + 1) << 16);
    }
    if ((reinterpret_cast<uintptr_t>(w2) & 15) == 0) {
      // W2 by 16-byte row chunks: hidden units 8 c8 .. 8 c8 + 7 of a row are,
      // by hid_of, slots 0-3 of lane (row mod 32) and of lane (row mod 32) +
      // 32 of one K chunk's fragment, at dwords 0-1 (first 8 of the chunk's
      // 16 units) or 2-3 (last 8): each load feeds two 8-byte LDS writes
      // (one 2-byte load per unit, scattered, took several times longer)
      // (eight rounds' loads before any is written, one memory round trip per
      // eight: the homogeneous 70B trace's evaluation 54 -> 39 us)
      constexpr int kRounds = HID * HID / 8 / kWgThreads < 8 ? HID * HID / 8 / kWgThreads : 8;
      for (int c0 = tid; c0 < HID * HID / 8; c0 += kRounds * kWgThreads) {
        u32x4 v[kRounds];
#pragma unroll
        for (int i = 0; i < kRounds; ++i)
          v[i] = *reinterpret_cast<const u32x4 *>(w2 + (size_t)(c0 + i * kWgThreads) * 8);
#pragma unroll
        for (int i = 0; i < kRounds; ++i) {
          const int c = c0 + i * kWgThreads;
          const int row = c / (HID / 8), col = (c % (HID / 8)) * 8;
          const int kc = 2 * (col >> 5) + ((col >> 4) & 1);
          const int frag = (row >> 5) * KC2 + kc;
          const int d0 = (frag * 64 + (row & 31)) * 4 + ((col & 8) ? 2 : 0);
          typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
          *reinterpret_cast<u32x2 *>(lds + OFF_W2 + d0) = u32x2{v[i][0], v[i][1]};
          *reinterpret_cast<u32x2 *>(lds + OFF_W2 + d0 + 32 * 4) = u32x2{v[i][2], v[i][3]};
        }
      }
    } else {
      for (int d = tid; d < W2_DW; d += kWgThreads) {
        const int q = d & 3, lane = (d >> 2) & 63, frag = d >> 8;
        const int kc = frag % KC2, mb = frag / KC2;
        const int row = mb * 32 + (lane & 31);
        const int s0 = (lane >> 5) * 8 + 2 * q;
        lds[OFF_W2 + d] = (uint32_t)w2[row * HID + hid_of(kc, s0)] |
                          ((uint32_t)w2[row * HID + hid_of(kc, s0 + 1)] << 16);
      }
    }
    for (int d = tid; d < B2_DW; d += kWgThreads) {
      const int r = d & 15, g = (d >> 4) & 1, mb = d >> 5;
      lds[OFF_B2 + d] = __builtin_bit_cast(uint32_t, bf16_to_f32(b2[out_of(mb, g, r)]));
    }
    for (int d = tid; d < W3_DW; d += kWgThreads) {
      const int r = d & 15, g = (d >> 4) & 1, mb = d >> 5;
      lds[OFF_W3 + d] = __builtin_bit_cast(uint32_t, bf16_to_f32(w3[out_of(mb, g, r)]));
    }
    if (tid == 0) lds[OFF_B3] = __builtin_bit_cast(uint32_t, bf16_to_f32(b3[0]));
  }

  // layer 3 over one 32-unit block of layer 2, in fp32: z += w3 . relu(h2)
  template <typename W3>
  __device__ static __forceinline__ void epilogue(const f32x16 &c0, const f32x16 &c1, const W3 &w3,
                                                  float &z0, float &z1) {
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      z0 = fmaf(w3[r], relu_f(c0[r]), z0);
      z1 = fmaf(w3[r], relu_f(c1[r]), z1);
    }
  }

  __device__ static __forceinline__ f32x16 mfma(const u32x4 &a, const u32x4 &b, const f32x16 &c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b),
                                                   c, 0, 0, 0);
  }

  __device__ static __forceinline__ void fence() { __builtin_amdgcn_sched_barrier(0); }

  __device__ static __forceinline__ u32x4 frag_w1(const uint32_t *lds, int mb, int kc, int lane) {
    return *(const u32x4 *)(lds + ((mb * KC1 + kc) * 64 + lane) * 4);
  }
  __device__ static __forceinline__ u32x4 frag_w2(const uint32_t *lds, int mb, int kc, int lane) {
    return *(const u32x4 *)(lds + OFF_W2 + ((mb * KC2 + kc) * 64 + lane) * 4);
  }

  // relu + bf16 rounding of register pairs [2 q0, 2 q1) of one layer-1 block
  // (every conversion before the first relu: no op waits on the one just
  // before it)
  __device__ static __forceinline__ void pack_part(const f32x16 &c0, const f32x16 &c1, u32x4 (&h0)[2],
                                                   u32x4 (&h1)[2], int q0, int q1) {
#pragma unroll
    for (int q = q0; q < q1; ++q) {
      h0[q >> 2][q & 3] = pack_bf16(c0[2 * q], c0[2 * q + 1]);
      h1[q >> 2][q & 3] = pack_bf16(c1[2 * q], c1[2 * q + 1]);
    }
#pragma unroll
    for (int q = q0; q < q1; ++q) {
      h0[q >> 2][q & 3] = relu_bf16x2(h0[q >> 2][q & 3]);
      h1[q >> 2][q & 3] = relu_bf16x2(h1[q >> 2][q & 3]);
    }
  }

  // ---- a fixed schedule of MFMA groups (hidden 128 and 256)
  // A group is one weight fragment times the two 32-record column blocks
  // (two MFMAs, 64 cycles of the matrix core), followed by a slice of VALU
  // work of another stage.  The table interleaves layer-1 blocks with the
  // first layer-2 chunks so that each layer-1 block is packed (relu, bf16)
  // in the groups right after it and before the chunk that consumes it,
  // and starts each layer-2 block's epilogue one group after that block's
  // last MFMA (and finishes it within the next block), so no VALU op waits
  // on an MFMA that is still in flight behind it and the matrix core never
  // drains.
  using Grp = SchedGrp;
  static constexpr int kNoV = 0, kPackV = 1, kEpiV = 2;
  __device__ static constexpr Grp sched(int i) {
    if constexpr (MB == 4) return KC1 == 1 ? kSched_4_1[i] : kSched_4_2[i];
    else return KC1 == 1 ? kSched_8_1[i] : kSched_8_2[i];
  }
  static constexpr int kNG = MB == 4 ? (KC1 == 1 ? sizeof(kSched_4_1) : sizeof(kSched_4_2)) / sizeof(Grp)
                                     : (KC1 == 1 ? sizeof(kSched_8_1) : sizeof(kSched_8_2)) / sizeof(Grp);

  struct S4 {
    u32x4 XB[2][KC1];
    u32x4 frag[3];
    f32x16 a1[2][2];
    u32x4 H0[MB][2], H1[MB][2];
    f32x16 c0, c1, p0, p1, bias;
    float w3r[2][16];
    float zacc[4];
    uint32_t lo[3];   // the lane's fragment offset (dwords) from LDS 0, 64 KB and 128 KB
    int lane, g;
  };

  // weight fragment of group I, from the lane's base address in LDS plus a
  // constant offset
  // (ds_read offsets are 16-bit byte offsets: fragments beyond 64 KB use a
  // second or third lane base, 64 KB and 128 KB further on)
  template <int I>
  __device__ static __forceinline__ u32x4 frag_of(const uint32_t *lds, const uint32_t (&lo)[3]) {
    constexpr Grp q = sched(I);
    constexpr int off = q.mk == 1 ? (q.mb * KC1 + q.kc) * 256 : OFF_W2 + (q.mb * KC2 + q.kc) * 256;
    return *(const u32x4 *)(lds + lo[off >> 14] + (off & 16383));
  }

  struct NoHook {
    template <class IC>
    __device__ __forceinline__ void operator()(IC) const {}
  };

  template <int I, class F = NoHook>
  __device__ static __forceinline__ void group(S4 &st, const uint32_t *lds, F &&hook = F{}) {
    constexpr Grp q = sched(I);
    // weight fragment of the group two ahead
    if constexpr (I + 2 < kNG && sched(I + 2).mk != 0) st.frag[(I + 2) % 3] = frag_of<I + 2>(lds, st.lo);
    const u32x4 a = st.frag[I % 3];
    if constexpr (q.mk == 1) {
      f32x16 &x0 = st.a1[q.mb & 1][0], &x1 = st.a1[q.mb & 1][1];
      if constexpr (q.kc == 0) {
        x0 = mfma(a, st.XB[0][0], f32x16{});
        x1 = mfma(a, st.XB[1][0], f32x16{});
      } else {
        x0 = mfma(a, st.XB[0][q.kc], x0);
        x1 = mfma(a, st.XB[1][q.kc], x1);
      }
    } else if constexpr (q.mk == 2) {
      if constexpr (q.kc == 0) {
        if constexpr (q.mb > 0) {
          // block mb-1 is complete: its accumulators feed the epilogue, and
          // its layer-3 weights are fetched a group before they are used
          st.p0 = st.c0;
          st.p1 = st.c1;
#pragma unroll
          for (int j = 0; j < 16; ++j)
            st.w3r[(q.mb - 1) & 1][j] = __builtin_bit_cast(float, lds[OFF_W3 + ((q.mb - 1) * 2 + st.g) * 16 + j]);
        }
        st.c1 = mfma(a, st.H1[0][0], st.bias);
        st.c0 = mfma(a, st.H0[0][0], st.bias);
      } else {
        st.c0 = mfma(a, st.H0[q.kc >> 1][q.kc & 1], st.c0);
        st.c1 = mfma(a, st.H1[q.kc >> 1][q.kc & 1], st.c1);
      }
      if constexpr (q.kc == KC2 / 2 && q.mb + 1 < MB)
        st.bias = *(const f32x16 *)(lds + OFF_B2 + ((q.mb + 1) * 2 + st.g) * 16);
      if constexpr (q.kc == KC2 - 1 && q.mb == MB - 1) {
#pragma unroll
        for (int j = 0; j < 16; ++j)
          st.w3r[q.mb & 1][j] = __builtin_bit_cast(float, lds[OFF_W3 + (q.mb * 2 + st.g) * 16 + j]);
      }
    }
    fence();
    if constexpr (q.vk == kPackV) {
      pack_part(st.a1[q.vb & 1][0], st.a1[q.vb & 1][1], st.H0[q.vb], st.H1[q.vb], 4 * q.vj, 4 * q.vj + 4);
    } else if constexpr (q.vk == kEpiV) {
      // layer 3 in fp32: relu through the sign bit, one FMA per hidden
      // unit with w3 staged as fp32 (a v_dot2c on bf16 pairs issues
      // alongside the MFMAs far worse than plain VALU ops: measured 1.7%
      // slower on the capacity grid)
#pragma unroll
      for (int j = q.vj; j < q.vj + q.vn; ++j) {
        const float *w = st.w3r[q.vb & 1];
        st.zacc[j & 1] = fmaf(w[2 * j], relu_f(st.p0[2 * j]), st.zacc[j & 1]);
        st.zacc[2 + (j & 1)] = fmaf(w[2 * j], relu_f(st.p1[2 * j]), st.zacc[2 + (j & 1)]);
        st.zacc[j & 1] = fmaf(w[2 * j + 1], relu_f(st.p0[2 * j + 1]), st.zacc[j & 1]);
        st.zacc[2 + (j & 1)] = fmaf(w[2 * j + 1], relu_f(st.p1[2 * j + 1]), st.zacc[2 + (j & 1)]);
      }
      // an empty use pins the slice here; otherwise the dot chain, whose
      // result is only needed at the end, is sunk below every MFMA
      asm volatile("" ::"v"(st.zacc[0]), "v"(st.zacc[1]), "v"(st.zacc[2]), "v"(st.zacc[3]));
    }
    hook(std::integral_constant<int, I>{});
    fence();
  }

  template <class F, int... I>
  __device__ static __forceinline__ void groups_h(S4 &st, const uint32_t *lds, F &hook,
                                                  std::integer_sequence<int, I...>) {
    (group<I>(st, lds, hook), ...);
  }

  // ---- the pieces of one spec's head (mlp4 runs them in order; the
  // software-pipelined spec loop of k_eval spreads the last block's
  // epilogue over the next spec's groups).  kPipe: the heads whose group
  // schedule that loop knows.  hook_at(I): what the loop does after group
  // I: the previous spec's last-block epilogue pairs [tp0, tp1), its eta,
  // its tail; the next spec's roofline, the features in the mask feat, the
  // squares [sq0, sq1) of a 32-input head, and the packing of layer-1 K
  // chunks [pk0, pk1).  The epilogue pairs come before the first group that
  // overwrites the last block's accumulators; the other pieces sit mostly
  // in groups with no VALU work of their own.
  struct Hook {
    int tp0, tp1;
    bool eta, tail, roof;
    uint32_t feat;
    int sq0, sq1, pk0, pk1;
  };
  static constexpr bool kPipe = (MB == 4 && KC1 == 1) || (MB == 8 && KC1 == 2);
  // the first group that overwrites the last block's accumulators (p0, p1)
  __device__ static constexpr int first_p_write() {
    for (int i = 0; i < kNG; ++i)
      if (sched(i).mk == 2 && sched(i).kc == 0 && sched(i).mb > 0) return i;
    return kNG;
  }
  __device__ static constexpr Hook hook_at(int I) {
    Hook h{0, 0, false, false, false, 0u, 0, 0, 0, 0};
    if constexpr (MB == 4) {
      // two waves per SIMD: the other wave's MFMAs cover larger slices
      if (I == 0) h.tp0 = 0, h.tp1 = 2;
      if (I == 5) h.tp0 = 2, h.tp1 = 4;
      if (I == 6) h.tp0 = 4, h.tp1 = 6;
      if (I == 11) h.tp0 = 6, h.tp1 = 8;
      if (I == 12) h.eta = true;
      if (I == 14) h.tail = true;
      if (I == 20) h.roof = true;
      if (I == 22) h.feat = 0xeu;
      if (I == 24) h.feat = 0xf0u;
      if (I == 28) h.feat = 0xff01u, h.pk0 = 0, h.pk1 = KC1;
    } else {
      // one wave per SIMD: slices small enough to issue in the shadow of
      // one group's MFMA pair, in groups without VALU work of their own
      constexpr int tp[8] = {0, 1, 4, 5, 8, 9, 12, 13};
      for (int j = 0; j < 8; ++j)
        if (I == tp[j]) h.tp0 = j, h.tp1 = j + 1;
      if (I == 16) h.eta = true;
      if (I == 20) h.tail = true;
      if (I == 35) h.roof = true;
      constexpr int ft[8] = {37, 39, 41, 43, 45, 47, 51, 53};   // features 1 .. 7, then 0 and 8 .. 15
      for (int f = 1; f < 8; ++f)
        if (I == ft[f - 1]) h.feat = 1u << f;
      if (I == ft[7]) h.feat = 0xff01u;
      if (I == 55) h.pk0 = 0, h.pk1 = 1;
      if (I == 57) h.sq0 = 0, h.sq1 = 8;
      if (I == 59) h.sq0 = 8, h.sq1 = 16;
      if (I == 61) h.pk0 = 1, h.pk1 = 2;
    }
    return h;
  }
  // every epilogue pair once, before the accumulators are overwritten;
  // every feature, square and chunk once, in order
  __device__ static constexpr bool hooks_ok() {
    int pairs = 0, last_tp = -1, eta = -1, tail = -1, roof = -1, pk = 0, sq = 0;
    uint32_t feats = 0;
    for (int i = 0; i < kNG; ++i) {
      const Hook h = hook_at(i);
      if (h.tp1 > h.tp0) {
        if (h.tp0 != pairs || i >= first_p_write()) return false;
        pairs = h.tp1, last_tp = i;
      }
      if (h.eta) eta = i;
      if (h.tail) tail = i;
      if (h.roof) roof = i;
      if (h.feat && (roof < 0 || (feats & h.feat))) return false;
      feats |= h.feat;
      if (h.sq1 > h.sq0) {
        if (h.sq0 != sq || feats != 0xffffu) return false;
        sq = h.sq1;
      }
      if (h.pk1 > h.pk0) {
        if (h.pk0 != pk) return false;
        for (int kc = h.pk0; kc < h.pk1; ++kc)
          if (kc == 0 ? feats != 0xffffu : sq < 16) return false;
        pk = h.pk1;
      }
    }
    return pairs == 8 && last_tp < eta && eta < tail && tail < roof && feats == 0xffffu && pk == KC1 &&
           (KC1 == 1 || sq == 16);
  }
  static_assert(!kPipe || hooks_ok(), "every hook once, in order, the epilogue before its accumulators go");
  __device__ static __forceinline__ void init_state(S4 &st) {
    st.lane = threadIdx.x & 63;
    st.g = st.lane >> 5;
    st.lo[0] = st.lane * 4;
    st.lo[1] = st.lo[0] + 16384;
    st.lo[2] = st.lo[0] + 32768;
    // opaque to the compiler, so it keeps the bases rather than forming
    // each address beyond 64 KB anew
    asm volatile("" : "+v"(st.lo[1]), "+v"(st.lo[2]));
#pragma unroll
    for (int j = 0; j < 4; ++j) st.zacc[j] = 0.0f;
  }
  // before a spec's groups: its features, the first fragments and b2; the
  // previous spec's partial layer-3 sums move to zp
  __device__ static __forceinline__ void begin_spec(S4 &st, const u32x4 (&XB)[2][KC1], const uint32_t *lds,
                                                    float (&zp)[4]) {
#pragma unroll
    for (int kc = 0; kc < KC1; ++kc) {
      st.XB[0][kc] = XB[0][kc];
      st.XB[1][kc] = XB[1][kc];
    }
    st.frag[0] = frag_of<0>(lds, st.lo);
    st.frag[1] = frag_of<1>(lds, st.lo);
    st.bias = *(const f32x16 *)(lds + OFF_B2 + st.g * 16);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      zp[j] = st.zacc[j];
      st.zacc[j] = 0.0f;
    }
    fence();
  }
  template <class F>
  __device__ static __forceinline__ void run_groups(S4 &st, const uint32_t *lds, F &hook) {
    groups_h(st, lds, hook, std::make_integer_sequence<int, kNG>{});
    // the last block's accumulators feed its epilogue in the next spec's groups
    st.p0 = st.c0;
    st.p1 = st.c1;
  }
  // register pairs [j0, j1) of the last block's epilogue into zp
  __device__ static __forceinline__ void tail_pairs(const S4 &st, float (&zp)[4], int j0, int j1) {
#pragma unroll
    for (int j = j0; j < j1; ++j) {
      const float *w = st.w3r[(MB - 1) & 1];
      zp[j & 1] = fmaf(w[2 * j], relu_f(st.p0[2 * j]), zp[j & 1]);
      zp[2 + (j & 1)] = fmaf(w[2 * j], relu_f(st.p1[2 * j]), zp[2 + (j & 1)]);
      zp[j & 1] = fmaf(w[2 * j + 1], relu_f(st.p0[2 * j + 1]), zp[j & 1]);
      zp[2 + (j & 1)] = fmaf(w[2 * j + 1], relu_f(st.p1[2 * j + 1]), zp[2 + (j & 1)]);
    }
  }
  // z: lanes l and l ^ 32 hold the two halves of the same record's dot
  // product; after the swap lane l < 32 adds block 0's halves of record l
  // and lane l >= 32 block 1's halves of record l.
  __device__ static __forceinline__ float tail_reduce(const float (&zp)[4], const uint32_t *lds) {
    uint32_t u0 = __builtin_bit_cast(uint32_t, zp[0] + zp[1]);
    uint32_t u1 = __builtin_bit_cast(uint32_t, zp[2] + zp[3]);
    swap32(u0, u1);
    return __builtin_bit_cast(float, u0) + __builtin_bit_cast(float, u1) +
           __builtin_bit_cast(float, lds[OFF_B3]);
  }

  // x -> bf16 pairs; the swap turns "own record" into the B layout of the
  // two 32-record column blocks
  __device__ static __forceinline__ void pack_x(const float (&x)[IN], u32x4 (&XB)[2][KC1], int kc0 = 0,
                                                int kc1 = KC1) {
    uint32_t P[IN / 2];
#pragma unroll
    for (int c = 8 * kc0; c < 8 * kc1; ++c) P[c] = pack_bf16(x[2 * c], x[2 * c + 1]);
#pragma unroll
    for (int kc = kc0; kc < kc1; ++kc) {
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        uint32_t lo = P[8 * kc + q], hi = P[8 * kc + 4 + q];
        swap32(lo, hi);
        XB[0][kc][q] = lo;
        XB[1][kc][q] = hi;
      }
    }
  }

  // one spec's head on the features XB: the groups, then the last block's
  // epilogue and the reduction
  __device__ static __forceinline__ float mlp4(const u32x4 (&XB)[2][KC1], const uint32_t *lds) {
    S4 st;
    init_state(st);
    float unused[4];
    begin_spec(st, XB, lds, unused);
    NoHook none;
    run_groups(st, lds, none);
    tail_pairs(st, st.zacc, 0, 8);
    return tail_reduce(st.zacc, lds);
  }

  // z of the lane's own record; x: that record's features (fp32).
  //
  // A SIMD's VALU and matrix core only overlap when VALU work is issued in
  // the shadow of in-flight MFMAs of the same wave, and the compiler does not
  // interleave on its own.  So the body is scheduled by hand: straight-line
  // groups fenced by sched_barrier, each holding the LDS prefetch of a later
  // weight fragment, one MFMA pair, and a few VALU ops of another stage:
  //   layer 1, block mb      | relu/bf16 packing of layer-1 block mb-1
  //   layer 2, block 0       | packing of the last layer-1 block
  //   layer 2, block mb >= 1 | epilogue of layer-2 block mb-1 (relu, bf16,
  //                            dot with w3)
  // Only the features, the last epilogue and the tail stay exposed.
  __device__ static __forceinline__ float mlp(const float (&x)[IN], const uint32_t *lds) {
    static_assert(MB == 2 || MB == 4 || MB == 8, "hidden 64, 128 or 256");
    if constexpr (MB == 4 || MB == 8) {
      u32x4 XB[2][KC1];
      pack_x(x, XB);
      return mlp4(XB, lds);
    } else {
      const int lane = threadIdx.x & 63, g = lane >> 5;
      // features -> bf16 pairs; the swap turns "own record" into the B
      // layout of the two 32-record column blocks
      uint32_t P[IN / 2];
#pragma unroll
      for (int c = 0; c < IN / 2; ++c) P[c] = pack_bf16(x[2 * c], x[2 * c + 1]);
      u32x4 XB[2][KC1];
#pragma unroll
      for (int kc = 0; kc < KC1; ++kc) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          uint32_t lo = P[8 * kc + q], hi = P[8 * kc + 4 + q];
          swap32(lo, hi);
          XB[0][kc][q] = lo;
          XB[1][kc][q] = hi;
        }
      }
      // ---- layer 1 | packing of the previous layer-1 block
      u32x4 H0[MB][2], H1[MB][2];
      f32x16 a1[2][2];
      u32x4 w1f[KC1];
#pragma unroll
      for (int kc = 0; kc < KC1; ++kc) w1f[kc] = frag_w1(lds, 0, kc, lane);
      fence();
#pragma unroll
      for (int mb = 0; mb < MB; ++mb) {
        u32x4 cur[KC1];
#pragma unroll
        for (int kc = 0; kc < KC1; ++kc) {
          cur[kc] = w1f[kc];
          if (mb + 1 < MB) w1f[kc] = frag_w1(lds, mb + 1, kc, lane);
        }
        a1[mb & 1][0] = f32x16{};
        a1[mb & 1][1] = f32x16{};
#pragma unroll
        for (int kc = 0; kc < KC1; ++kc) {
          a1[mb & 1][0] = mfma(cur[kc], XB[0][kc], a1[mb & 1][0]);
          a1[mb & 1][1] = mfma(cur[kc], XB[1][kc], a1[mb & 1][1]);
        }
        if (mb > 0) pack_part(a1[(mb - 1) & 1][0], a1[(mb - 1) & 1][1], H0[mb - 1], H1[mb - 1], 0, 8);
        fence();
      }
      // ---- layer 2: weight fragments prefetched two chunks ahead
      constexpr int NCH = MB * KC2;   // (block, chunk) pairs in order
      u32x4 wf[3];
      wf[0] = frag_w2(lds, 0, 0, lane);
      wf[1] = frag_w2(lds, 0, 1, lane);
      f32x16 bias = *(const f32x16 *)(lds + OFF_B2 + g * 16);
      f32x16 c0 = {}, c1 = {}, p0 = {}, p1 = {};
      float w3r[16];
      float z0 = 0.0f, z1 = 0.0f;
      fence();
#pragma unroll
      for (int i = 0; i < NCH; ++i) {
        const int mb = i / KC2, kc = i % KC2;
        if (i + 2 < NCH) wf[(i + 2) % 3] = frag_w2(lds, (i + 2) / KC2, (i + 2) % KC2, lane);
        if (kc == 0 && mb > 0) {
          // block mb-1's accumulators become the epilogue's inputs
          p0 = c0;
          p1 = c1;
#pragma unroll
          for (int q = 0; q < 16; ++q) w3r[q] = __builtin_bit_cast(float, lds[OFF_W3 + ((mb - 1) * 2 + g) * 16 + q]);
        }
        const u32x4 a = wf[i % 3];
        if (kc == 0) {
          c1 = mfma(a, H1[0][0], bias);
          c0 = mfma(a, H0[0][0], bias);
        } else {
          c0 = mfma(a, H0[kc >> 1][kc & 1], c0);
          c1 = mfma(a, H1[kc >> 1][kc & 1], c1);
        }
        if (kc == KC2 / 2 && mb + 1 < MB) bias = *(const f32x16 *)(lds + OFF_B2 + ((mb + 1) * 2 + g) * 16);
        if (mb == 0) {
          // pack the last layer-1 block over the first PG groups, all of
          // which come before chunk 2 (MB - 1), its first consumer
          constexpr int PG = 2 * (MB - 1) < 4 ? 2 * (MB - 1) : 4;
          if (kc < PG) pack_part(a1[(MB - 1) & 1][0], a1[(MB - 1) & 1][1], H0[MB - 1], H1[MB - 1],
                                 kc * 8 / PG, (kc + 1) * 8 / PG);
        } else {
          // chunk kc's share of block mb-1's epilogue: register pairs
          // [8 kc / KC2, 8 (kc + 1) / KC2) of the 8
#pragma unroll
          for (int q = kc * 8 / KC2; q < (kc + 1) * 8 / KC2; ++q) {
            z0 = fmaf(w3r[2 * q], relu_f(p0[2 * q]), z0);
            z1 = fmaf(w3r[2 * q], relu_f(p1[2 * q]), z1);
            z0 = fmaf(w3r[2 * q + 1], relu_f(p0[2 * q + 1]), z0);
            z1 = fmaf(w3r[2 * q + 1], relu_f(p1[2 * q + 1]), z1);
          }
          // an empty use pins this part here; otherwise the dot chain, whose
          // result is only needed at the end, is sunk below every MFMA
          asm volatile("" ::"v"(z0), "v"(z1));
        }
        fence();
      }
#pragma unroll
      for (int q = 0; q < 16; ++q) w3r[q] = __builtin_bit_cast(float, lds[OFF_W3 + ((MB - 1) * 2 + g) * 16 + q]);
      epilogue(c0, c1, w3r, z0, z1);
      // lanes l and l ^ 32 hold the two halves of the same record's dot
      // product; after the swap lane l < 32 adds block 0's halves of record
      // l and lane l >= 32 block 1's halves of record l.
      uint32_t u0 = __builtin_bit_cast(uint32_t, z0), u1 = __builtin_bit_cast(uint32_t, z1);
      swap32(u0, u1);
      return __builtin_bit_cast(float, u0) + __builtin_bit_cast(float, u1) +
             __builtin_bit_cast(float, lds[OFF_B3]);
    }
  }
};

// ------------------------------------------------------------ fp32 MFMA head
// fp32 operands on the bf16 matrix instruction, which does 16 times the work of
// the fp32 one per cycle: every operand is split exactly into three bfloat16
// pieces of 8 bits (x = x0 + x1 + x2, each the rest rounded to nearest), and of
// the nine products of pieces the six down to 2^-17 of the whole are formed,
// each exact in fp32.  What is left out (x1 y2 + x2 y1 + x2 y2, |x1| <= 2^-8 and
// |x2| <= 2^-17 of the binade) is below 2^-24 of a product, the rounding of one
// fp32 product.  The leading products and the others
// are summed apart (fp32, in the instruction) and added at the end, so that
// the leading sum is rounded once per 16 terms rather than once per 2: eta's
// root mean square error against 64 bits went from 4.8e-8 to 4.7e-8 (16-128)
// and from 4.6e-8 to 4.2e-8 (32-128), its largest from 2.1e-7 to 1.2e-7.
// 480 instructions of 32 cycles per wave and spec (32-128) instead of 640 of
// 64: the fp32 grid's 704k pairs 303 -> 161 us, the matrix cores busy 51% of the
// cycles by the counters, launch and staging among them (running the split of one
// block under the products of the next, by the compiler's group barriers or by
// hand, gave nothing).  Orientation, lane layout and hidden-unit order are the
// bf16 head's.
template <int IN, int HID>
struct HeadF32 {
  static constexpr bool kRaw = false;
  using B = HeadBF16<IN, HID>;
  static constexpr int MB = HID / 32;
  static constexpr int KC1 = IN / 16, KC2 = HID / 16;
  static constexpr int kFrag = 3 * 64 * 4;             // dwords of one fragment's three pieces
  static constexpr int W1_DW = MB * KC1 * kFrag;
  static constexpr int W2_DW = MB * KC2 * kFrag;
  static constexpr int B2_DW = MB * 2 * 16;
  static constexpr int W3_DW = MB * 2 * 16;
  static constexpr int OFF_W2 = W1_DW;
  static constexpr int OFF_B2 = OFF_W2 + W2_DW;
  static constexpr int OFF_W3 = OFF_B2 + B2_DW;
  static constexpr int OFF_B3 = OFF_W3 + W3_DW;
  static constexpr int OFF_WIDE = OFF_B3 + 4;
  static constexpr int LDS_DW = OFF_WIDE + 4;
  static constexpr bool kMlp = true;

  // The pieces hold |v| < 2^127.99 (above, the leading one rounds to infinity, and
  // what is left of infinity is NaN), exactly from 2^-102 up (below, up to 2^-126 is
  // lost).  They are taken for weights W1 and W2 below 2^52, or W1 below 2^-10 and
  // W2 below 2^62, b2 below 2^126 and w3 below 2^10: with features below 2^5 (their
  // squares below 2^10) and not below 2^-102, h1 then is below 2^67 (2^5) and
  // h2 - b2 below 2^126, and what the pieces lose moves h2 by less than 2^-42 and z
  // by less than 2^-25.  Other weights (infinities and NaN among them), and spec
  // vectors that give larger features, go through mlp_f32.
  static constexpr uint32_t kW12 = 0x59800000u;   // 2^52
  static constexpr uint32_t kW2 = 0x5E800000u, kW1 = 0x3A800000u;   // 2^62, 2^-10
  static constexpr uint32_t kB2 = 0x7E800000u, kW3 = 0x44800000u;   // 2^126, 2^10
  static constexpr uint32_t kBig = 1, kBigW2 = 2, kLargeW2 = 4, kUsualW1 = 8;
  __device__ static __forceinline__ uint32_t size_of(float v) {   // orders like |v|, NaN above all
    return __builtin_bit_cast(uint32_t, v) & 0x7FFFFFFFu;
  }

  // a pair of values as three packed pairs of pieces
  __device__ static __forceinline__ void split(float a, float b, uint32_t &p0, uint32_t &p1, uint32_t &p2) {
    p0 = pack_bf16(a, b);
    a -= __builtin_bit_cast(float, p0 << 16);
    b -= __builtin_bit_cast(float, p0 & 0xFFFF0000u);
    p1 = pack_bf16(a, b);
    a -= __builtin_bit_cast(float, p1 << 16);
    b -= __builtin_bit_cast(float, p1 & 0xFFFF0000u);
    p2 = pack_bf16(a, b);
  }

  // one value of any size as three pieces that sum to it
  __device__ static void split_wide(float v, uint32_t (&p)[3]) {
    const uint32_t top = __builtin_bit_cast(uint32_t, v) & 0xFFFF0000u;
    const bool finite = fabsf(v) < __builtin_inff();
    const float rest = finite ? v - __builtin_bit_cast(float, top) : 0.0f;
    p[0] = __builtin_isnan(v) ? 0x7FC0u : top >> 16;
    p[1] = pack_bf16(rest, 0.0f) & 0xFFFFu;
    p[2] = pack_bf16(rest - bf16_to_f32(p[1]), 0.0f) & 0xFFFFu;
  }

  // weights d, d + kWgThreads, ... of a layer's n fragments' (KC of a row of blocks,
  // stride its inputs); returns the largest size_of.  WIDE: of any size.
  template <bool WIDE, int KC, class K>
  __device__ static __forceinline__ uint32_t stage_layer(uint32_t *lds, const float *w, int stride, int tid, K &&k0) {
    uint32_t most = 0;
    // (eight rounds' loads in flight, as in the bf16 head; both layers' counts are multiples)
#pragma unroll WIDE ? 1 : 8
    for (int i = 0; i < MB * KC * 256 / kWgThreads; ++i) {
      const int d = tid + i * kWgThreads;
      const int q = d & 3, lane = (d >> 2) & 63, frag = d >> 8;
      const int kc = frag % KC, mb = frag / KC;
      const float *v = w + (mb * 32 + (lane & 31)) * stride + k0(kc, (lane >> 5) * 8 + 2 * q);
      uint32_t *o = lds + frag * kFrag + (d & 255);
      if constexpr (WIDE) {
        uint32_t a[3], b[3];
        split_wide(v[0], a);
        split_wide(v[1], b);
#pragma unroll
        for (int i = 0; i < 3; ++i) o[256 * i] = a[i] | b[i] << 16;
      } else {
        split(v[0], v[1], o[0], o[256], o[512]);
        most = max(most, max(size_of(v[0]), size_of(v[1])));
      }
    }
    return most;
  }

  __device__ static void stage(uint32_t *lds, int fam, const EvalParams &p) {
    const float *w1 = (const float *)p.w1 + (size_t)fam * HID * IN;
    const float *w2 = (const float *)p.w2 + (size_t)fam * HID * HID;
    const float *b2 = (const float *)p.b2 + (size_t)fam * HID;
    const float *w3 = (const float *)p.w3 + (size_t)fam * HID;
    float *f = (float *)lds;
    // (addresses formed here rather than kept across the work loop, as in the bf16 head)
    int tid = (int)threadIdx.x;
    asm volatile("" : "+v"(tid));
    uint32_t big = 0;
    auto in1 = [](int kc, int slot) { return kc * 16 + slot; };
    auto in2 = [](int kc, int slot) { return B::hid_of(kc, slot); };   // (of an even slot and the next: consecutive units)
    const uint32_t m1 = stage_layer<false, KC1>(lds, w1, IN, tid, in1);
    const uint32_t m2 = stage_layer<false, KC2>(lds + OFF_W2, w2, HID, tid, in2);
    static_assert(B2_DW <= kWgThreads, "a thread per bias");
    if (const int d = tid; d < B2_DW) {
      const int r = d & 15, g = (d >> 4) & 1, mb = d >> 5;
      const float b = b2[B::out_of(mb, g, r)], w = w3[B::out_of(mb, g, r)];
      f[OFF_B2 + d] = b;
      f[OFF_W3 + d] = w;
      if (size_of(b) >= kB2 || size_of(w) >= kW3) big = kBig;
    }
    if (threadIdx.x == 0) f[OFF_B3] = ((const float *)p.b3)[fam];
    // (a word per wave, so that none is reset)
    const uint32_t sizes = (__ballot(big != 0 || m1 >= kW12) ? kBig : 0u) | (__ballot(m2 >= kW2) ? kBigW2 : 0u) |
                           (__ballot(m2 >= kW12) ? kLargeW2 : 0u) | (__ballot(m1 >= kW1) ? kUsualW1 : 0u);
    if ((threadIdx.x & 63) == 0) lds[OFF_WIDE + (threadIdx.x >> 6)] = sizes;
    if (max(m1, m2) >= kB2) {   // (a thread writes the same places)
      stage_layer<true, KC1>(lds, w1, IN, tid, in1);
      stage_layer<true, KC2>(lds + OFF_W2, w2, HID, tid, in2);
    }
  }

  // whether the staged family's weights are beyond the pieces
  __device__ static __forceinline__ bool wide_weights(const uint32_t *lds) {
    const u32x4 w = *(const u32x4 *)(lds + OFF_WIDE);
    const uint32_t sizes = __builtin_amdgcn_readfirstlane(w[0] | w[1] | w[2] | w[3]);
    return (sizes & (kBig | kBigW2)) != 0 || (sizes & (kLargeW2 | kUsualW1)) == (kLargeW2 | kUsualW1);
  }

  // The head on the fp32 instruction, for weights and features of any size: a
  // fragment's lane holds the operand's row l % 32 at the slots of its half, and so
  // does each of the eight 32x32x2 products here (K = 2: one slot of either half).
  __device__ static __forceinline__ void product_f32(const uint32_t *frag, int lane, const float (&b)[2][8],
                                                     f32x16 (&c)[2]) {
    const u32x4 a0 = *(const u32x4 *)(frag + lane * 4), a1 = *(const u32x4 *)(frag + 256 + lane * 4),
                a2 = *(const u32x4 *)(frag + 512 + lane * 4);
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const int sh = j & 1 ? 0 : 16;
      auto piece = [&](uint32_t v) { return __builtin_bit_cast(float, (v << sh) & 0xFFFF0000u); };
      const float a = piece(a0[j >> 1]) + piece(a1[j >> 1]) + piece(a2[j >> 1]);
      c[0] = __builtin_amdgcn_mfma_f32_32x32x2f32(a, b[0][j], c[0], 0, 0, 0);
      c[1] = __builtin_amdgcn_mfma_f32_32x32x2f32(a, b[1][j], c[1], 0, 0, 0);
    }
  }

  __device__ static __forceinline__ float mlp_f32(const float (&x)[IN], const uint32_t *lds) {
    int lane = threadIdx.x & 63;
    asm volatile("" : "+v"(lane));   // (its addresses formed here, not kept across the spec loop)
    const int g = lane >> 5;
    const float *f = (const float *)lds;
    float X[KC1][2][8];
#pragma unroll
    for (int kc = 0; kc < KC1; ++kc)
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        uint32_t lo = __builtin_bit_cast(uint32_t, x[16 * kc + j]), hi = __builtin_bit_cast(uint32_t, x[16 * kc + 8 + j]);
        swap32(lo, hi);
        X[kc][0][j] = __builtin_bit_cast(float, lo);
        X[kc][1][j] = __builtin_bit_cast(float, hi);
      }
    float H[KC2][2][8];
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) {
      f32x16 c[2] = {f32x16{}, f32x16{}};
#pragma unroll
      for (int kc = 0; kc < KC1; ++kc) product_f32(lds + (mb * KC1 + kc) * kFrag, lane, X[kc], c);
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) H[2 * mb + (r >> 3)][i][r & 7] = fmaxf(c[i][r], 0.0f);
    }
    float z[2] = {0.0f, 0.0f};
#pragma unroll 1
    for (int mb = 0; mb < MB; ++mb) {
      const f32x16 bias = *(const f32x16 *)(f + OFF_B2 + (mb * 2 + g) * 16);
      f32x16 c[2] = {bias, bias};
#pragma unroll
      for (int kc = 0; kc < KC2; ++kc) product_f32(lds + OFF_W2 + (mb * KC2 + kc) * kFrag, lane, H[kc], c);
      const float *w3 = f + OFF_W3 + (mb * 2 + g) * 16;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        z[0] = fmaf(w3[r], fmaxf(c[0][r], 0.0f), z[0]);
        z[1] = fmaf(w3[r], fmaxf(c[1][r], 0.0f), z[1]);
      }
    }
    uint32_t a0 = __builtin_bit_cast(uint32_t, z[0]), a1 = __builtin_bit_cast(uint32_t, z[1]);
    swap32(a0, a1);
    return __builtin_bit_cast(float, a0) + __builtin_bit_cast(float, a1) + f[OFF_B3];
  }

  // hi += a0 b0; lo += the five products below it; for the two column blocks
  // in turn, so that no instruction waits for the one before it
  __device__ static __forceinline__ void product(const uint32_t *frag, int lane, const u32x4 (&b)[3], const u32x4 (&d)[3],
                                                 f32x16 (&hi)[2], f32x16 (&lo)[2]) {
    const u32x4 a0 = *(const u32x4 *)(frag + lane * 4), a1 = *(const u32x4 *)(frag + 256 + lane * 4),
                a2 = *(const u32x4 *)(frag + 512 + lane * 4);
    lo[0] = B::mfma(a2, b[0], lo[0]);
    lo[1] = B::mfma(a2, d[0], lo[1]);
    hi[0] = B::mfma(a0, b[0], hi[0]);
    hi[1] = B::mfma(a0, d[0], hi[1]);
    lo[0] = B::mfma(a1, b[1], lo[0]);
    lo[1] = B::mfma(a1, d[1], lo[1]);
    lo[0] = B::mfma(a0, b[2], lo[0]);
    lo[1] = B::mfma(a0, d[2], lo[1]);
    lo[0] = B::mfma(a1, b[0], lo[0]);
    lo[1] = B::mfma(a1, d[0], lo[1]);
    lo[0] = B::mfma(a0, b[1], lo[0]);
    lo[1] = B::mfma(a0, d[1], lo[1]);
  }

  __device__ static __forceinline__ float mlp(const float (&x)[IN], const uint32_t *lds) {
    const int lane = threadIdx.x & 63, g = lane >> 5;
    const float *f = (const float *)lds;
    u32x4 X[2][KC1][3];
    {
      uint32_t P[3][IN / 2];
#pragma unroll
      for (int c = 0; c < IN / 2; ++c) split(x[2 * c], x[2 * c + 1], P[0][c], P[1][c], P[2][c]);
#pragma unroll
      for (int kc = 0; kc < KC1; ++kc)
#pragma unroll
        for (int i = 0; i < 3; ++i)
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            uint32_t lo = P[i][8 * kc + q], hi = P[i][8 * kc + 4 + q];
            swap32(lo, hi);
            X[0][kc][i][q] = lo;
            X[1][kc][i][q] = hi;
          }
    }
    u32x4 H[2][KC2][3];
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) {
      f32x16 hi[2] = {f32x16{}, f32x16{}}, lo[2] = {f32x16{}, f32x16{}};
#pragma unroll
      for (int kc = 0; kc < KC1; ++kc) product(lds + (mb * KC1 + kc) * kFrag, lane, X[0][kc], X[1][kc], hi, lo);
      // registers 8 h .. 8 h + 7 of the block are K chunk 2 mb + h of layer 2
#pragma unroll
      for (int c = 0; c < 2; ++c)
#pragma unroll
        for (int q = 0; q < 8; ++q) {
          uint32_t p0, p1, p2;
          split(relu_f(hi[c][2 * q] + lo[c][2 * q]), relu_f(hi[c][2 * q + 1] + lo[c][2 * q + 1]), p0, p1, p2);
          H[c][2 * mb + (q >> 2)][0][q & 3] = p0;
          H[c][2 * mb + (q >> 2)][1][q & 3] = p1;
          H[c][2 * mb + (q >> 2)][2][q & 3] = p2;
        }
    }
    float z[2] = {0.0f, 0.0f};
#pragma unroll 1
    for (int mb = 0; mb < MB; ++mb) {
      const f32x16 bias = *(const f32x16 *)(f + OFF_B2 + (mb * 2 + g) * 16);
      f32x16 hi[2] = {bias, bias}, lo[2] = {f32x16{}, f32x16{}};
#pragma unroll
      for (int kc = 0; kc < KC2; ++kc)
        product(lds + OFF_W2 + (mb * KC2 + kc) * kFrag, lane, H[0][kc], H[1][kc], hi, lo);
      const float *w3 = f + OFF_W3 + (mb * 2 + g) * 16;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        z[0] = fmaf(w3[r], relu_f(hi[0][r] + lo[0][r]), z[0]);
        z[1] = fmaf(w3[r], relu_f(hi[1][r] + lo[1][r]), z[1]);
      }
    }
    uint32_t a0 = __builtin_bit_cast(uint32_t, z[0]), a1 = __builtin_bit_cast(uint32_t, z[1]);
    swap32(a0, a1);
    return __builtin_bit_cast(float, a0) + __builtin_bit_cast(float, a1) + f[OFF_B3];
  }
};

struct HeadOne {
  static constexpr int LDS_DW = 1;
  static constexpr bool kMlp = false;
  __device__ static void stage(uint32_t *, int, const EvalParams &) {}
  template <int IN>
  __device__ static float mlp(const float (&)[IN], const uint32_t *) { return 0.0f; }
};

// kMinWg: workgroups per CU the register allocator must fit (2 = two waves
// per SIMD, at most 256 registers per lane).
template <int KIND> struct KindOf;
template <> struct KindOf<kEtaOne> { using H = HeadOne; static constexpr int IN = 16; };
template <> struct KindOf<kBoundedOnly> { using H = HeadOne; static constexpr int IN = 16; };
template <> struct KindOf<kF32_16_64> { using H = HeadF32<16, 64>; static constexpr int IN = 16; };
template <> struct KindOf<kF32_16_128> { using H = HeadF32<16, 128>; static constexpr int IN = 16; };
template <> struct KindOf<kF32_32_64> { using H = HeadF32<32, 64>; static constexpr int IN = 32; };
template <> struct KindOf<kF32_32_128> { using H = HeadF32<32, 128>; static constexpr int IN = 32; };
template <> struct KindOf<kBF16_16_64> { using H = HeadBF16<16, 64>; static constexpr int IN = 16; };
template <> struct KindOf<kBF16_16_128> { using H = HeadBF16<16, 128>; static constexpr int IN = 16; };
template <> struct KindOf<kBF16_16_256> { using H = HeadBF16<16, 256>; static constexpr int IN = 16; };
template <> struct KindOf<kBF16_32_64> { using H = HeadBF16<32, 64>; static constexpr int IN = 32; };
template <> struct KindOf<kBF16_32_128> { using H = HeadBF16<32, 128>; static constexpr int IN = 32; };
template <> struct KindOf<kBF16_32_256> { using H = HeadBF16<32, 256>; static constexpr int IN = 32; };

// ------------------------------------------------------------ segmented scan
// Inclusive scan of a wave's 64 values, segmented by sorted keys, with DPP
// lane moves (no LDS round trips), in Hillis-Steele form: within each row
// of 16 lanes every lane adds the partial of the lane 1, 2, 4 and 8 below
// it (the last two only for lanes 4..15 and 8..15), then lane 15 of each
// row is added into rows 1 and 3 and lane 31 into rows 2 and 3.  A step's
// factor is 1 where its source lane holds the same key, so, the keys being
// sorted, the source's partial covers only lanes of the same segment; 0
// otherwise.  Sums are built in at most 6 levels of adds of non-negative
// terms, so the fp32 result errs by at most 6 * 2^-24 relative; tiles and
// families are then summed in fp64.

// key of the DPP source lane, or a value unequal to key where the pattern
// has no source (bound_ctrl off: such lanes keep `old`)
template <int CTRL, int ROW, int BANK>
__device__ __forceinline__ uint32_t dpp_key(uint32_t key) {
  return (uint32_t)__builtin_amdgcn_update_dpp((int)(key ^ 1u), (int)key, CTRL, ROW, BANK, false);
}

// Factor of each seg_scan step (row_shr:1, 2, 4, 8, row_bcast:15, 31).
__device__ __forceinline__ void seg_factors(uint32_t key, float (&f)[6]) {
  f[0] = dpp_key<0x111, 0xf, 0xf>(key) == key ? 1.0f : 0.0f;
  f[1] = dpp_key<0x112, 0xf, 0xf>(key) == key ? 1.0f : 0.0f;
  f[2] = dpp_key<0x114, 0xf, 0xe>(key) == key ? 1.0f : 0.0f;
  f[3] = dpp_key<0x118, 0xf, 0xc>(key) == key ? 1.0f : 0.0f;
  f[4] = dpp_key<0x142, 0xa, 0xf>(key) == key ? 1.0f : 0.0f;
  f[5] = dpp_key<0x143, 0xc, 0xf>(key) == key ? 1.0f : 0.0f;
}

// Each step is one v_fmac_f32 with its first source read through DPP
// (v += f * v[source lane]); lanes a step's bank or row mask leaves out keep
// v, and lanes whose source lies outside the row read 0 (bound_ctrl).  A DPP
// read of a VGPR written by the VALU op just before needs two wait states,
// hence the s_nop 1 before every step (the compiler does not see into the
// block, so the waits are explicit).
__device__ __forceinline__ float seg_scan(float v, const float (&f)[6]) {
  asm volatile(
      "s_nop 1\n"
      "v_fmac_f32_dpp %0, %0, %1 row_shr:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
      "s_nop 1\n"
      "v_fmac_f32_dpp %0, %0, %2 row_shr:2 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
      "s_nop 1\n"
      "v_fmac_f32_dpp %0, %0, %3 row_shr:4 row_mask:0xf bank_mask:0xe\n"
      "s_nop 1\n"
      "v_fmac_f32_dpp %0, %0, %4 row_shr:8 row_mask:0xf bank_mask:0xc\n"
      "s_nop 1\n"
      "v_fmac_f32_dpp %0, %0, %5 row_bcast:15 row_mask:0xa bank_mask:0xf\n"
      "s_nop 1\n"
      "v_fmac_f32_dpp %0, %0, %6 row_bcast:31 row_mask:0xc bank_mask:0xf\n"
      : "+v"(v)
      : "v"(f[0]), "v"(f[1]), "v"(f[2]), "v"(f[3]), "v"(f[4]), "v"(f[5]));
  return v;
}

// ------------------------------------------------------------ evaluation
// Workgroup = 4 waves; a workgroup tile is 4 consecutive 64-record wave
// tiles of one family, so the family's head is staged in LDS once and
// shared.  Workgroups stride over workgroup tiles and restage only when the
// family changes (records are family-major).
template <int KIND> struct MinWg { static constexpr int value = 1; };
template <> struct MinWg<kF32_16_64> { static constexpr int value = 2; };
template <> struct MinWg<kF32_32_64> { static constexpr int value = 2; };
template <> struct MinWg<kBF16_16_64> { static constexpr int value = 2; };
template <> struct MinWg<kBF16_16_128> { static constexpr int value = 2; };
template <> struct MinWg<kBF16_32_64> { static constexpr int value = 2; };
template <> struct MinWg<kBF16_32_128> { static constexpr int value = 2; };

// One wave's tile: 64 consecutive records of one family (nvalid = 0 for an
// idle wave of a family's last workgroup tile).
struct Tile {
  int fam, tile_in_fam, nvalid;
  int64_t row0, fam_lo, fam_hi;
};

// fam0: a family at or before the tile's (workgroups walk tiles in order)
__device__ __forceinline__ Tile locate(const EvalParams &p, int wt, int wave, int fam0) {
  Tile t;
  int fam = fam0;
  while (wt >= p.wgt_off[fam + 1]) ++fam;
  t.fam = fam;
  t.tile_in_fam = (wt - p.wgt_off[fam]) * kWgWaves + wave;
  t.fam_lo = p.fam_off[fam];
  t.fam_hi = p.fam_off[fam + 1];
  t.row0 = t.fam_lo + (int64_t)t.tile_in_fam * kTileRows;
  const int64_t left = t.fam_hi - t.row0;
  t.nvalid = left <= 0 ? 0 : (left < kTileRows ? (int)left : kTileRows);
  return t;
}

// The record fields a lane's family uses (the others are never read), plus
// the steps just before and after the tile within its family: prev and next
// by scalar loads, or (VEC) pn by one vector load, the one before in lane 0
// and the one after in the other lanes (see tile_edges).
struct Fields {
  uint32_t st, m, n, k, a, b, prev, next, pn;
  float mult;   // dispatches the record stands for (1 without a multiplicity array)
};

template <bool MULT, bool VEC>
__device__ __forceinline__ Fields load_fields(const EvalParams &p, const Tile &t, int lane) {
  Fields f = {0, 0, 0, 0, 0, 0, kNoKey, kNoKey, kNoKey, 1.0f};
  if (t.nvalid == 0) return f;
  // wave-uniform bases plus a 32-bit lane offset (no per-lane 64-bit
  // address arithmetic)
  const uint32_t off = (uint32_t)(lane < t.nvalid ? lane : 0);
  const int64_t r0 = t.row0;
  const int fam = t.fam;
  const bool grouped = fam == KS_GROUPED_GEMM;
  const bool attn = fam == KS_ATTN_PREFILL || fam == KS_ATTN_DECODE;
  f.st = (p.step + r0)[off];
  f.n = (p.n + r0)[off];
  if (!grouped && !attn) f.m = (p.m + r0)[off];
  if (fam != KS_RMSNORM && fam != KS_SILU_MUL && fam != KS_EMBED) f.k = (p.k + r0)[off];
  if (grouped || attn) f.a = (p.a + r0)[off];
  if (grouped) f.b = (p.b + r0)[off];
  if constexpr (MULT) {
    if (p.mult) f.mult = (float)(p.mult + r0)[off];   // exact below 2^24
  }
  const bool hp = t.row0 > t.fam_lo, hn = t.row0 + kTileRows < t.fam_hi;
  if constexpr (VEC) {
    // one vector load for both neighbours (each lane's address stays inside
    // the family: the tile's first row where a neighbour does not exist).
    // In a short loop a scalar load here costs its whole latency: the next
    // scalar load of the spec loop waits for it (scalar loads complete out
    // of order, so waits are for all of them).
    const int pn_off = lane == 0 ? (hp ? -1 : 0) : (hn ? kTileRows : 0);
    f.pn = (p.step + r0)[pn_off];
  } else {
    if (hp) f.prev = p.step[t.row0 - 1];
    if (hn) f.next = p.step[t.row0 + kTileRows];
  }
  return f;
}

// the steps just before and after tile t (kNoKey where the family ends)
template <bool VEC>
__device__ __forceinline__ void tile_edges(const Tile &t, const Fields &f, uint32_t &prev, uint32_t &next) {
  if constexpr (VEC) {
    prev = t.row0 > t.fam_lo ? __builtin_amdgcn_readlane(f.pn, 0) : kNoKey;
    next = t.row0 + kTileRows < t.fam_hi ? __builtin_amdgcn_readlane(f.pn, 1) : kNoKey;
  } else {
    prev = f.prev;
    next = f.next;
  }
}

// Variants, each a separate instantiation so that the kernels without them
// keep their registers and schedule: kVarGrid compiles Tier B routing in,
// kVarMult weights each record's step-sum term by its multiplicity, kVarUniq
// takes the different records k_unique found (each one's t for every spec is
// stored, no step sums or per-pair outputs) and, with kVarRest, beside them
// every record of the families left out (grouped GEMMs, and those whose
// different records did not fit): one launch, whose parts fill each other's last round
// (MoE trace 61 -> 54 us), but the code of both (homogeneous 70B trace, where
// nothing is left out: 46 us with it, 39 without; 16 specs of a 7B trace whose
// records do not repeat, 880 us of head work, 3% in all).
enum : int { kVarGrid = 1, kVarMult = 2, kVarUniq = 4, kVarRest = 8, kNumVars = 16 };

// heads with limits on their weights and features, beyond which they take mlp_f32
template <class H, class = void> struct SizedOK : std::false_type {};
template <class H> struct SizedOK<H, std::void_t<decltype(H::kW12)>> : std::true_type {};

// heads that take the software-pipelined spec loop
template <class H, class = void> struct PipeOK : std::false_type {};
template <class H> struct PipeOK<H, std::enable_if_t<H::kPipe>> : std::true_type {};

// How many ranges to split S specs into for `tiles` tiles on `grid` workgroups:
// the fewest spec evaluations in a row (an item's setup counts for 0.8 of one),
// over one to four rounds of the grid.  (As many ranges as fill the grid, a
// remainder taking a second round, took 475 us where this takes 307, fp32 grid.)
// spec_cost: that of k rounds (0: one range), and its ranges.
__host__ __device__ inline uint32_t spec_cost(uint32_t tiles, uint32_t grid, uint32_t S, uint32_t k, uint32_t &ranges) {
  ranges = 1;
  uint32_t per = S;
  if (k > 0 && tiles > 0) {
    uint32_t c = k * grid / tiles;
    c = c < 1 ? 1 : c < S ? c : S;
    per = (S + c - 1) / c;
    ranges = (S + per - 1) / per;
  }
  return (tiles * ranges + grid - 1) / grid * (5 * per + 4);
}

// Tiles that fill the grid by themselves are split only for an eighth less: two
// specs in two ranges (27 for 28) took 43 us where one range takes 35 (342 tiles on
// 256 workgroups, bf16 32-256, GEMMs on the bounded head), sixteen in three (136
// for 168) 172 and 202 (290 tiles, a collapsed mixture of experts).
inline int spec_ranges(uint32_t tiles, uint32_t grid, uint32_t S) {
  uint32_t best = 1, cost = ~0u, whole = 0;
  for (uint32_t k = 0; k <= 4; ++k) {
    uint32_t c, t = spec_cost(tiles, grid, S, k, c);
    if (k == 0) whole = t;
    if (t < cost) cost = t, best = c;
  }
  return tiles < grid || 8 * cost <= 7 * whole ? (int)best : 1;
}

// The work of the unique-record variant, formed on the device (the different
// records are counted there).  Items of different records are four (64-record
// tile, spec range) pairs of one family, one per wave, so that a family's last
// tiles do not leave waves idle; items of the other families' records are
// workgroup tiles and spec ranges as without this variant.
struct UniqTiles {
  int wgt[KS_NFAM + 1], cnt[KS_NFAM], spec_chunk, n_chunks;   // different records
  int d_wgt[KS_NFAM + 1], d_chunk, d_chunks;                  // every record
};

// By one wave: lane f has family f, and lanes 0 .. 4 and 8 .. 12 price the spec
// ranges of the different records and of the others (one thread that did it all
// took 5 to 10 us, with its divisions in a row).
__device__ __forceinline__ void uniq_tiles(const EvalParams &p, int grid, UniqTiles &u) {
  const int lane = threadIdx.x & 63, f = lane < KS_NFAM ? lane : 0;
  const uint32_t over = p.u_over[f], count = p.u_count[f];   // (in flight together)
  const bool on = ((p.uniq_mask >> f) & 1u) && !over;
  const int cnt = lane < KS_NFAM && on ? (int)min(count, p.u_cap[f]) : 0;
  const int t64 = (cnt + kTileRows - 1) / kTileRows;
  int rest = lane < KS_NFAM && !on ? p.wgt_off[f + 1] - p.wgt_off[f] : 0, tiles = t64, all = rest;
#pragma unroll
  for (int off = 1; off < 16; off <<= 1) {
    tiles += __shfl_xor(tiles, off);
    all += __shfl_xor(all, off);
  }
  // (each family's last item of different records may be partly filled)
  const bool other = lane >= 8;
  const uint32_t n = other ? (uint32_t)all : (uint32_t)(tiles + kWgWaves - 1) / kWgWaves;
  const uint32_t g = other ? (uint32_t)grid : (uint32_t)max(grid - KS_NFAM, 1);
  uint32_t c = 1, cost = ~0u;
  // four full rounds and more take one range (and the products below stay small)
  if ((lane & 7) == 0 || ((lane & 7) <= 4 && n < 4 * g)) cost = spec_cost(n, g, (uint32_t)p.n_specs, lane & 7, c);
#pragma unroll
  for (int off = 1; off < 8; off <<= 1) {
    const uint32_t c2 = __shfl_xor(c, off), t2 = __shfl_xor(cost, off);
    if (t2 < cost || (t2 == cost && c2 < c)) cost = t2, c = c2;
  }
  const int cu = __builtin_amdgcn_readlane((int)c, 0), cd = __builtin_amdgcn_readlane((int)c, 8);
  int items = (t64 * cu + kWgWaves - 1) / kWgWaves;
  if (lane < KS_NFAM) u.cnt[lane] = cnt;
#pragma unroll
  for (int off = 1; off < 16; off <<= 1) {
    const int i2 = __shfl_up(items, off), r2 = __shfl_up(rest, off);
    if (lane >= off) items += i2, rest += r2;
  }
  if (lane < KS_NFAM) {
    u.wgt[lane + 1] = items;
    u.d_wgt[lane + 1] = rest;
  }
  if (lane == 0) {
    u.wgt[0] = u.d_wgt[0] = 0;
    u.n_chunks = cu;
    u.spec_chunk = (p.n_specs + cu - 1) / cu;
    u.d_chunks = cd;
    u.d_chunk = (p.n_specs + cd - 1) / cd;
  }
}

// item w of the different records, this wave's tile and spec range: row0 counts
// the records from the family's first
__device__ __forceinline__ Tile locate_uniq(const UniqTiles &u, int w, int wave, int &range) {
  Tile t;
  int fam = 0;
  while (w >= __builtin_amdgcn_readfirstlane(u.wgt[fam + 1])) ++fam;
  const int i = (w - __builtin_amdgcn_readfirstlane(u.wgt[fam])) * kWgWaves + wave;
  const int c = __builtin_amdgcn_readfirstlane(u.n_chunks);
  t.fam = fam;
  t.tile_in_fam = c == 1 ? i : i / c;
  range = c == 1 ? 0 : i % c;
  t.fam_lo = 0;
  t.fam_hi = __builtin_amdgcn_readfirstlane(u.cnt[fam]);
  t.row0 = (int64_t)t.tile_in_fam * kTileRows;
  const int64_t left = t.fam_hi - t.row0;
  t.nvalid = left <= 0 ? 0 : (left < kTileRows ? (int)left : kTileRows);
  return t;
}

// workgroup tile wt of the families whose every record is evaluated
__device__ __forceinline__ Tile locate_rest(const EvalParams &p, const UniqTiles &u, int wt, int wave) {
  int fam = 0;
  while (wt >= __builtin_amdgcn_readfirstlane(u.d_wgt[fam + 1])) ++fam;
  return locate(p, p.wgt_off[fam] + wt - __builtin_amdgcn_readfirstlane(u.d_wgt[fam]), wave, fam);
}

__device__ __forceinline__ Fields load_uniq(const EvalParams &p, const Tile &t, int lane) {
  Fields f = {0, 0, 0, 0, 0, 0, kNoKey, kNoKey, kNoKey, 1.0f};
  if (t.nvalid == 0) return f;
  const uint32_t off = (uint32_t)(lane < t.nvalid ? lane : 0);
  const size_t row = (p.u_list + p.u_base[t.fam] + t.row0)[off];
  const int fam = t.fam;
  const bool attn = fam == KS_ATTN_PREFILL || fam == KS_ATTN_DECODE;
  f.n = p.n[row];
  if (attn) {
    f.st = p.step[row];   // (the other families' latency does not depend on the step)
    f.a = p.a[row];
  } else {
    f.m = p.m[row];
  }
  if (fam != KS_RMSNORM && fam != KS_SILU_MUL && fam != KS_EMBED) f.k = p.k[row];
  return f;
}

// Spec s's per-pair outputs of the lane's record and its segmented step sum:
// a tail lane stores its segment's sum to dst[s] (dst: the tile's carry
// slots or the (family, step) partials, one per spec, contiguous), a record
// of multiplicity m adding m t (one fp32 rounding).
// (UNIQ: with u_dst, a different record's t to u_dst[s] instead.)
template <bool MULT, bool UNIQ, bool REST>
__device__ __forceinline__ void spec_tail(const EvalParams &p, int s, float t_roof, float eta, float t, bool valid,
                                          bool live, int64_t row, float tfac, const float (&fac)[6], double *dst,
                                          float *u_dst) {
  if constexpr (UNIQ) {
    if (!REST || u_dst) {
      if (valid) {
        u_dst[s] = t;
        if (p.u_pair) {
          u_dst[p.u_pair + s] = t_roof;
          u_dst[2 * p.u_pair + s] = eta;
        }
      }
      return;
    }
  }
  // (the per-pair test first: a call without per-pair outputs forms no
  // address)
  if ((p.o_troof || p.o_eta || p.o_t) && valid) {
    const size_t i = (size_t)s * (size_t)p.fam_off[KS_NFAM] + (size_t)row;
    if (p.o_troof) p.o_troof[i] = t_roof;
    if (p.o_eta) p.o_eta[i] = eta;
    if (p.o_t) p.o_t[i] = t;
  }
  if (p.partial) {
    const float v = seg_scan(MULT ? t * tfac : (live ? t : 0.0f), fac);
    if (dst) dst[s] = (double)v;
  }
}

// work items per workgroup below which the heads take contiguous ranges
constexpr int kBlockedItems = 32;

// the workgroup tile and the spec range of work item w: w / n and w % n,
// with no integer division in the usual case of one range of all specs
__device__ __forceinline__ int item_tile(int w, int n) {
  if (n == 1) return w;
  return w / n;
}
__device__ __forceinline__ int item_range(int w, int n) {
  if (n == 1) return 0;
  return w % n;
}

template <int KIND, int VAR>
__global__ __launch_bounds__(kWgThreads, MinWg<KIND>::value) void k_eval(EvalParams p) {
  constexpr bool GRID = (VAR & kVarGrid) != 0;
  constexpr bool UNIQ = (VAR & kVarUniq) != 0;
  constexpr bool REST = !UNIQ || (VAR & kVarRest) != 0;
  constexpr bool MULT = (VAR & (kVarMult | kVarRest)) != 0;   // (kVarRest: if there are any)
  using H = typename KindOf<KIND>::H;
  constexpr int IN = KindOf<KIND>::IN;
  __shared__ __align__(16) uint32_t lds[H::LDS_DW];   // 16-byte fragment reads, 8-byte staging writes
  __shared__ float bnd_lds[32];   // the bounded head of the staged family: g then a
  __shared__ float grid_lds[KS_GRID_MAX_NODES];   // the staged family's measured grid
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // work item w: workgroup tile w / n_chunks, specs [s0, s1) of range w % n_chunks
  int n_chunks = p.n_chunks, spec_chunk = p.spec_chunk;
  int n_work = p.wgt_off[KS_NFAM] * n_chunks, n_uniq = 0;
  __shared__ UniqTiles ut;
  if constexpr (UNIQ) {
    if (threadIdx.x < 64) uniq_tiles(p, (int)gridDim.x, ut);
    __syncthreads();
    n_chunks = __builtin_amdgcn_readfirstlane(ut.d_chunks);
    spec_chunk = __builtin_amdgcn_readfirstlane(ut.d_chunk);
    n_work = __builtin_amdgcn_readfirstlane(ut.d_wgt[KS_NFAM]) * n_chunks;
    n_uniq = __builtin_amdgcn_readfirstlane(ut.wgt[KS_NFAM]);
  }
  // tiles without a head, and the heads that run one wave per SIMD, take
  // their neighbour steps by a vector load (the scalar loads' round trip is
  // waited for by the next scalar or LDS wait, which one wave per SIMD
  // cannot cover; with two waves per SIMD the vector load measured no
  // better overall)
  constexpr bool VEC = !H::kMlp || MinWg<KIND>::value == 1;
  int staged = -1;
  bool wide_head = false;   // the staged family's weights
  // With few work items per workgroup the heads take a contiguous range of
  // them, so that a workgroup meets one or two families and stages their
  // weights into LDS once or twice (striding over the grid it restaged them
  // at nearly every item); with many, striding balances the families'
  // different per-tile costs better, and so it does for calls where some
  // families take the bounded head or a grid (far cheaper tiles than the
  // MLP's); the HBM-bound kinds always stride, which keeps the chip's loads
  // in one window.  (The bounds are wave-uniform: readfirstlane keeps them
  // in scalar registers.)
  const int G = (int)gridDim.x, b = (int)blockIdx.x;
  const bool blocked = H::kMlp && !GRID && p.bounded_mask == 0u && n_work < kBlockedItems * G;
  const int w_begin = blocked ? __builtin_amdgcn_readfirstlane(b * (n_work / G) + min(b, n_work % G)) : b;
  const int w_end =
      blocked ? __builtin_amdgcn_readfirstlane(w_begin + n_work / G + (b < n_work % G ? 1 : 0)) : n_work;
  const int w_step = blocked ? 1 : G;
  // The different records' items, after those: contiguous ranges from the last
  // workgroup back (the first ones have the remainder of the others).
  const int ub = G - 1 - b;
  const int u_begin = UNIQ ? __builtin_amdgcn_readfirstlane(ub * (n_uniq / G) + min(ub, n_uniq % G)) : 0;
  const int u_end = UNIQ ? __builtin_amdgcn_readfirstlane(u_begin + n_uniq / G + (ub < n_uniq % G ? 1 : 0)) : 0;
  // the next tile's fields are loaded while the current one is evaluated
  Tile tn = {};
  Fields fn = {0, 0, 0, 0, 0, 0, kNoKey, kNoKey, kNoKey, 1.0f};
  int range_n = 0;
  bool uniq_n = false;
  // item w of every record's, or (w at or past w_end) item u of the different ones
  auto fetch = [&](int w, int u) {
    uniq_n = false;
    if (REST && w < w_end) {
      range_n = item_range(w, n_chunks);
      if constexpr (UNIQ) tn = locate_rest(p, ut, item_tile(w, n_chunks), wave);
      else tn = locate(p, item_tile(w, n_chunks), wave, tn.fam);
      fn = load_fields<MULT, VEC>(p, tn, lane);
    } else if constexpr (UNIQ) {
      if (u < u_end) {
        uniq_n = true;
        tn = locate_uniq(ut, u, wave, range_n);
        fn = load_uniq(p, tn, lane);
      }
    }
  };
  fetch(w_begin, u_begin);
  for (int w = w_begin, u = u_begin; (REST && w < w_end) || (UNIQ && u < u_end);) {
    const Tile tc = tn;
    const Fields fc = fn;
    const int range = range_n;
    const bool uq = UNIQ && (!REST || uniq_n);
    if (REST && w < w_end) w += w_step;
    else ++u;
    fetch(w, u);
    const int chunk = uq ? __builtin_amdgcn_readfirstlane(ut.spec_chunk) : spec_chunk;
    const int s_lo = range * chunk;
    const int s_hi = min(s_lo + chunk, p.n_specs);
    const int fam = tc.fam;
    // this family takes the bounded head (the plain eta = 1 stream has none)
    const bool bnd = KIND != kEtaOne && ((p.bounded_mask >> fam) & 1u);
    // ... and a measured grid that routes some of its records
    const bool grd = GRID && ((p.grid_mask >> fam) & 1u);
    if (H::kMlp || (KIND != kEtaOne && (p.bounded_mask || GRID))) {
      if (fam != staged) {
        __syncthreads();
        if (bnd) {
          if (threadIdx.x < 32) bnd_lds[threadIdx.x] = p.bounded[fam * 32 + threadIdx.x];
        } else {
          if constexpr (H::kMlp) H::stage(lds, fam, p);
        }
        if (grd) {
          const float *src = p.grid + (size_t)fam * p.grid_nodes;
          for (int i = threadIdx.x; i < p.grid_nodes; i += kWgThreads) grid_lds[i] = src[i];
        }
        __syncthreads();
        staged = fam;
        if constexpr (SizedOK<H>::value) wide_head = !bnd && H::wide_weights(lds);
      }
    }
    if (tc.nvalid == 0) continue;
    const int nvalid = tc.nvalid;
    const bool valid = lane < nvalid;
    const int64_t row = tc.row0 + (valid ? lane : 0);

    uint32_t bad = 0;
    if ((int64_t)fc.st >= p.n_steps) bad |= kErrStep;
    RowC rc;
    // F, Bt and the feature row count in fp32 as they are formed (a few
    // roundings, within 1e-6 relative of the exact counts) when no count is
    // written: no 64-bit products or 64-bit to float conversions.  Calls
    // with a measured grid keep the exact path, so that a record's cell is
    // the one the exact features give.
    if (!GRID && !p.o_flops && !p.o_bytes && !p.o_blocks) {
      const CntF cf = record_counts_f(fam, fc.m, fc.n, fc.k, fc.a, fc.b, fc.st, p, bad);
      rc = row_consts(cf.B, cf.F, cf.Bt, cf.M, fc.n, fc.k);
    } else {
      const Cnt c = record_counts(fam, fc.m, fc.n, fc.k, fc.a, fc.b, fc.st, p, bad);
      if (!uq && valid) {
        if (p.o_flops) p.o_flops[row] = c.F;
        if (p.o_bytes) p.o_bytes[row] = c.Bt;
        if (p.o_blocks) p.o_blocks[row] = c.B;
      }
      rc = row_consts(c.B, (float)c.F, (float)c.Bt, (float)c.M, fc.n, fc.k);
    }
    if (valid && bad) atomicOr(p.err, bad);
    const bool live = valid && !(bad & kErrStep);
    const bool small = __ballot(rc.B >= kSmallB) == 0;   // wave-uniform

    float fac[6];
    float tfac = 0.0f;
    double *dst = nullptr;
    float *u_dst = nullptr;
    if (uq) {
      u_dst = p.u_t + ((size_t)p.u_base[fam] + (size_t)tc.row0 + (size_t)(valid ? lane : 0)) * (size_t)p.n_specs;
    } else {
      // segment structure of this tile (spec-independent): keys are sorted
      const uint32_t key = live ? fc.st : kNoKey;
      const uint32_t key_dn = dpp_key<0x130, 0xf, 0xf>(key);   // wave_shl:1, lane 63: unequal
      const bool is_tail = live && key_dn != key;
      const uint32_t key0 = __builtin_amdgcn_readfirstlane(key);
      uint32_t prev, next;
      tile_edges<VEC>(tc, fc, prev, next);
      const bool to_carry = is_tail && key == key0 && prev == key0;
      const int tile_id = p.tile_off[fam] + tc.tile_in_fam;
      if (p.range) {
        // the (family, step) record range, written where its global first
        // and last records are
        const uint32_t key_up = dpp_key<0x138, 0xf, 0xf>(key);   // wave_shr:1
        const bool head = live && (lane == 0 ? prev != key : key_up != key);
        const bool tail = live && (lane == nvalid - 1 ? next != key : key_dn != key);
        if (head) p.range[2 * ((size_t)fam * p.n_steps + key)] = (uint32_t)row;
        if (tail) p.range[2 * ((size_t)fam * p.n_steps + key) + 1] = (uint32_t)(row + 1);
      }
      // A tail lane stores its segment's sum (seg_scan): into the tile's carry
      // slot if the segment continues from the previous tile, else into the
      // (spec, family, step) partial.
      seg_factors(key, fac);
      // the scan input is m t for a live record of multiplicity m (1 without
      // a multiplicity array) and 0 otherwise: one product per spec instead
      // of a select.  A lane that is not live either repeats lane 0's record
      // (a tail lane past nvalid, whose t is finite whenever lane 0's is) or
      // is flagged bad data; both sit at or after the wave's last live lane or
      // carry a flagged record, so the scan of every live segment is unchanged.
      tfac = MULT ? (live ? fc.mult : 0.0f) : 0.0f;
      // (spec-minor layout: a tail lane's sums for all specs are one
      // contiguous run, so its stores fill whole cache lines)
      if (p.partial && is_tail) {
        if (to_carry)
          dst = p.carry + (size_t)tile_id * (size_t)p.n_specs;
        else
          dst = p.partial + ((size_t)fam * (size_t)p.n_steps + key) * (size_t)p.n_specs;
      }
    }

    if constexpr (PipeOK<H>::value && !GRID) {
      if (!bnd) {
        // Software-pipelined spec loop: spec s's MFMA groups carry, in their
        // VALU slots, the last block's epilogue and the tail of spec s - 1
        // (early groups) and the roofline and features of spec s + 1 (late
        // groups), so that no VALU work of a spec stands outside the MFMA
        // stream.  Spec s - 1's last-block accumulators and layer-3 partial
        // sums live on in the head state (p0/p1, zp) until its epilogue
        // has read them.
        using S4 = typename H::S4;
        S4 st;
        H::init_state(st);
        // specs s_lo + s, s = 0 .. S - 1
        const int S = s_hi - s_lo;
        SpecC sc = spec_at(p.spec_c, s_lo);
        Roof o = small ? roofline<true>(rc, sc) : roofline<false>(rc, sc);
        constexpr int KC1 = H::KC1;
        u32x4 XB[2][KC1];
        {
          float x[IN];
          features<IN, H::kRaw>(rc, sc, o, x);
          H::pack_x(x, XB);
        }
        float zp[4] = {0.0f, 0.0f, 0.0f, 0.0f};
        float tr_prev = 0.0f, t0_prev = 0.0f;
        // one spec's groups; NEXT: whether a next spec exists (the last
        // spec's groups are a second copy without the next spec's work)
        auto spec_iter = [&](int s, auto next_c) {
          constexpr bool NEXT = decltype(next_c)::value;
          const SpecC sn = spec_at(p.spec_c, s_lo + (NEXT ? s + 1 : s));
          Roof on;
          u32x4 XBn[2][KC1];
          float xn[IN];
          float eta_prev = 1.0f;
          const float tr_cur = o.t_roof, t0_cur = sc.t0;
          H::begin_spec(st, XB, lds, zp);
          // after each group, its share of the neighbouring specs' work
          // (hook_at)
          auto hook = [&](auto ic) {
            constexpr int I = decltype(ic)::value;
            constexpr typename H::Hook a = H::hook_at(I);
            if constexpr (a.tp1 > a.tp0) H::tail_pairs(st, zp, a.tp0, a.tp1);
            if constexpr (a.eta) eta_prev = 1.0f + __expf(-H::tail_reduce(zp, lds));
            if constexpr (a.tail) {
              if (s > 0)
                spec_tail<MULT, UNIQ, REST>(p, s_lo + s - 1, tr_prev, eta_prev, fmaxf(tr_prev * eta_prev, t0_prev), valid, live,
                                      row, tfac, fac, dst, u_dst);
            }
            if constexpr (NEXT && a.roof) on = small ? roofline<true>(rc, sn) : roofline<false>(rc, sn);
            if constexpr (NEXT && a.feat != 0u) {
#pragma unroll
              for (int i = 0; i < 16; ++i)
                if ((a.feat >> i) & 1u) xn[i] = feature<H::kRaw>(i, rc, sn, on);
            }
            if constexpr (NEXT && a.sq1 > a.sq0) {
#pragma unroll
              for (int i = a.sq0; i < a.sq1; ++i) xn[16 + i] = xn[i] * xn[i];
            }
            if constexpr (NEXT && a.pk1 > a.pk0) H::pack_x(xn, XBn, a.pk0, a.pk1);
          };
          H::run_groups(st, lds, hook);
          tr_prev = tr_cur;
          t0_prev = t0_cur;
          if constexpr (NEXT) {
            o = on;
            sc = sn;
#pragma unroll
            for (int kc = 0; kc < KC1; ++kc) {
              XB[0][kc] = XBn[0][kc];
              XB[1][kc] = XBn[1][kc];
            }
          }
        };
        for (int s = 0; s + 1 < S; ++s) spec_iter(s, std::true_type{});
        spec_iter(S - 1, std::false_type{});
        // the last spec's epilogue and tail
        float zl[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) zl[j] = st.zacc[j];
        H::tail_pairs(st, zl, 0, 4);
        H::tail_pairs(st, zl, 4, 8);
        const float eta = 1.0f + __expf(-H::tail_reduce(zl, lds));
        spec_tail<MULT, UNIQ, REST>(p, s_lo + S - 1, tr_prev, eta, fmaxf(tr_prev * eta, t0_prev), valid, live, row, tfac,
                              fac, dst, u_dst);
        continue;
      }
    }
    bool rest = false;   // some of the specs are beyond the pieces' limits
    for (int s = s_lo; s < s_hi; ++s) {
      const SpecC sc = spec_at(p.spec_c, s);
      if constexpr (SizedOK<H>::value) {
        if (!sc.usual || wide_head) {
          rest = true;
          continue;
        }
      }
      const Roof o = small ? roofline<true>(rc, sc) : roofline<false>(rc, sc);
      float eta = 1.0f;
      // Tier B first: the family's other head runs only if some record of
      // the wave is not routed to the grid
      bool routed = false;
      float eta_g = 0.0f;
      if (grd) eta_g = grid_eta(rc, sc, o, p, grid_lds, routed);
      const bool other = !grd || __ballot(valid && !routed) != 0;
      if (bnd) {
        if (other) {
          float x[16];
          features<16>(rc, sc, o, x);
          eta = bounded_eta(x, o.W, bnd_lds);
        }
      } else {
        if constexpr (H::kMlp) {
          if (other) {
            float x[IN];
            features<IN, H::kRaw>(rc, sc, o, x);
            const float z = H::mlp(x, lds);
            eta = 1.0f + __expf(-z);
          }
        }
      }
      if (routed) eta = eta_g;
      const float t = fmaxf(o.t_roof * eta, sc.t0);
      // (without a grid the source is a per-family constant, written by
      // k_fill_source instead, so the plain kernels keep their registers)
      if constexpr (GRID && !UNIQ) {
        if (valid && p.o_src) p.o_src[(size_t)s * (size_t)p.fam_off[KS_NFAM] + (size_t)row] = routed ? 2 : (bnd ? 1 : 0);
      }
      spec_tail<MULT, UNIQ, REST>(p, s, o.t_roof, eta, t, valid, live, row, tfac, fac, dst, u_dst);
    }
    if constexpr (SizedOK<H>::value) {
      // those, in a loop of their own that costs the others no registers
      for (int s = s_lo; rest && s < s_hi; ++s) {
        const SpecC sc = spec_at(p.spec_c, s);
        if (sc.usual && !wide_head) continue;
        const Roof o = small ? roofline<true>(rc, sc) : roofline<false>(rc, sc);
        float x[IN], eta;
        features<IN>(rc, sc, o, x);
        if (bnd) {
          float x16[16];
          features<16>(rc, sc, o, x16);
          eta = bounded_eta(x16, o.W, bnd_lds);
        } else {
          eta = 1.0f + __expf(-H::mlp_f32(x, lds));
        }
        bool routed = false;
        float eta_g = 0.0f;
        if (grd) eta_g = grid_eta(rc, sc, o, p, grid_lds, routed);
        if (routed) eta = eta_g;
        const float t = fmaxf(o.t_roof * eta, sc.t0);
        if constexpr (GRID && !UNIQ) {
          if (valid && p.o_src) p.o_src[(size_t)s * (size_t)p.fam_off[KS_NFAM] + (size_t)row] = routed ? 2 : (bnd ? 1 : 0);
        }
        spec_tail<MULT, UNIQ, REST>(p, s, o.t_roof, eta, t, valid, live, row, tfac, fac, dst, u_dst);
      }
    }
  }
}

// ------------------------------------------------------------ eta = 1 stream
// The pure roofline (eta = 1, Eq. 2), or the bounded head on its families,
// for every (spec, record) pair: its per-pair outputs and/or the step sums
// (Sec. 5.7).  A wave takes a workgroup tile on its own (256 consecutive
// records of one family: four 64-record tiles) and each lane four
// consecutive records of it, so that each 16-lane DPP row holds exactly one
// 64-record tile.  A lane loads its four records of a field with one
// 16-byte load, so the wave's load of a field covers the tile's 1 KB
// contiguously.  Per spec a lane writes its four records' per-pair outputs
// as one vector store each, and sums their t in runs of equal step (one FMA
// each); one
// segmented scan per row then joins the lanes' last runs, and each run's
// tail record adds the carry-in of the lanes before it.  The cross-lane
// work is thus per four records instead of per record.  Runs are split at
// the 64-record tile boundaries as in k_eval, and the partial sums, carries
// and record ranges are the ones k_eval writes, so k_finish reads either
// alike.
constexpr int kStreamR = 4;                       // records per lane
static_assert(kWave * kStreamR == kWgRows, "a wave of the stream takes one workgroup tile");
static_assert(kTileRows == 16 * kStreamR, "a 64-record tile is one 16-lane row");

// what a launch of the stream computes: step sums, per-pair outputs, and
// whether records carry multiplicities (step sums only)
enum : int { kStrSums = 1, kStrPair = 2, kStrMult = 4, kStrBnd = 8 };

// The bounded analytical head in the stream (families with their bounded
// bit; the others keep eta = 1).  Its two logits g . x and a . x are split
// into the spec-independent features (x0, x8 .. x15: one partial sum per
// record and logit, formed once per tile) and the spec-dependent ones (x1 ..
// x7, per spec); the parameters are read through the scalar cache.
struct SBnd {
  float zg[kStreamR], za[kStreamR];   // g . x and a . x over x0, x8 .. x15
  float la[kStreamR];                 // log2(F / max(Bt, 1))
  float bf[kStreamR];                 // B
  float rb[kStreamR];                 // 1 / max(B, 1)
  float rbt[kStreamR];                // 1 / max(Bt, 1)
};

__device__ __forceinline__ float bnd_param(const float *base, int i) {
#if defined(__HIP_DEVICE_COMPILE__)
  typedef const __attribute__((address_space(4))) float *CPtr;
  return ((CPtr)base)[i];
#else
  return base[i];
#endif
}

// fields a family's counts read besides step and n
constexpr bool uses_m(int fam) {
  return fam != KS_GROUPED_GEMM && fam != KS_ATTN_PREFILL && fam != KS_ATTN_DECODE;
}
constexpr bool uses_k(int fam) { return fam != KS_RMSNORM && fam != KS_SILU_MUL && fam != KS_EMBED; }
constexpr bool uses_a(int fam) {
  return fam == KS_GROUPED_GEMM || fam == KS_ATTN_PREFILL || fam == KS_ATTN_DECODE;
}
constexpr bool uses_b(int fam) { return fam == KS_GROUPED_GEMM; }
constexpr bool uses_field(int fam, int f) {
  return f == 0 || f == 2 || (f == 1 && uses_m(fam)) || (f == 3 && uses_k(fam)) || (f == 4 && uses_a(fam)) ||
         (f == 5 && uses_b(fam));
}
// a workgroup tile of the stream: family, first row, valid rows, first tile id
struct STile {
  int fam, nvalid, tile0;
  int64_t row0;
  bool hp, hn;   // a record of the family exists just before / after it
};

// workgroup tile wt, one of family fam's
__device__ __forceinline__ STile stream_locate(const EvalParams &p, int wt, int fam) {
  STile t;
  const int in_fam = wt - p.wgt_off[fam];
  const int64_t lo = p.fam_off[fam], hi = p.fam_off[fam + 1];
  t.fam = fam;
  t.row0 = lo + (int64_t)in_fam * kWgRows;
  const int64_t left = hi - t.row0;
  t.nvalid = left < kWgRows ? (int)left : kWgRows;
  t.tile0 = p.tile_off[fam] + in_fam * kWgWaves;
  t.hp = in_fam > 0;
  t.hn = left > kWgRows;
  return t;
}

// Inclusive segmented scan within each 16-lane row (row_shr 1, 2, 4, 8):
// v += g[i] * v[lane - 2^i], g[i] = 1 where that lane's key is this lane's
// (keys sorted, so the lanes between share it too).  Lanes without a source
// in the row read 0 (bound_ctrl) or are left out by the bank mask.
__device__ __forceinline__ float row_scan(float v, const float (&g)[4]) {
  asm volatile(
      "s_nop 1\n"
      "v_fmac_f32_dpp %0, %0, %1 row_shr:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
      "s_nop 1\n"
      "v_fmac_f32_dpp %0, %0, %2 row_shr:2 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
      "s_nop 1\n"
      "v_fmac_f32_dpp %0, %0, %3 row_shr:4 row_mask:0xf bank_mask:0xe\n"
      "s_nop 1\n"
      "v_fmac_f32_dpp %0, %0, %4 row_shr:8 row_mask:0xf bank_mask:0xc\n"
      : "+v"(v)
      : "v"(g[0]), "v"(g[1]), "v"(g[2]), "v"(g[3]));
  return v;
}

// Block counts below 2^22: the wave count W = ceil(B / N) in fp32 as the
// ceiling of (B - 1/2) fl(1/N).  B - 1/2 is exact, and the two roundings
// move the quotient by at most (B/N) (2^-23 + 2^-48) < 1/(2N), while
// (B - 1/2)/N lies at least 1/(2N) away from every integer (B and N are
// integers), so the ceiling is exact.
constexpr uint32_t kStreamSmallB = 1u << 22;

// What the spec loop needs of a lane's four records besides their roofline
// operands.  Runs never mix live and other records (those carry key
// kNoKey), so the t of a record that is not live never reaches a stored
// sum and needs no masking.  Per-record flags are bits of one word (bit j:
// record j) so that they take one register rather than a lane mask each.
struct SRec {
  uint32_t key[kStreamR];
  float fj[kStreamR];      // 1: record j continues the run of record j - 1
  float mf[kStreamR];      // the record's multiplicity (step sums with multiplicities)
  uint32_t off[kStreamR];  // with 32-bit offsets: byte offset of record j's sum slot from the spec-0 partial
  uint32_t ptail;          // bit j: record j ends a run within its 64-record tile
  uint32_t to_carry;       // bit j: ... and that run continues from the previous tile
  uint32_t first;          // bit j: record j is in the lane's first run
  float g[4], fc;          // row-scan factors; the lane's first run continues the lane before
  int tile;
};

// A family starts at any record, so its quads are 16-byte accesses at 4-byte
// alignment, which global memory takes (a wave's access is contiguous; off
// alignment it touches one more cache line).  One access per record for the
// families off 16-byte alignment, nine of ten in a trace with an odd number of
// steps, took 176 us where this takes 132 (t_kernel of 28.9M records for two
// specs; 126 and 124 at 40,000 steps), all outputs for eight specs 251 and 175.
typedef uint32_t u32x4_any __attribute__((ext_vector_type(4), aligned(4)));
typedef float f32x4_any __attribute__((ext_vector_type(4), aligned(4)));

// a lane's four consecutive records (4 lane .. 4 lane + 3 of the tile) of
// one field array, base: the tile's first record: one 16-byte load when the
// four are valid, else one load per record with its index clamped to the
// tile's valid rows (nvalid >= 1).
// The 16-byte loads are non-temporal: every record is read once per call.
// (Their address is formed before the branch: formed inside it, it shares
// registers with the other side's loads, whose wait then comes before the
// 16-byte load, and a tile's fourth field waits for its first.  A call of
// 1.33M records for two specs with the bounded head took 30.8 us so, 30.1
// with the address before; 58,872 records for ten specs 13.1 and 12.6 in the
// stream alone.)
__device__ __forceinline__ u32x4 load_quad(const uint32_t *base, int lane, int nvalid) {
  typedef const __attribute__((address_space(1))) u32x4_any *Quad;
  Quad q = (Quad)(reinterpret_cast<const char *>(base) + (uint32_t)(16 * lane));
  asm volatile("" : "+v"(q));
  if (kStreamR * lane + kStreamR - 1 < nvalid) {
    const u32x4_any v = __builtin_nontemporal_load(q);
    return u32x4{v[0], v[1], v[2], v[3]};
  }
  u32x4 r;
#pragma unroll
  for (int j = 0; j < kStreamR; ++j) {
    const int i = kStreamR * lane + j;
    r[j] = base[i < nvalid ? i : nvalid - 1];
  }
  return r;
}

// four consecutive per-pair values of a lane (records 4 lane .. 4 lane + 3
// of the tile) at base + 4 lane (base: the tile's first record, the same
// for the whole wave, so the lane's part is a 32-bit offset): one 16-byte
// store (non-temporal: nothing here reads it back) when all four are valid,
// else one store per valid record
__device__ __forceinline__ void store_quad(float *base, int lane, int nvalid, const float (&v)[kStreamR]) {
  float *q = reinterpret_cast<float *>(reinterpret_cast<char *>(base) + (uint32_t)(16 * lane));
  if (kStreamR * lane + kStreamR - 1 < nvalid) {
    __builtin_nontemporal_store(f32x4_any{v[0], v[1], v[2], v[3]}, reinterpret_cast<f32x4_any *>(q));
  } else {
#pragma unroll
    for (int j = 0; j < kStreamR; ++j)
      if (kStreamR * lane + j < nvalid) q[j] = v[j];
  }
}

// Spec loop.  W = ceil(B / N) as the ceiling of (B - 1/2) / N: in fp32 for
// block counts below 2^22 (as above), else in fp64, exact by the same
// argument below 2^51 (the exact path of k_eval assumes B < 2^52); then
// F u / P = W (F / B) (N / P), the first factor per record and the second
// per spec.  BH: B - 1/2 per record, as float or double; frb, btf: F / B
// and Bt per record.  part: the partials of the tile's family ([step][spec]).
// The sum slots are addressed as the spec's uniform base plus the records'
// 32-bit byte offsets r.off (the launcher takes this kernel for step sums
// only when the partial and carry regions span less than 4 GiB), so a spec
// costs no per-lane address arithmetic.  With one or two specs (BUF) a
// tail's sums are stored after the loop, both specs' in one 16-byte store
// (its slots are adjacent and 16-byte aligned); with more, each spec's as
// it is formed.
template <int VAR, bool BND, bool BUF, class BH>
__device__ __forceinline__ void stream_specs(const EvalParams &p, const STile &tc, int lane, const SRec &r,
                                             const BH (&bh)[kStreamR], const float (&frb)[kStreamR],
                                             const float (&btf)[kStreamR], double *part, bool any_tail,
                                             const SBnd &q, const float *prm) {
  constexpr bool SUMS = (VAR & kStrSums) != 0, PAIR = (VAR & kStrPair) != 0, MULT = (VAR & kStrMult) != 0;
  const size_t n_rows = (size_t)p.fam_off[KS_NFAM];
  // spec s: per-pair outputs, and (SUMS) each record's run sum so far in
  // v: a tail record's v is its stored sum
  auto spec = [&](int s, float (&v)[kStreamR]) {
    const SpecC sc = spec_at(p.spec_c, s);
    const float np = sc.n_f * sc.rcp_p;
    float t[kStreamR], tr[kStreamR], eta[kStreamR];
#pragma unroll
    for (int j = 0; j < kStreamR; ++j) {
      float W;
      if constexpr (sizeof(BH) == sizeof(float))
        W = ceilf(bh[j] * sc.rcp_n);
      else
        W = (float)ceil(bh[j] * sc.rcp_nd);
      const float tc_ = W * (frb[j] * np), tm = btf[j] * sc.rcp_bw;
      tr[j] = fmaxf(tc_, tm);
      if constexpr (BND) {
        // x1 .. x7 of this spec (Sec. 5.3 feature list; u = W N / B, and
        // a record without blocks has u = 1), then the bounded head
#pragma clang fp contract(off)
        const float u = q.bf[j] > 0.0f ? W * sc.n_f * q.rb[j] : 1.0f;   // (1 / B for B >= 1)
        float x[8];
        x[1] = fmaxf(q.la[j] + sc.lr, -20.0f) * (1.0f / 16);
        x[2] = log2f_fast(fmaf(q.bf[j], sc.rcp_n, 1.0f)) * (1.0f / 16);
        x[3] = rcpf(u);
        x[4] = log2f_fast(1.0f + W) * (1.0f / 16);
        x[5] = fminf(1.0f, sc.l2 * q.rbt[j]);
        x[6] = log2f_fast(fmaxf(tr[j] * sc.rcp_t0, 0x1p-20f)) * (1.0f / 16);
        const float den = tc_ + tm;
        x[7] = den > 0.0f ? tc_ * rcpf(den) : 0.0f;
        float zg = q.zg[j], za = q.za[j];
#pragma unroll
        for (int i = 1; i < 8; ++i) {
          zg = fmaf(bnd_param(prm, i), x[i], zg);
          za = fmaf(bnd_param(prm, 16 + i), x[i], za);
        }
        const float w = fmaxf(W, 1.0f);
        const float eg = __expf(-zg), ea = __expf(-za);
        eta[j] = (1.0f + eg) * (w * (1.0f + ea)) * rcpf((w - 1.0f) + w * ea);
        t[j] = fmaxf(tr[j] * eta[j], sc.t0);
      } else {
        eta[j] = 1.0f;
        t[j] = fmaxf(tr[j], sc.t0);
      }
    }
    if constexpr (PAIR) {
      const size_t i0 = (size_t)s * n_rows + (size_t)tc.row0;
      if (p.o_troof) store_quad(p.o_troof + i0, lane, tc.nvalid, tr);
      if (p.o_eta) store_quad(p.o_eta + i0, lane, tc.nvalid, eta);
      if (p.o_t) store_quad(p.o_t + i0, lane, tc.nvalid, t);
    }
    if constexpr (SUMS) {
      float acc[kStreamR];
#pragma unroll
      for (int j = 0; j < kStreamR; ++j) {
        const float x = MULT ? t[j] * r.mf[j] : t[j];
        acc[j] = j == 0 ? x : fmaf(r.fj[j], acc[j - 1], x);
      }
      // the run ending at this lane's last record, over the row's lanes so far
      const float x = row_scan(acc[kStreamR - 1], r.g);
      // what the lanes before add to this lane's first run (0 at a row start)
      const float cin = r.fc * __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(
                                                           0, __builtin_bit_cast(int, x), 0x111, 0xf, 0xf, true));
#pragma unroll
      for (int j = 0; j < kStreamR; ++j) v[j] = ((r.first >> j) & 1u) ? acc[j] + cin : acc[j];
    }
  };
  if constexpr (BUF && SUMS) {
    float v0[kStreamR], v1[kStreamR];
    spec(0, v0);
    const bool two = p.n_specs == 2;
    if (two) spec(1, v1);
    if (any_tail) {
      if (two) {
        typedef double f64x2 __attribute__((ext_vector_type(2)));
#pragma unroll
        for (int j = 0; j < kStreamR; ++j)
          if ((r.ptail >> j) & 1u)
            *reinterpret_cast<f64x2 *>(reinterpret_cast<char *>(part) + r.off[j]) = f64x2{(double)v0[j], (double)v1[j]};
      } else {
#pragma unroll
        for (int j = 0; j < kStreamR; ++j)
          if ((r.ptail >> j) & 1u) *reinterpret_cast<double *>(reinterpret_cast<char *>(part) + r.off[j]) = (double)v0[j];
      }
    }
  } else {
    for (int s = 0; s < p.n_specs; ++s) {
      float v[kStreamR];
      spec(s, v);
      if constexpr (SUMS) {
        if (any_tail) {
#pragma unroll
          for (int j = 0; j < kStreamR; ++j)
            if ((r.ptail >> j) & 1u) *reinterpret_cast<double *>(reinterpret_cast<char *>(part + s) + r.off[j]) = (double)v[j];
        }
      }
    }
  }
}

// the spec loop's instance: bounded head or not, one or two specs (whose
// sums are stored after the loop) or more
template <int VAR, class BH>
__device__ __forceinline__ void stream_dispatch(const EvalParams &p, const STile &tc, int lane, const SRec &r,
                                                const BH (&bh)[kStreamR], const float (&frb)[kStreamR],
                                                const float (&btf)[kStreamR], double *part, bool any_tail,
                                                const SBnd &q, const float *prm, bool bnd) {
  constexpr bool B = (VAR & kStrBnd) != 0;
  if (p.n_specs <= 2) {
    if (bnd)
      stream_specs<VAR, B, true>(p, tc, lane, r, bh, frb, btf, part, any_tail, q, prm);
    else
      stream_specs<VAR, false, true>(p, tc, lane, r, bh, frb, btf, part, any_tail, q, prm);
  } else {
    if (bnd)
      stream_specs<VAR, B, false>(p, tc, lane, r, bh, frb, btf, part, any_tail, q, prm);
    else
      stream_specs<VAR, false, false>(p, tc, lane, r, bh, frb, btf, part, any_tail, q, prm);
  }
}

// A tile's loads: the lane's four records of each field its family uses
// (16 bytes per lane and field, so the wave's load of a field covers the
// tile contiguously; zero for the unused fields), the multiplicities, and
// the steps just before and after the tile (lane 0 and lane 1 of one load;
// each address inside the family: the tile's first row where a neighbour
// does not exist).
struct SLoad {
  u32x4 f[6];
  u32x4 mult;
  uint32_t pn;
};

template <int FAM, int VAR>
__device__ __forceinline__ void stream_load(const EvalParams &p, const STile &t, int lane, SLoad &o) {
  const uint32_t *src[6] = {p.step, p.m, p.n, p.k, p.a, p.b};
#pragma unroll
  for (int f = 0; f < 6; ++f) {
    o.f[f] = u32x4{0, 0, 0, 0};
    if (uses_field(FAM, f)) o.f[f] = load_quad(src[f] + t.row0, lane, t.nvalid);
  }
  if constexpr ((VAR & kStrMult) != 0) o.mult = load_quad(p.mult + t.row0, lane, t.nvalid);
  o.pn = 0;
  if constexpr ((VAR & kStrSums) != 0) {
    const int pn_off = lane == 0 ? (t.hp ? -1 : 0) : (t.hn ? kWgRows : 0);
    o.pn = (p.step + t.row0)[pn_off];
  }
}

// One workgroup tile of family FAM, its loads in `in`; rng and part: the
// family's range table and partials.
template <int FAM, int VAR>
__device__ __forceinline__ void stream_tile(const EvalParams &p, const STile &tc, int lane, uint32_t *rng,
                                            double *part, const SLoad &in) {
  constexpr bool SUMS = (VAR & kStrSums) != 0, PAIR = (VAR & kStrPair) != 0, MULT = (VAR & kStrMult) != 0;
  uint32_t v[6][kStreamR];
#pragma unroll
  for (int f = 0; f < 6; ++f) {
#pragma unroll
    for (int j = 0; j < kStreamR; ++j) v[f][j] = uses_field(FAM, f) ? in.f[f][j] : 0u;
  }
  SRec r;
  if constexpr (MULT) {
#pragma unroll
    for (int j = 0; j < kStreamR; ++j) r.mf[j] = (float)in.mult[j];   // exact below 2^24
  }
  const uint32_t pn = in.pn;

  // per record: counts and the spec-independent roofline operands; exact
  // (u64) when the per-record counts are written, else in fp32
  uint32_t bad = 0;
  bool live[kStreamR];
  bool big = false;
  uint64_t B[kStreamR];
  float Ff[kStreamR], Btf[kStreamR], Mf[kStreamR];
  // a step at or past n_steps (none can be when n_steps >= 2^32)
  const bool lim = p.n_steps <= (int64_t)UINT32_MAX;
  const uint32_t n_steps32 = (uint32_t)p.n_steps;
  const bool exact = PAIR && (p.o_flops || p.o_bytes || p.o_blocks);   // wave-uniform
#pragma unroll
  for (int j = 0; j < kStreamR; ++j) {
    const bool valid = kStreamR * lane + j < tc.nvalid;
    uint32_t b = 0;
    if (lim && v[0][j] >= n_steps32) b |= kErrStep;
    if (PAIR && exact) {
      const Cnt c = record_counts(FAM, v[1][j], v[2][j], v[3][j], v[4][j], v[5][j], v[0][j], p, b);
      if (valid) {
        const size_t row = (size_t)tc.row0 + (size_t)(kStreamR * lane + j);
        if (p.o_flops) p.o_flops[row] = c.F;
        if (p.o_bytes) p.o_bytes[row] = c.Bt;
        if (p.o_blocks) p.o_blocks[row] = c.B;
      }
      B[j] = c.B;
      Ff[j] = (float)c.F;
      Btf[j] = (float)c.Bt;
      Mf[j] = (float)c.M;
    } else {
      const CntF cf = record_counts_f(FAM, v[1][j], v[2][j], v[3][j], v[4][j], v[5][j], v[0][j], p, b);
      B[j] = cf.B;
      Ff[j] = cf.F;
      Btf[j] = cf.Bt;
      Mf[j] = cf.M;
    }
    if (valid) bad |= b;
    live[j] = valid && !(b & kErrStep);
    r.key[j] = live[j] ? v[0][j] : kNoKey;
    big |= B[j] >= kStreamSmallB;
  }
  if (bad) atomicOr(p.err, bad);
  const bool small = __ballot(big) == 0;   // wave-uniform

  bool any_tail = false;
  if constexpr (SUMS) {
    const uint32_t prev = tc.hp ? __builtin_amdgcn_readlane(pn, 0) : kNoKey;
    const uint32_t next = tc.hn ? __builtin_amdgcn_readlane(pn, 1) : kNoKey;
    // neighbours: the record before this lane's first (lane 0: the tile
    // edge) and after its last (lane 63: the tile edge)
    const uint32_t kp =
        (uint32_t)__builtin_amdgcn_update_dpp((int)prev, (int)r.key[kStreamR - 1], 0x138, 0xf, 0xf, false);
    const uint32_t kn = (uint32_t)__builtin_amdgcn_update_dpp((int)next, (int)r.key[0], 0x130, 0xf, 0xf, false);
    const int row_lane = lane & 15;
    r.tile = tc.tile0 + (lane >> 4);
    // the key of the row's first record and of the record before the row
    // (row_newbcast:0 gives each row its lane 0)
    const uint32_t rk0 = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)r.key[0], 0x150, 0xf, 0xf, false);
    const uint32_t rkp = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)kp, 0x150, 0xf, 0xf, false);
    r.ptail = r.to_carry = r.first = 0;
    uint32_t heads = 0, ends = 0;   // bit j: record j starts / ends its (family, step) range
#pragma unroll
    for (int j = 0; j < kStreamR; ++j) {
      const uint32_t key = r.key[j];
      const uint32_t before = j == 0 ? kp : r.key[j - 1];
      const uint32_t after = j == kStreamR - 1 ? kn : r.key[j + 1];
      r.fj[j] = j > 0 && key == before ? 1.0f : 0.0f;
      heads |= (live[j] && before != key ? 1u : 0u) << j;
      ends |= (live[j] && after != key ? 1u : 0u) << j;
      // a run's last record within its 64-record tile
      const bool pt = live[j] && (after != key || (j == kStreamR - 1 && row_lane == 15));
      r.ptail |= (pt ? 1u : 0u) << j;
      r.to_carry |= (key == rk0 && rkp == rk0 ? 1u : 0u) << j;
      r.first |= (key == r.key[0] ? 1u : 0u) << j;
    }
    // the (family, step) record range, written where its global first and
    // last records are
    const uint32_t row_l = (uint32_t)tc.row0 + (uint32_t)(kStreamR * lane);
#pragma unroll
    for (int j = 0; j < kStreamR; ++j) {
      if ((heads >> j) & 1u) rng[2 * (size_t)r.key[j]] = row_l + j;
      if ((ends >> j) & 1u) rng[2 * (size_t)r.key[j] + 1] = row_l + j + 1;
    }
    any_tail = __ballot(r.ptail != 0) != 0;
    {
      // carries lie after the partials: their offset from this family's
      // partials is (carry - part) + tile S 8
      const uint32_t S8 = (uint32_t)p.n_specs * 8u;
      const uint32_t cbase = (uint32_t)((const char *)p.carry - (const char *)part) + (uint32_t)r.tile * S8;
#pragma unroll
      for (int j = 0; j < kStreamR; ++j) r.off[j] = ((r.to_carry >> j) & 1u) ? cbase : r.key[j] * S8;
    }
    r.fc = row_lane != 0 && kp == r.key[0] ? 1.0f : 0.0f;
    // row-scan factors on the lanes' last keys
    const uint32_t kl = r.key[kStreamR - 1];
    r.g[0] = dpp_key<0x111, 0xf, 0xf>(kl) == kl ? 1.0f : 0.0f;
    r.g[1] = dpp_key<0x112, 0xf, 0xf>(kl) == kl ? 1.0f : 0.0f;
    r.g[2] = dpp_key<0x114, 0xf, 0xe>(kl) == kl ? 1.0f : 0.0f;
    r.g[3] = dpp_key<0x118, 0xf, 0xc>(kl) == kl ? 1.0f : 0.0f;
  }
  // the bounded head's spec-independent part (families with their bit set)
  SBnd q;
  const float *prm = nullptr;
  const bool bnd = (VAR & kStrBnd) != 0 && ((p.bounded_mask >> FAM) & 1u);   // wave-uniform
  if constexpr ((VAR & kStrBnd) != 0) {
    if (bnd) {
      prm = p.bounded + FAM * 32;
      // read the parameters again in each tile rather than hold them in
      // scalar registers across the family's tiles
      asm volatile("" : "+s"(prm));
#pragma unroll
      for (int j = 0; j < kStreamR; ++j) {
#pragma clang fp contract(off)
        const float bf = (float)B[j];
        const float rb = rcpf(fmaxf(bf, 1.0f));
        q.bf[j] = bf;
        q.rb[j] = rb;
        q.rbt[j] = rcpf(fmaxf(Btf[j], 1.0f));
        // log2(0) = -inf for F = 0; the clamps of x0 and x1 take it
        q.la[j] = log2f_fast(Ff[j] * q.rbt[j]);
        float xi[9];
        xi[0] = fmaxf(q.la[j], -10.0f) * (1.0f / 16);
        xi[1] = log2f_fast(1.0f + Ff[j]) * (1.0f / 64);
        xi[2] = log2f_fast(1.0f + Btf[j]) * (1.0f / 48);
        xi[3] = log2f_fast(1.0f + Mf[j]) * (1.0f / 24);
        xi[4] = log2f_fast(1.0f + (float)v[2][j]) * (1.0f / 24);
        xi[5] = log2f_fast(1.0f + (float)v[3][j]) * (1.0f / 24);   // 0 for the families without K
        xi[6] = log2f_fast(1.0f + Ff[j] * rb) * (1.0f / 48);
        xi[7] = log2f_fast(1.0f + Btf[j] * rb) * (1.0f / 40);
        xi[8] = 1.0f;
        // x0, x8 .. x15 of the feature list: parameter indices 0, 8 .. 15
        float zg = bnd_param(prm, 0) * xi[0], za = bnd_param(prm, 16) * xi[0];
#pragma unroll
        for (int i = 1; i < 9; ++i) {
          zg = fmaf(bnd_param(prm, 7 + i), xi[i], zg);
          za = fmaf(bnd_param(prm, 23 + i), xi[i], za);
        }
        q.zg[j] = zg;
        q.za[j] = za;
      }
    }
  }
  float frb[kStreamR];
  if (small) {
    float bh[kStreamR];
#pragma unroll
    for (int j = 0; j < kStreamR; ++j) {
      const float Bf = (float)(uint32_t)B[j];
      bh[j] = Bf - 0.5f;
      frb[j] = Ff[j] * rcpf(fmaxf(Bf, 1.0f));
    }
    stream_dispatch<VAR>(p, tc, lane, r, bh, frb, Btf, part, any_tail, q, prm, bnd);
  } else {
    double bh[kStreamR];
#pragma unroll
    for (int j = 0; j < kStreamR; ++j) {
      bh[j] = (double)B[j] - 0.5;
      frb[j] = Ff[j] * rcpf(fmaxf((float)B[j], 1.0f));
    }
    stream_dispatch<VAR>(p, tc, lane, r, bh, frb, Btf, part, any_tail, q, prm, bnd);
  }
}

// Waves per SIMD the register allocator must fit, at least: six for the
// plain step sums (seven spills and measured slower); the other variants
// take what their registers allow.
template <int VAR> struct StreamOcc {
  static constexpr int value =
      VAR == kStrSums ? 6 : ((VAR & kStrBnd) && (VAR & kStrSums) && (VAR & kStrPair) ? 3 : 4);
};

// The wave's tiles of family FAM, from tile wt on in steps of stride (wt
// advances past them).  Looping over one family at a time keeps the
// family's constants and code out of the other families' loops (fewer live
// registers than dispatching on the family per tile); issuing a tile's
// loads a tile ahead measured no faster.
template <int FAM, int VAR>
__device__ __forceinline__ void stream_family(const EvalParams &p, int &wt, int stride, int lane) {
  const int end = p.wgt_off[FAM + 1];
  if (wt >= end) return;
  uint32_t *rng = nullptr;
  double *part = nullptr;
  if constexpr ((VAR & kStrSums) != 0) {
    rng = p.range + 2 * (size_t)FAM * (size_t)p.n_steps;
    part = p.partial + (size_t)FAM * (size_t)p.n_steps * (size_t)p.n_specs;
  }
  for (; wt < end; wt += stride) {
    const STile t = stream_locate(p, wt, FAM);
    SLoad in;
    stream_load<FAM, VAR>(p, t, lane, in);
    stream_tile<FAM, VAR>(p, t, lane, rng, part, in);
  }
}

template <int VAR>
__global__ __launch_bounds__(kWgThreads) __attribute__((amdgpu_waves_per_eu(StreamOcc<VAR>::value)))
void k_stream(EvalParams p) {
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int stride = (int)gridDim.x * kWgWaves;
  // Workgroups go to the eight XCDs round-robin (workgroup b to XCD b mod
  // 8).  With step sums they are renumbered so that each XCD takes one
  // contiguous eighth of the tiles of every pass over the grid: the partial
  // sums and record ranges of consecutive steps (several to a cache line)
  // are then written from one XCD's L2 instead of up to eight, each holding
  // a partial line (per-pair outputs alone measured faster without it).
  int b = (int)blockIdx.x;
  if ((VAR & kStrSums) != 0 && (gridDim.x & 7u) == 0u) b = (b & 7) * (int)(gridDim.x >> 3) + (b >> 3);
  int wt = b * kWgWaves + wave;
  stream_family<KS_GEMM, VAR>(p, wt, stride, lane);
  stream_family<KS_LM_HEAD, VAR>(p, wt, stride, lane);
  stream_family<KS_GROUPED_GEMM, VAR>(p, wt, stride, lane);
  stream_family<KS_ATTN_PREFILL, VAR>(p, wt, stride, lane);
  stream_family<KS_ATTN_DECODE, VAR>(p, wt, stride, lane);
  stream_family<KS_RMSNORM, VAR>(p, wt, stride, lane);
  stream_family<KS_ROPE, VAR>(p, wt, stride, lane);
  stream_family<KS_SILU_MUL, VAR>(p, wt, stride, lane);
  stream_family<KS_KV_WRITE, VAR>(p, wt, stride, lane);
  stream_family<KS_EMBED, VAR>(p, wt, stride, lane);
  static_assert(KS_EMBED == KS_NFAM - 1, "every family has its loop");
}

#if KS_HEADS == 0
// ------------------------------------------------------------ record counts
// The exact counts of the records whose latency another record's evaluation
// gave (the families of uniq_mask): HBM-bound, a row per thread.
__global__ void k_counts(EvalParams p) {
  const int64_t n_rows = p.fam_off[KS_NFAM];
  int f = 0;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n_rows; i += (int64_t)gridDim.x * blockDim.x) {
    while (i >= p.fam_off[f + 1]) ++f;
    if (!((p.uniq_mask >> f) & 1u) || p.u_over[f]) continue;
    const bool attn = f == KS_ATTN_PREFILL || f == KS_ATTN_DECODE;
    uint32_t bad = 0;
    const Cnt c = record_counts(f, attn ? 0u : p.m[i], p.n[i], uses_k(f) ? p.k[i] : 0u, attn ? p.a[i] : 0u, 0u,
                                attn ? p.step[i] : 0u, p, bad);
    if (p.o_flops) p.o_flops[i] = c.F;
    if (p.o_bytes) p.o_bytes[i] = c.Bt;
    if (p.o_blocks) p.o_blocks[i] = c.B;
  }
}

// ------------------------------------------------------------ eta source
// Per pair, where eta came from when no grid routes any pair: 1 for the
// families on the bounded head, 0 (the head of the mode) for the others.
__global__ void k_fill_source(uint8_t *src, EvalParams p) {
  const int64_t n_rows = p.fam_off[KS_NFAM];
  const int64_t total = (int64_t)p.n_specs * n_rows;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < total;
       i += (int64_t)gridDim.x * blockDim.x) {
    const int64_t row = i % n_rows;
    int f = 0;
    while (row >= p.fam_off[f + 1]) ++f;
    src[i] = (uint8_t)((p.bounded_mask >> f) & 1u);
  }
}
#endif

#if KS_HEADS == 0
// ------------------------------------------------------------ validation
__global__ void k_validate(ValidateParams p) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  const int64_t t0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  uint32_t bad = 0;
  for (int64_t i = t0; i < p.n_rows; i += stride) {
    int f = 0;
    while (i >= p.fam_off[f + 1]) ++f;
    const uint32_t st = p.step[i];
    if ((int64_t)st >= p.n_steps) bad |= kErrStep;
    if (i > p.fam_off[f] && p.step[i - 1] > st) bad |= kErrOrder;
    const uint32_t m = p.m[i], n = p.n[i], k = p.k[i], a = p.a[i], b = p.b[i];
    if (m >= (1u << 24) || n >= (1u << 18) || k >= (1u << 18)) bad |= kErrRange;
    if (p.mult && p.mult[i] >= (1u << 24)) bad |= kErrRange;
    if ((f == KS_ATTN_PREFILL || f == KS_ATTN_DECODE) && (n >= 4096u || k >= 4096u || a >= 4096u))
      bad |= kErrRange;
    if (f == KS_GROUPED_GEMM) {
      if (a > 1024u || (uint64_t)b + a > (uint64_t)p.n_expert_rows) {
        bad |= kErrExpert;
      } else {
        uint64_t ms, act, tiles;
        expert_sums(p.expert_rows, b, a, ms, act, tiles);
        if (ms >= (1ull << 24)) bad |= kErrRange;
      }
    }
  }
  for (int64_t j = t0; j < p.n_steps; j += stride) {
    if (p.req_off[j] > p.req_off[j + 1] || (int64_t)p.req_off[j + 1] > p.n_req) bad |= kErrReq;
    if (p.agg[2 * p.n_steps + j] >= (1ull << 40)) bad |= kErrRange;
    if (p.tp && p.tp[j] < 1u) bad |= kErrRange;
  }
  if (t0 == 0 && p.n_steps > 0 && p.req_off[0] != 0) bad |= kErrReq;
  for (int64_t r = t0; r < p.n_req; r += stride)
    if (p.req_q[r] >= (1u << 24) || p.req_h[r] >= (1u << 24)) bad |= kErrRange;
  for (int64_t s = t0; s < p.n_specs; s += stride) {
    const ks_spec sp = p.specs[s];
    const bool ok = sp.peak_flops > 0.0 && sp.peak_flops < 1e30 && sp.hbm_bw > 0.0 && sp.hbm_bw < 1e30 &&
                    sp.t0 >= 0.0 && sp.t0 < 1e3 && sp.l2_bytes >= 0.0 && sp.l2_bytes < 1e30 &&
                    sp.ar_beta > 0.0 && sp.ar_beta < 1e30 && sp.ar_alpha0 >= 0.0 && sp.ar_alpha0 < 1e3 &&
                    sp.ar_alpha_log2p >= 0.0 && sp.ar_alpha_log2p < 1e3 && sp.n_cu >= 1u && sp.n_cu <= 65535u;
    if (!ok) bad |= kErrSpec;
  }
  if (bad) atomicOr(p.err, bad);
}
#endif

// ------------------------------------------------------------ launchers
// The persistent grid: as many workgroups as are resident at once (the
// occupancy the compiled kernel's registers and LDS allow, times the CU
// count), so no workgroup of the head kinds waits for another to finish.
// Cached per device and kernel.
constexpr int kMaxDevices = 64;
static std::atomic<int> g_resident[kMaxDevices][kNumKinds][kNumVars];

template <int KIND, int VAR>
static hipError_t resident_wgs(int *out) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  std::atomic<int> *slot = dev < kMaxDevices ? &g_resident[dev][KIND][VAR] : nullptr;
  int r = slot ? slot->load(std::memory_order_relaxed) : 0;
  if (r == 0) {
    int per_cu = 0, n_cu = 0;
    e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_eval<KIND, VAR>, kWgThreads, 0);
    if (e != hipSuccess) return e;
    e = hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, dev);
    if (e != hipSuccess) return e;
    r = (per_cu < 1 ? 1 : per_cu) * (n_cu < 1 ? 1 : n_cu);
    if (slot) slot->store(r, std::memory_order_relaxed);
  }
  *out = r;
  return hipSuccess;
}

template <int KIND, int VAR>
static hipError_t launch_grid(const EvalParams &p, hipStream_t s) {
  int cap = 0;
  const hipError_t e = resident_wgs<KIND, VAR>(&cap);
  if (e != hipSuccess) return e;
  const int n_wgt = p.wgt_off[KS_NFAM];
  // Too few record tiles to fill the GPU (e.g. one serving round of many
  // spec vectors): split the spec loop into ranges, each a work item of its
  // own, so that ranges of the same tile run on different CUs.  The sums
  // and outputs of different specs are disjoint; the record ranges are
  // written alike by every range.
  EvalParams q = p;
  q.spec_chunk = p.n_specs;
  q.n_chunks = 1;
  if (n_wgt < 4 * cap && p.n_specs > 1) {
    q.n_chunks = spec_ranges(n_wgt, cap, p.n_specs);
    q.spec_chunk = (p.n_specs + q.n_chunks - 1) / q.n_chunks;
  }
  const int64_t work = (int64_t)n_wgt * q.n_chunks;
  const int grid = work < cap ? (int)work : cap;
  hipLaunchKernelGGL((k_eval<KIND, VAR>), dim3(grid), dim3(kWgThreads), 0, s, q);
  return hipGetLastError();
}

template <int KIND>
hipError_t launch_kind(const EvalParams &p, hipStream_t s) {
  // multiplicities matter only for the step sums
  const bool mult = p.mult && p.partial;
  if (p.grid_mask)
    return mult ? launch_grid<KIND, kVarGrid | kVarMult>(p, s) : launch_grid<KIND, kVarGrid>(p, s);
  return mult ? launch_grid<KIND, kVarMult>(p, s) : launch_grid<KIND, 0>(p, s);
}

template <int KIND, int VAR>
static hipError_t launch_uniq_var(const EvalParams &p, hipStream_t s) {
  int cap = 0;
  const hipError_t e = resident_wgs<KIND, VAR>(&cap);
  if (e != hipSuccess) return e;
  // (how much work there is is known on the device only: workgroups without
  // any leave at once)
  const int64_t most = (int64_t)p.wgt_off[KS_NFAM] * p.n_specs;
  hipLaunchKernelGGL((k_eval<KIND, VAR>), dim3((unsigned)(most < cap ? most : cap)), dim3(kWgThreads), 0, s, p);
  return hipGetLastError();
}

template <int KIND>
hipError_t launch_uniq(const EvalParams &p, hipStream_t s) {
  if (p.uniq->rest)
    return p.grid_mask ? launch_uniq_var<KIND, kVarUniq | kVarRest | kVarGrid>(p, s)
                       : launch_uniq_var<KIND, kVarUniq | kVarRest>(p, s);
  return p.grid_mask ? launch_uniq_var<KIND, kVarUniq | kVarGrid>(p, s) : launch_uniq_var<KIND, kVarUniq>(p, s);
}

// This file is compiled once per KS_HEADS (in parallel): 1 the fp32 heads, 2 the
// bf16 heads up to hidden 128, 3 those of 256, 0 everything else.
#if KS_HEADS == 1
template hipError_t launch_kind<kF32_16_64>(const EvalParams &, hipStream_t);
template hipError_t launch_uniq<kF32_16_64>(const EvalParams &, hipStream_t);
template hipError_t launch_kind<kF32_16_128>(const EvalParams &, hipStream_t);
template hipError_t launch_uniq<kF32_16_128>(const EvalParams &, hipStream_t);
template hipError_t launch_kind<kF32_32_64>(const EvalParams &, hipStream_t);
template hipError_t launch_uniq<kF32_32_64>(const EvalParams &, hipStream_t);
template hipError_t launch_kind<kF32_32_128>(const EvalParams &, hipStream_t);
template hipError_t launch_uniq<kF32_32_128>(const EvalParams &, hipStream_t);
#endif
#if KS_HEADS == 2
template hipError_t launch_kind<kBF16_16_64>(const EvalParams &, hipStream_t);
template hipError_t launch_uniq<kBF16_16_64>(const EvalParams &, hipStream_t);
template hipError_t launch_kind<kBF16_16_128>(const EvalParams &, hipStream_t);
template hipError_t launch_uniq<kBF16_16_128>(const EvalParams &, hipStream_t);
template hipError_t launch_kind<kBF16_32_64>(const EvalParams &, hipStream_t);
template hipError_t launch_uniq<kBF16_32_64>(const EvalParams &, hipStream_t);
template hipError_t launch_kind<kBF16_32_128>(const EvalParams &, hipStream_t);
template hipError_t launch_uniq<kBF16_32_128>(const EvalParams &, hipStream_t);
#endif
#if KS_HEADS == 3
template hipError_t launch_kind<kBF16_16_256>(const EvalParams &, hipStream_t);
template hipError_t launch_uniq<kBF16_16_256>(const EvalParams &, hipStream_t);
template hipError_t launch_kind<kBF16_32_256>(const EvalParams &, hipStream_t);
template hipError_t launch_uniq<kBF16_32_256>(const EvalParams &, hipStream_t);
#endif
#if KS_HEADS == 0
extern template hipError_t launch_kind<kF32_16_64>(const EvalParams &, hipStream_t);
extern template hipError_t launch_uniq<kF32_16_64>(const EvalParams &, hipStream_t);
extern template hipError_t launch_kind<kF32_16_128>(const EvalParams &, hipStream_t);
extern template hipError_t launch_uniq<kF32_16_128>(const EvalParams &, hipStream_t);
extern template hipError_t launch_kind<kF32_32_64>(const EvalParams &, hipStream_t);
extern template hipError_t launch_uniq<kF32_32_64>(const EvalParams &, hipStream_t);
extern template hipError_t launch_kind<kF32_32_128>(const EvalParams &, hipStream_t);
extern template hipError_t launch_uniq<kF32_32_128>(const EvalParams &, hipStream_t);
extern template hipError_t launch_kind<kBF16_16_64>(const EvalParams &, hipStream_t);
extern template hipError_t launch_uniq<kBF16_16_64>(const EvalParams &, hipStream_t);
extern template hipError_t launch_kind<kBF16_16_128>(const EvalParams &, hipStream_t);
extern template hipError_t launch_uniq<kBF16_16_128>(const EvalParams &, hipStream_t);
extern template hipError_t launch_kind<kBF16_32_64>(const EvalParams &, hipStream_t);
extern template hipError_t launch_uniq<kBF16_32_64>(const EvalParams &, hipStream_t);
extern template hipError_t launch_kind<kBF16_32_128>(const EvalParams &, hipStream_t);
extern template hipError_t launch_uniq<kBF16_32_128>(const EvalParams &, hipStream_t);
extern template hipError_t launch_kind<kBF16_16_256>(const EvalParams &, hipStream_t);
extern template hipError_t launch_uniq<kBF16_16_256>(const EvalParams &, hipStream_t);
extern template hipError_t launch_kind<kBF16_32_256>(const EvalParams &, hipStream_t);
extern template hipError_t launch_uniq<kBF16_32_256>(const EvalParams &, hipStream_t);

static int grid_for(int64_t n, int block, int cap) {
  int64_t g = (n + block - 1) / block;
  if (g < 1) g = 1;
  return (int)(g < cap ? g : cap);
}

hipError_t launch_clear(uint32_t *err, uint32_t *range, int64_t n_range, hipStream_t s) {
  hipLaunchKernelGGL(k_clear, dim3(grid_for(n_range, 256, 2048)), dim3(256), 0, s, err, range, n_range,
                     (const ks_spec *)nullptr, 0, (SpecC *)nullptr);
  return hipGetLastError();
}

hipError_t launch_attn_agg(const uint32_t *req_off, const uint32_t *q, const uint32_t *h, int64_t n_steps,
                           int64_t n_req, uint64_t *agg, uint32_t *err, hipStream_t s) {
  if (n_steps == 0) return hipSuccess;
  hipLaunchKernelGGL(k_attn_agg, dim3(grid_for(n_steps, 256 / kAggLanes, 8192)), dim3(256), 0, s, req_off, q, h,
                     n_steps, n_req, agg, err);
  return hipGetLastError();
}

hipError_t launch_spec_prep(const ks_spec *specs, int32_t n_specs, SpecC *out, uint32_t *err, hipStream_t s) {
  hipLaunchKernelGGL(k_spec_prep, dim3(grid_for(n_specs, 256, 4096)), dim3(256), 0, s, specs, n_specs, out, err);
  return hipGetLastError();
}

// up to this many specs the clear kernel's first workgroup forms the spec
// constants (one launch less); more take their own grid
constexpr int32_t kFusedSpecs = 1024;

hipError_t launch_prologue(uint32_t *err, uint32_t *range, int64_t n_range, const ks_spec *specs, int32_t n_specs,
                           SpecC *out, const uint32_t *req_off, const uint32_t *q, const uint32_t *h, int64_t n_steps,
                           int64_t n_req, uint64_t *agg, hipStream_t s) {
  hipLaunchKernelGGL(k_prologue, dim3(1), dim3(kPrologueThreads), 0, s, err, range, n_range, specs, n_specs, out, req_off,
                     q, h, n_steps, n_req, agg);
  return hipGetLastError();
}

hipError_t launch_clear_prep(uint32_t *err, uint32_t *range, int64_t n_range, const ks_spec *specs,
                             int32_t n_specs, SpecC *out, hipStream_t s) {
  const bool fused = n_specs <= kFusedSpecs;
  hipLaunchKernelGGL(k_clear, dim3(grid_for(n_range, 256, 2048)), dim3(256), 0, s, err, range, n_range, specs,
                     fused ? n_specs : 0, out);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || fused) return e;
  return launch_spec_prep(specs, n_specs, out, err, s);
}

// k_stream: every eta = 1 evaluation (per-pair outputs and/or step sums,
// with or without multiplicities); grid-stride over workgroup tiles, one
// per wave.  As many workgroups as are resident, cached per device and
// variant.
constexpr int kNumStreamVars = 16;
// Workgroups per CU of a variant, at most (0: as many as are resident):
// the per-pair outputs alone fit seven waves per SIMD in registers and
// measured faster at five.
template <int VAR> struct StreamWgCap {
  static constexpr int value = VAR == kStrPair ? 5 : 0;
};
static std::atomic<int> g_stream_resident[kMaxDevices][kNumStreamVars];

template <int VAR>
static hipError_t launch_stream(const EvalParams &p, hipStream_t s) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  std::atomic<int> *slot = dev < kMaxDevices ? &g_stream_resident[dev][VAR] : nullptr;
  int cap = slot ? slot->load(std::memory_order_relaxed) : 0;
  if (cap == 0) {
    int per_cu = 0, n_cu = 0;
    e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_stream<VAR>, kWgThreads, 0);
    if (e != hipSuccess) return e;
    e = hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, dev);
    if (e != hipSuccess) return e;
    if (StreamWgCap<VAR>::value > 0 && per_cu > StreamWgCap<VAR>::value) per_cu = StreamWgCap<VAR>::value;
    cap = (per_cu < 1 ? 1 : per_cu) * (n_cu < 1 ? 1 : n_cu);
    if (slot) slot->store(cap, std::memory_order_relaxed);
  }
  const int n_wgt = p.wgt_off[KS_NFAM];
  const int need = (n_wgt + kWgWaves - 1) / kWgWaves;
  hipLaunchKernelGGL((k_stream<VAR>), dim3(need < cap ? need : cap), dim3(kWgThreads), 0, s, p);
  return hipGetLastError();
}

// eta = 1 (no bounded or grid family: those select the head-less kind)
static hipError_t launch_eta_one(const EvalParams &p, hipStream_t s) {
  if (p.grid_mask || p.bounded_mask) return hipErrorInvalidValue;
  // the stream addresses the sum slots by 32-bit offsets from the partials:
  // step sums whose partial and carry regions (carries after partials) span
  // 4 GiB or more take the one-record-per-lane kernel instead (its
  // head-less kind without bounded or grid families is eta = 1)
  if (p.partial) {
    const bool after = p.carry > p.partial;
    const uint64_t span = after ? (uint64_t)((const char *)p.carry - (const char *)p.partial) +
                                      (uint64_t)p.n_tiles * (uint64_t)p.n_specs * sizeof(double)
                                : ~0ull;
    if (span >= (1ull << 32)) return launch_kind<kBoundedOnly>(p, s);
  }
  const bool sums = p.partial && p.range;
  const bool pair = p.o_flops || p.o_bytes || p.o_blocks || p.o_troof || p.o_eta || p.o_t;
  // multiplicities matter only for the step sums
  const bool mult = sums && p.mult;
  if (!sums) return launch_stream<kStrPair>(p, s);
  if (mult) return pair ? launch_stream<kStrSums | kStrPair | kStrMult>(p, s) : launch_stream<kStrSums | kStrMult>(p, s);
  return pair ? launch_stream<kStrSums | kStrPair>(p, s) : launch_stream<kStrSums>(p, s);
}

// no MLP family and no grid: the bounded families and eta = 1 for the rest,
// on the stream (same 4 GiB condition for the sum slots)
static hipError_t launch_bounded_stream(const EvalParams &p, hipStream_t s) {
  if (p.partial) {
    const bool after = p.carry > p.partial;
    const uint64_t span = after ? (uint64_t)((const char *)p.carry - (const char *)p.partial) +
                                      (uint64_t)p.n_tiles * (uint64_t)p.n_specs * sizeof(double)
                                : ~0ull;
    if (span >= (1ull << 32)) return launch_kind<kBoundedOnly>(p, s);
  }
  const bool sums = p.partial && p.range;
  const bool pair = p.o_flops || p.o_bytes || p.o_blocks || p.o_troof || p.o_eta || p.o_t;
  const bool mult = sums && p.mult;
  constexpr int B = kStrBnd;
  if (!sums) return launch_stream<B | kStrPair>(p, s);
  if (mult)
    return pair ? launch_stream<B | kStrSums | kStrPair | kStrMult>(p, s) : launch_stream<B | kStrSums | kStrMult>(p, s);
  return pair ? launch_stream<B | kStrSums | kStrPair>(p, s) : launch_stream<B | kStrSums>(p, s);
}

static hipError_t launch_direct(int kind, const EvalParams &p, hipStream_t s) {
  if (p.wgt_off[KS_NFAM] == 0) return hipSuccess;
  switch (kind) {
    case kEtaOne: return launch_eta_one(p, s);
    case kBoundedOnly: return p.grid_mask ? launch_kind<kBoundedOnly>(p, s) : launch_bounded_stream(p, s);
    case kF32_16_64: return launch_kind<kF32_16_64>(p, s);
    case kF32_16_128: return launch_kind<kF32_16_128>(p, s);
    case kF32_32_64: return launch_kind<kF32_32_64>(p, s);
    case kF32_32_128: return launch_kind<kF32_32_128>(p, s);
    case kBF16_16_64: return launch_kind<kBF16_16_64>(p, s);
    case kBF16_16_128: return launch_kind<kBF16_16_128>(p, s);
    case kBF16_16_256: return launch_kind<kBF16_16_256>(p, s);
    case kBF16_32_64: return launch_kind<kBF16_32_64>(p, s);
    case kBF16_32_128: return launch_kind<kBF16_32_128>(p, s);
    case kBF16_32_256: return launch_kind<kBF16_32_256>(p, s);
    default: return hipErrorInvalidValue;
  }
}

static hipError_t launch_uniq_kind(int kind, const EvalParams &p, hipStream_t s) {
  switch (kind) {
    case kF32_16_64: return launch_uniq<kF32_16_64>(p, s);
    case kF32_16_128: return launch_uniq<kF32_16_128>(p, s);
    case kF32_32_64: return launch_uniq<kF32_32_64>(p, s);
    case kF32_32_128: return launch_uniq<kF32_32_128>(p, s);
    case kBF16_16_64: return launch_uniq<kBF16_16_64>(p, s);
    case kBF16_16_128: return launch_uniq<kBF16_16_128>(p, s);
    case kBF16_16_256: return launch_uniq<kBF16_16_256>(p, s);
    case kBF16_32_64: return launch_uniq<kBF16_32_64>(p, s);
    case kBF16_32_128: return launch_uniq<kBF16_32_128>(p, s);
    case kBF16_32_256: return launch_uniq<kBF16_32_256>(p, s);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_eval(int kind, const EvalParams &p, hipStream_t s) {
  if (!p.uniq) return launch_direct(kind, p, s);
  hipError_t e = launch_unique(*p.uniq, s);
  if (e == hipSuccess) e = launch_uniq_kind(kind, p, s);
  if (e == hipSuccess && p.uniq->pair) e = launch_spread(*p.uniq, p, s);
  if (e == hipSuccess && (p.o_flops || p.o_bytes || p.o_blocks)) {
    hipLaunchKernelGGL(k_counts, dim3(grid_for(p.fam_off[KS_NFAM], 256, 8192)), dim3(256), 0, s, p);
    e = hipGetLastError();
  }
  return e;
}

hipError_t launch_fill_source(const EvalParams &p, hipStream_t s) {
  const int64_t total = (int64_t)p.n_specs * p.fam_off[KS_NFAM];
  if (!p.o_src || total == 0) return hipSuccess;
  hipLaunchKernelGGL(k_fill_source, dim3(grid_for(total, 256, 8192)), dim3(256), 0, s, p.o_src, p);
  return hipGetLastError();
}

hipError_t launch_validate(const ValidateParams &p, hipStream_t s) {
  hipLaunchKernelGGL(k_validate, dim3(1024), dim3(256), 0, s, p);
  return hipGetLastError();
}

#endif  // KS_HEADS == 0

}  // namespace ks
