// The last kernel of a call with step sums: per (step, spec) the body's sum over
// the families, then the step's all-reduce and assembly (Eq. 3, Eq. 4).
#include <hip/hip_runtime.h>

#include "ks_internal.h"

namespace ks {

// per (spec, step): t_body, t_comm (Eq. 3, two all-reduces per layer),
// t_gpu and t_step (Eq. 4).  The partial sums are spec-minor and the
// outputs step-minor, so a workgroup takes a tile of kFinSteps steps x
// kFinSpecs specs (kFinSpecs a power of two, at least the spec count or
// 16): it reads with the spec fastest, passes the three results through
// LDS, and writes with the step fastest.
constexpr int kFinThreads = 256;

struct StepOut {
  double body, gpu, step;
};

__device__ __forceinline__ StepOut assemble(const FinishParams &p, double body, int64_t j, int s) {
  const ks_spec sp = p.specs[s];
  const double P = (double)p.tp[j];
  const double Sb = (double)p.agg[j] * (double)p.hidden[j] * (double)p.elem_bytes;
  double t_ar = 0.0;
  if (P > 1.0) t_ar = sp.ar_alpha0 + sp.ar_alpha_log2p * log2(P) + 2.0 * (P - 1.0) / P * Sb / sp.ar_beta;
  const double comm = 2.0 * (double)p.layers[j] * t_ar;
  const double gpu = p.host.body_scale * body + comm;
  const double step = fmax(gpu + (double)p.n_launch[j] * p.host.c_disp, p.host.ell) +
                      fmax(0.0, p.host.c_ovl - gpu) + p.host.c_tail;
  return StepOut{body, gpu, step};
}

__device__ __forceinline__ void store_step(const FinishParams &p, const StepOut &r, int64_t j, int s) {
  const size_t o = (size_t)s * (size_t)p.n_steps + (size_t)j;
  p.t_body[o] = r.body;
  p.t_gpu[o] = r.gpu;
  p.t_step[o] = r.step;
  if (p.own && p.own[j] == (uint32_t)s) p.lat[j] = r.step;
}

__global__ __launch_bounds__(kFinThreads) void k_finish(FinishParams p, int spec_bits) {
  __shared__ StepOut res[kFinThreads];
  const int tps = 1 << spec_bits;                 // specs per tile
  const int tst = kFinThreads >> spec_bits;        // steps per tile
  const int64_t n_st = (p.n_steps + tst - 1) / tst;
  const int64_t n_sp = (p.n_specs + tps - 1) / tps;
  const int tid = threadIdx.x;
  for (int64_t tile = blockIdx.x; tile < n_st * n_sp; tile += gridDim.x) {
    const int64_t j0 = (tile % n_st) * tst;
    const int s0 = (int)(tile / n_st) * tps;
    // phase 1: thread (step jj, spec ss), spec fastest
    {
      const int ss = tid & (tps - 1), jj = tid >> spec_bits;
      const int s = s0 + ss;
      const int64_t j = j0 + jj;
      if (s < p.n_specs && j < p.n_steps) {
        const size_t S = (size_t)p.n_specs;
        // every family's range, then its partial and first carry, are
        // loaded before any is summed (independent loads in flight together
        // instead of a chain of ten); the sum keeps family order: partial,
        // then the carries of its later tiles
        uint32_t r0[KS_NFAM], r1[KS_NFAM];
#pragma unroll
        for (int f = 0; f < KS_NFAM; ++f) {
          r0[f] = p.range[2 * (f * p.n_steps + j)];
          r1[f] = p.range[2 * (f * p.n_steps + j) + 1];
        }
        bool any[KS_NFAM];
        int t_first[KS_NFAM], t_last[KS_NFAM];
        double part[KS_NFAM], car1[KS_NFAM];
#pragma unroll
        for (int f = 0; f < KS_NFAM; ++f) {
          // clamped to the family's rows: a range left half-written by
          // unsorted input (reported by ks_validate) still indexes only this
          // family's tiles
          const int64_t base = p.fam_off[f], top = p.fam_off[f + 1];
          int64_t a = r0[f], b = r1[f];
          a = a < base ? base : (a > top ? top : a);
          b = b < base ? base : (b > top ? top : b);
          any[f] = a < b;
          t_first[f] = any[f] ? p.tile_off[f] + (int)((a - base) / kTileRows) : 0;
          t_last[f] = any[f] ? p.tile_off[f] + (int)((b - 1 - base) / kTileRows) : 0;
          part[f] = any[f] ? p.partial[((size_t)f * (size_t)p.n_steps + (size_t)j) * S + s] : 0.0;
          car1[f] = t_last[f] > t_first[f] ? p.carry[(size_t)(t_first[f] + 1) * S + s] : 0.0;
        }
        double body = 0.0;
#pragma unroll
        for (int f = 0; f < KS_NFAM; ++f) {
          if (!any[f]) continue;
          body += part[f];
          if (t_last[f] > t_first[f]) body += car1[f];
          for (int t = t_first[f] + 2; t <= t_last[f]; ++t) body += p.carry[(size_t)t * S + s];
        }
        res[ss * tst + jj] = assemble(p, body, j, s);
      }
    }
    __syncthreads();
    // phase 2: thread (spec ss, step jj), step fastest
    {
      const int jj = tid % tst, ss = tid / tst;
      const int s = s0 + ss;
      const int64_t j = j0 + jj;
      if (s < p.n_specs && j < p.n_steps) store_step(p, res[ss * tst + jj], j, s);
    }
    __syncthreads();
  }
}

// ------------------------------------------------------------ different records
// The families whose different records were evaluated (by whole waves).  (One
// scalar load where all fit: each thread's own flag took 1.1 us of 25 on a
// collapsed 70B trace.)
__device__ __forceinline__ uint32_t families_taken(const FinishParams &p) {
  if (p.u_over[KS_NFAM] == 0) return p.uniq_mask;
  const int lane = threadIdx.x & 63;
  return (uint32_t)__ballot(lane < KS_NFAM && ((p.uniq_mask >> lane) & 1u) && !p.u_over[lane < KS_NFAM ? lane : 0]);
}

// The body's terms of one family that the evaluation kernel summed itself
// (grouped GEMMs, and families whose different records did not fit): the
// partial, then the carries of its later tiles.
__device__ __forceinline__ double direct_sum(const FinishParams &p, int f, uint32_t r0, uint32_t r1, int64_t j, int s) {
  const int64_t base = p.fam_off[f], top = p.fam_off[f + 1];
  int64_t a = r0, b = r1;
  a = a < base ? base : (a > top ? top : a);
  b = b < base ? base : (b > top ? top : b);
  if (a >= b) return 0.0;
  const size_t S = (size_t)p.n_specs;
  const int t_first = p.tile_off[f] + (int)((a - base) / kTileRows);
  const int t_last = p.tile_off[f] + (int)((b - 1 - base) / kTileRows);
  double sum = p.partial[((size_t)f * (size_t)p.n_steps + (size_t)j) * S + s];
#pragma unroll 2
  for (int t = t_first + 1; t <= t_last; ++t) sum += p.carry[(size_t)t * S + s];
  return sum;
}

// The entries of one (family, step): piece by piece (a piece per chunk of
// records the step reaches into), each ended by its last entry.  take(u, w, n)
// is called with up to four at a time, in order: the indices of their different
// records (all valid) and their weights (0 past the last).  Their loads are in
// flight together.  Every index is bounded, whatever unsorted records left in
// the tables.
template <class F>
__device__ __forceinline__ void uniq_entries(const FinishParams &p, int f, uint32_t first, uint32_t end_row, F &&take) {
  if (first == 0) return;
  const uint32_t per = p.u_chunk_entries[f], e00 = p.u_ent_off[f];   // per: a power of two
  uint32_t e = first - 1, c = (e - e00) >> (31 - __builtin_clz(per));
  for (;;) {
    const uint32_t end = min(e00 + (c + 1) * per, p.u_ent_end);
    for (bool more = e < end; more; e += 4) {
      UniqEntry x[4];
      uint32_t u[4];
      float w[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) x[i] = p.u_ent[min(e + i, end - 1)];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        more = more && e + i < end;
        w[i] = more ? fabsf(x[i].weight) : 0.0f;
        u[i] = more ? x[i].id & kUniqIndex : 0u;
        if (more && (x[i].id & kUniqSlot)) u[i] = p.u_slot[min(u[i], p.u_slots - 1)];
        more = more && !__builtin_signbitf(x[i].weight);
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) u[i] = min(u[i], p.u_total - 1);
      take(u, w);
    }
    ++c;
    if (p.fam_off[f] + (int64_t)c * kUniqChunk >= min((int64_t)end_row, p.fam_off[f + 1])) return;
    e = e00 + c * per;
  }
}

// Up to kFewSpecs spec vectors: a thread per step and family walks the family's
// entries (the chain of dependent loads, directory, entry, slot, t, once for
// all the tile's families) and sums every spec; then a thread per step and spec
// adds the families in order: 8.6 us for 8000 steps (a thread per step and spec that
// walked the ten families one after the other took 20 to 26), 12.9 for 20,000, 20
// for 40,000 with a record per layer and 25 for 80,000 collapsed.  NS: the spec
// count rounded up to a power of two.
constexpr int kFewSpecs = 4;
constexpr int kFewSteps = 16;

template <int NS>
__global__ __launch_bounds__(kFinThreads) __attribute__((amdgpu_waves_per_eu(6))) void k_finish_few(FinishParams p) {
  __shared__ double part[kFewSteps][KS_NFAM][NS];
  const int tid = threadIdx.x, f = tid & 15, jj = tid >> 4;
  const uint32_t uniq = families_taken(p);
  const int64_t n_st = (p.n_steps + kFewSteps - 1) / kFewSteps;
  for (int64_t tile = blockIdx.x; tile < n_st; tile += gridDim.x) {
    const int64_t j0 = tile * kFewSteps, j = j0 + jj;
    if (f < KS_NFAM && j < p.n_steps) {
      const uint32_t d0 = p.range[2 * (f * p.n_steps + j)], d1 = p.range[2 * (f * p.n_steps + j) + 1];
      double sum[NS] = {};
      if ((uniq >> f) & 1u) {
        uniq_entries(p, f, d0, d1, [&](const uint32_t (&u)[4], const float (&w)[4]) {
          float t[4][NS];
#pragma unroll
          for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int s = 0; s < NS; ++s)
              t[i][s] = s < p.n_specs && w[i] != 0.0f ? p.u_t[(size_t)u[i] * (size_t)p.n_specs + s] : 0.0f;
#pragma unroll
          for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int s = 0; s < NS; ++s) sum[s] += (double)w[i] * (double)t[i][s];
        });
      } else {
#pragma unroll
        for (int s = 0; s < NS; ++s)
          if (s < p.n_specs) sum[s] = direct_sum(p, f, d0, d1, j, s);
      }
#pragma unroll
      for (int s = 0; s < NS; ++s) part[jj][f][s] = sum[s];
    }
    __syncthreads();
    const int s = tid / kFewSteps, js = tid % kFewSteps;
    if (s < p.n_specs && j0 + js < p.n_steps) {
      double body = 0.0;
#pragma unroll
      for (int g = 0; g < KS_NFAM; ++g) body += part[js][g][s];
      store_step(p, assemble(p, body, j0 + js, s), j0 + js, s);
    }
    __syncthreads();
  }
}

// More spec vectors: a workgroup's tile of steps lists its steps' entries in
// LDS once for all the tile's specs (a thread per step and family, then packed
// step by step), and its (step, spec) threads add the listed t, whose loads do
// not wait on each other.
constexpr int kListSteps = 16;     // steps of a tile, at most
constexpr int kListEntries = 8;    // entries listed per step and family; a thread that has more walks them again

__global__ __launch_bounds__(kFinThreads) void k_finish_list(FinishParams p, int spec_bits) {
  __shared__ StepOut res[kFinThreads];
  __shared__ uint2 own[kListSteps * KS_NFAM][kListEntries];      // {index, weight}
  __shared__ uint2 list[kListSteps][KS_NFAM * kListEntries];
  __shared__ uint32_t count[kListSteps * KS_NFAM];
  __shared__ uint32_t total[kListSteps], rest[kListSteps];        // rest: families with more entries or sums of their own
  const uint32_t uniq = families_taken(p);
  const int tps = 1 << spec_bits;
  const int tst = min(kFinThreads >> spec_bits, kListSteps);
  const int64_t n_st = (p.n_steps + tst - 1) / tst;
  const int64_t n_sp = (p.n_specs + tps - 1) / tps;
  const int tid = threadIdx.x;
  const size_t S = (size_t)p.n_specs;
  for (int64_t tile = blockIdx.x; tile < n_st * n_sp; tile += gridDim.x) {
    const int64_t j0 = (tile % n_st) * tst;
    const int s0 = (int)(tile / n_st) * tps;
    const int q = tid, fq = q % KS_NFAM, jq = q / KS_NFAM;
    uint32_t mine = 0;
    if (tid < kListSteps) rest[tid] = 0;
    __syncthreads();
    if (jq < tst && j0 + jq < p.n_steps) {
      const uint32_t *d = p.range + 2 * (fq * p.n_steps + j0 + jq);
      if ((uniq >> fq) & 1u) {
        uint32_t seen = 0;
        uniq_entries(p, fq, d[0], d[1], [&](const uint32_t (&u)[4], const float (&w)[4]) {
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            if (w[i] == 0.0f) continue;
            if (seen < kListEntries) own[q][seen] = uint2{u[i], __builtin_bit_cast(uint32_t, w[i])};
            ++seen;
          }
        });
        if (seen > kListEntries) atomicOr(rest + jq, 1u << fq);
        mine = min(seen, (uint32_t)kListEntries);
      } else if (p.fam_off[fq + 1] > p.fam_off[fq]) {
        atomicOr(rest + jq, 1u << fq);
      }
    }
    if (jq < tst) count[q] = mine;
    __syncthreads();
    if (jq < tst) {
      uint32_t at = 0;
      for (int g = 0; g < fq; ++g) at += count[jq * KS_NFAM + g];
      for (uint32_t i = 0; i < mine; ++i) list[jq][at + i] = own[q][i];
      if (fq == KS_NFAM - 1) total[jq] = at + mine;
    }
    __syncthreads();
    const int ss = tid & (tps - 1), jj = tid >> spec_bits;
    const int s = s0 + ss;
    const int64_t j = j0 + jj;
    if (jj < tst && s < p.n_specs && j < p.n_steps) {
      double body = 0.0;
      const uint32_t n = total[jj];
      const float *t = p.u_t + s;
      for (uint32_t i = 0; i < n; i += 8) {
        float v[8], w[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) {
          const uint2 x = list[jj][min(i + k, n - 1)];
          w[k] = i + k < n ? __builtin_bit_cast(float, x.y) : 0.0f;
          v[k] = t[(size_t)x.x * S];
        }
#pragma unroll
        for (int k = 0; k < 8; ++k)
          if (i + k < n) body += (double)w[k] * (double)v[k];
      }
      for (uint32_t left = rest[jj]; left; left &= left - 1) {
        const int f = __builtin_ctz(left);
        const uint32_t *d = p.range + 2 * (f * p.n_steps + j);
        if ((uniq >> f) & 1u) {
          uint32_t seen = 0;
          uniq_entries(p, f, d[0], d[1], [&](const uint32_t (&u)[4], const float (&w)[4]) {
#pragma unroll
            for (int i = 0; i < 4; ++i)
              if (w[i] != 0.0f && seen++ >= kListEntries) body += (double)w[i] * (double)t[(size_t)u[i] * S];
          });
        } else {
          body += direct_sum(p, f, d[0], d[1], j, s);
        }
      }
      res[ss * tst + jj] = assemble(p, body, j, s);
    }
    __syncthreads();
    if (tid < tps * tst) {
      const int js = tid % tst, sw = s0 + tid / tst;
      if (sw < p.n_specs && j0 + js < p.n_steps) store_step(p, res[tid], j0 + js, sw);
    }
    __syncthreads();
  }
}

static dim3 fin_grid(int64_t tiles) { return dim3((unsigned)(tiles < 8192 ? tiles : 8192)); }

hipError_t launch_finish(const FinishParams &p, hipStream_t s) {
  if (p.n_steps == 0) return hipSuccess;
  const bool uniq = p.uniq_mask != 0;
  if (uniq && p.n_specs <= kFewSpecs) {
    const dim3 grid = fin_grid((p.n_steps + kFewSteps - 1) / kFewSteps);
    if (p.n_specs == 1) hipLaunchKernelGGL(k_finish_few<1>, grid, dim3(kFinThreads), 0, s, p);
    else if (p.n_specs == 2) hipLaunchKernelGGL(k_finish_few<2>, grid, dim3(kFinThreads), 0, s, p);
    else hipLaunchKernelGGL(k_finish_few<4>, grid, dim3(kFinThreads), 0, s, p);
    return hipGetLastError();
  }
  // specs per tile: the spec count rounded up to a power of two, at most 16 (32
  // over listed entries: each further tile lists them again)
  int bits = 0;
  while (bits < (uniq ? 5 : 4) && (1 << bits) < p.n_specs) ++bits;
  int64_t tst = kFinThreads >> bits;
  if (uniq && tst > kListSteps) tst = kListSteps;
  const int64_t tiles = ((p.n_steps + tst - 1) / tst) * (((int64_t)p.n_specs + (1 << bits) - 1) >> bits);
  if (uniq)
    hipLaunchKernelGGL(k_finish_list, fin_grid(tiles), dim3(kFinThreads), 0, s, p, bits);
  else
    hipLaunchKernelGGL(k_finish, fin_grid(tiles), dim3(kFinThreads), 0, s, p, bits);
  return hipGetLastError();
}

}  // namespace ks
