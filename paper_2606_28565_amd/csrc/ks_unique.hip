// The different records of a call on gfx950: the records of a step repeat
// from layer to layer (decoder layers are homogeneous, Sec. 5.7), and steps
// with equal token counts dispatch equal dense kernels, so a call with an
// MLP head evaluates each different record once and the step sums weight it.
//
//   k_unique   per chunk of 1024 records of one family: runs of equal step
//              (pieces), each piece's period (the layer's kernel list), its
//              first period as entries (which record, how many of it); every
//              entry's record leaves its row in a slot of the family's table
//   k_join     the slots' rows become the different records; an entry whose
//              slot holds the same record refers to it, one whose slot another
//              record took is a different record of its own
//
// A piece of length n has period q in 1 .. 4 if every record equals the one q
// before it: then its first q records, record r standing for ceil((n - r) / q)
// of them, are all there is to evaluate.  Without such a q every record is an
// entry.  Records are equal when their fields are: slots only say which record
// to compare with, so a slot may hold any of the rows stored to it, and no
// compare-and-swap settles whose (a table with one, in one pass, spent 40% of
// the pass on it: a serving trace's few batch sizes meet at the same slots,
// whose atomic operations follow one another at about 60 ns).
#include <hip/hip_runtime.h>

#include "ks_agg.h"
#include "ks_internal.h"

namespace ks {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
// four consecutive words at any word address (global loads need no more)
typedef uint32_t u32x4_any __attribute__((ext_vector_type(4), aligned(4)));

constexpr int kUqThreads = 256;
constexpr uint32_t kUqNoStep = 0xFFFFFFFFu;
static_assert(kUniqChunk == 4 * kUqThreads, "four consecutive records per thread");

// records base[4 t .. 4 t + 3] of a chunk of n (n >= 1), past its end the last one
__device__ __forceinline__ u32x4 chunk_quad(const uint32_t *base, int t, int n) {
  if (4 * t + 3 < n) {
    const u32x4_any v = *reinterpret_cast<const u32x4_any *>(base + 4 * t);
    return u32x4{v[0], v[1], v[2], v[3]};
  }
  u32x4 v;
#pragma unroll
  for (int j = 0; j < 4; ++j) v[j] = base[4 * t + j < n ? 4 * t + j : n - 1];
  return v;
}

// lane - 1's value; lane 0 keeps `first`
__device__ __forceinline__ uint32_t from_prev(uint32_t first, uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp((int)first, (int)v, 0x138, 0xf, 0xf, false);   // wave_shr:1
}

// lane + 1's value; lane 63 keeps `last`
__device__ __forceinline__ uint32_t from_next(uint32_t last, uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp((int)last, (int)v, 0x130, 0xf, 0xf, false);   // wave_shl:1
}

// inclusive prefix of v over the wave's lanes (row shifts by 1, 2, 4 and 8
// lanes, then the two row broadcasts)
__device__ __forceinline__ uint32_t wave_prefix(uint32_t v) {
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xf, 0xf, false);
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xf, 0xf, false);
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xf, 0xf, false);
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xf, 0xf, false);
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xa, 0xf, false);
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xc, 0xf, false);
  return v;
}

// sums of the waves before this one, and of all, from the waves' own in LDS
__device__ __forceinline__ uint32_t waves_before(const uint32_t *wave_sum, uint32_t &total) {
  const int wave = threadIdx.x >> 6;
  uint32_t base = 0;
  total = 0;
#pragma unroll
  for (int w = 0; w < kUqThreads / 64; ++w) {
    if (w < wave) base += wave_sum[w];
    total += wave_sum[w];
  }
  return base;
}

// The slot of a record in its family's table: attention's is its step's, a
// dense one's is its m off a place of its (n, k), so that the token counts of
// one kernel meet in a slot only a table's size apart.
__device__ __forceinline__ uint32_t slot_of(const UniqParams &p, int f, uint32_t step, uint32_t m, uint32_t n,
                                            uint32_t k) {
  if (f == KS_ATTN_PREFILL || f == KS_ATTN_DECODE) return p.slot_off[f] + step;
  const uint32_t place = (uint32_t)((((unsigned long long)n << 32 | k) * 0x9E3779B97F4A7C15ull) >> 40);
  return p.slot_off[f] + ((m + place) & p.slot_mask[f]);
}

// Family f's different records do not fit: all its records are evaluated.
__device__ __forceinline__ void no_room(const UniqParams &p, int f) {
  p.over[f] = 1u;
  p.over[KS_NFAM] = 1u;
}

// What k_unique's passes share in LDS.
struct UniqShared {
  uint32_t bad_of[kUniqChunk];        // per piece: bit q - 1, some record differs from the one q before; then its period
  uint32_t start_of[kUniqChunk + 1];  // per piece: first record, then the chunk's end
  uint32_t ent_of[kUniqChunk + 1];    // per piece: first entry, then the chunk's end
  uint16_t piece_of[kUniqChunk];      // per entry
  uint32_t heads[kUqThreads / 64], entries[kUqThreads / 64];
};

// Entry e of the chunk.
__device__ __forceinline__ void chunk_entry(const UniqParams &p, const UniqShared &sh, int f, int64_t row0, uint32_t e,
                                            uint32_t ent0) {
  const bool attn = f == KS_ATTN_PREFILL || f == KS_ATTN_DECODE;
  const bool has_k = f != KS_RMSNORM && f != KS_SILU_MUL && f != KS_EMBED;
  const uint32_t t = sh.piece_of[e], r = e - sh.ent_of[t], b = sh.start_of[t], q = sh.bad_of[t];
  const uint32_t times = (sh.start_of[t + 1] - b - r + q - 1) / q;
  const uint32_t row = (uint32_t)row0 + b + r;
  const uint32_t st = p.step[row], mult = p.mult ? p.mult[row] : 1u, n = p.n[row];
  const uint32_t m = attn ? 0u : p.m[row], k = !attn && has_k ? p.k[row] : 0u;
  UniqEntry out = {kUniqNone, 0.0f};
  if ((int64_t)st < p.n_steps) {
    // a plain store (of one word, into this die's cache): whichever row a slot
    // ends up with is compared before it is used.  Agent scope, each store on
    // its own to memory, took five times as long (551 for 107 us on a 70B batch).
    const uint32_t s = slot_of(p, f, st, m, n, k);
    __hip_atomic_store(p.slot_row + s, row + 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    p.ent_slot[ent0 + e] = s;
    out = {row, (float)((double)times * (double)mult)};
  }
  // the sign bit marks a piece's last entry
  if (e + 1 == sh.ent_of[t + 1]) out.weight = -out.weight;
  p.ent[ent0 + e] = out;
}

// Bound by the stream of records with eight workgroups per CU resident (a chunk
// is a chain of four barriers and two memory round trips, some 6 us): 28.9M
// records of a 70B batch in 114 us (491 MB read and 71 written by the counters,
// 4.9 TB/s), 7.2M in 37, 390,000 in 8.
__global__ __launch_bounds__(kUqThreads) __attribute__((amdgpu_waves_per_eu(8))) void k_unique(UniqParams p, int n_agg) {
  __shared__ __align__(16) UniqShared sh;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int c = (int)blockIdx.x - n_agg;
  if (c < 0) {
    attn_agg(p.req_off, p.req_q, p.req_h, p.n_steps, p.n_req, p.agg, p.err, (int64_t)blockIdx.x * kUqThreads + tid,
             (int64_t)n_agg * kUqThreads);
    return;
  }
  int f = 0;
  while (c >= p.chunk_off[f + 1]) ++f;
  const bool attn = f == KS_ATTN_PREFILL || f == KS_ATTN_DECODE;
  const bool has_k = f != KS_RMSNORM && f != KS_SILU_MUL && f != KS_EMBED;
  const int64_t row0 = p.fam_off[f] + (int64_t)(c - p.chunk_off[f]) * kUniqChunk;
  const int64_t left = p.fam_off[f + 1] - row0;
  const int n = left < kUniqChunk ? (int)left : kUniqChunk;

  // the fields a family's latency depends on within a step: (m, n, k) or
  // attention's (a, n, k); and the multiplicity
  const uint32_t *src[4] = {attn ? p.a + row0 : p.m + row0, p.n + row0, has_k ? p.k + row0 : nullptr,
                            p.mult ? p.mult + row0 : nullptr};
  const u32x4 st = chunk_quad(p.step + row0, tid, n);
  u32x4 v[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) v[i] = src[i] ? chunk_quad(src[i], tid, n) : u32x4{0, 0, 0, 0};
  // the four records before this lane's: the lane before, or for the first
  // lane of a wave the end of the wave before (none before the chunk); and the
  // step of the one after
  u32x4 pst = {kUqNoStep, kUqNoStep, kUqNoStep, kUqNoStep}, pv[4] = {};
  uint32_t nst = kUqNoStep, before = kUqNoStep;   // before: of the chunk's first record
  if (lane == 0 && tid > 0) {
    pst = chunk_quad(p.step + row0, tid - 1, n);
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (src[i]) pv[i] = chunk_quad(src[i], tid - 1, n);
  }
  const bool more_before = row0 > p.fam_off[f];
  if (tid == 0 && more_before) before = p.step[row0 - 1];
  if (lane == 63 && 4 * tid + 4 < left) nst = p.step[row0 + 4 * tid + 4];
  *reinterpret_cast<u32x4 *>(sh.bad_of + 4 * tid) = u32x4{0, 0, 0, 0};
  nst = from_next(nst, st[0]);
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    pst[j] = from_prev(pst[j], st[j]);
#pragma unroll
    for (int i = 0; i < 4; ++i) pv[i][j] = from_prev(pv[i][j], v[i][j]);
  }
  uint32_t bad[4], heads = 0, flag = 0;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int r = 4 * tid + j;
    const bool in = r < n;
    bad[j] = 0;
#pragma unroll
    for (int q = 1; q <= 4; ++q) {
      const uint32_t s = j >= q ? st[j - q] : pst[j - q + 4];
      uint32_t d = 0;
#pragma unroll
      for (int i = 0; i < 4; ++i) d |= v[i][j] ^ (j >= q ? v[i][j - q] : pv[i][j - q + 4]);
      bad[j] |= (in && s == st[j] && d != 0 ? 1u : 0u) << (q - 1);
    }
    const bool head = in && (r == 0 || (j > 0 ? st[j - 1] : pst[3]) != st[j]);
    heads |= (head ? 1u : 0u) << j;
    // the (family, step) directory's end row, where its global last record is
    const bool end = in && (r + 1 == (int64_t)left || (j < 3 ? st[j + 1] : nst) != st[j]);
    if (in && (int64_t)st[j] >= p.n_steps) flag = kErrStep;
    else if (end) p.dir[2 * ((size_t)f * (size_t)p.n_steps + st[j]) + 1] = (uint32_t)(row0 + r + 1);
  }
  if (flag) {
    atomicOr(p.err, flag);
    if (p.pair) no_room(p, f);
  }
  uint32_t piece = 0;
  {
    uint32_t all = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const uint64_t b = __ballot((heads >> j) & 1u);
      piece += __builtin_amdgcn_mbcnt_hi((uint32_t)(b >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)b, 0u));
      all += (uint32_t)__popcll(b);
    }
    if (lane == 0) sh.heads[wave] = all;
  }
  __syncthreads();
  uint32_t n_pieces;
  piece += waves_before(sh.heads, n_pieces);
  // a record's piece is the last head at or before it; the lane's bits are
  // joined while the piece stays the same
  const uint32_t piece0 = piece;
  {
    uint32_t acc = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      if ((heads >> j) & 1u) {
        if (acc) atomicOr(sh.bad_of + piece - 1, acc);
        acc = 0;
        sh.start_of[piece] = (uint32_t)(4 * tid + j);
        ++piece;
      }
      acc |= bad[j];
    }
    if (acc) atomicOr(sh.bad_of + piece - 1, acc);
  }
  if (tid == 0) sh.start_of[n_pieces] = (uint32_t)n;
  __syncthreads();
  // pieces 4 t .. 4 t + 3: period, entries
  uint32_t per[4], cnt[4], sum = 0;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const uint32_t t = 4 * tid + i;
    per[i] = cnt[i] = 0;
    if (t < n_pieces) {
      const uint32_t len = sh.start_of[t + 1] - sh.start_of[t], b = sh.bad_of[t];
      per[i] = !(b & 1u) ? 1u : !(b & 2u) ? 2u : !(b & 4u) ? 3u : !(b & 8u) ? 4u : len;
      cnt[i] = per[i] < len ? per[i] : len;
    }
    sum += cnt[i];
  }
  const uint32_t incl = wave_prefix(sum);
  if (lane == 63) sh.entries[wave] = incl;
  __syncthreads();
  uint32_t n_ent;
  uint32_t e0 = waves_before(sh.entries, n_ent) + incl - sum;
  // no room: in the chunk, or for the family's different records (which a rule
  // on each chunk's entries keeps below the family's room, so that it does not
  // hang on which of the records that share a slot was stored last)
  const uint32_t slots = p.chunk_entries[f];
  if (n_ent > min(slots, 4u * n_pieces + p.spare[f])) {
    if (tid == 0) no_room(p, f);
    return;
  }
  const uint32_t ent0 = p.ent_off[f] + (uint32_t)(c - p.chunk_off[f]) * slots;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const uint32_t t = 4 * tid + i;
    if (t >= n_pieces) break;
    sh.ent_of[t] = e0;
    sh.bad_of[t] = per[i];
    for (uint32_t r = 0; r < cnt[i]; ++r) sh.piece_of[e0 + r] = (uint16_t)t;
    e0 += cnt[i];
  }
  if (tid == 0) {
    sh.ent_of[n_pieces] = n_ent;
    p.chunk_count[c] = n_ent;
  }
  __syncthreads();
  if (p.pair) {
    // each row's entry: the same place in its piece's first period
    uint32_t t = piece0;
    uint16_t e[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      t += (heads >> j) & 1u;
      const uint32_t i = 4 * tid + j;
      e[j] = (int)i < n ? (uint16_t)(sh.ent_of[t - 1] + (i - sh.start_of[t - 1]) % sh.bad_of[t - 1]) : 0;
    }
    *reinterpret_cast<ushort4 *>(p.row_entry + (size_t)c * kUniqChunk + 4 * tid) = ushort4{e[0], e[1], e[2], e[3]};
  }
  // the directory's first entry, where the (family, step)'s global first record is
  {
    uint32_t t = piece0;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      if (!((heads >> j) & 1u)) continue;
      const bool first = 4 * tid + j > 0 || !more_before || before != st[0];
      if (first && (int64_t)st[j] < p.n_steps)
        p.dir[2 * ((size_t)f * (size_t)p.n_steps + st[j])] = ent0 + sh.ent_of[t] + 1;
      ++t;
    }
  }
  for (uint32_t e = tid; e < n_ent; e += kUqThreads) chunk_entry(p, sh, f, row0, e, ent0);
}

// The fields of a row that decide its latency within its family (attention:
// and step, which its slot implies).
struct UniqKey {
  uint32_t x, n, k;
};
__device__ __forceinline__ UniqKey key_of(const UniqParams &p, int f, uint32_t row) {
  const bool attn = f == KS_ATTN_PREFILL || f == KS_ATTN_DECODE;
  const bool has_k = f != KS_RMSNORM && f != KS_SILU_MUL && f != KS_EMBED;
  return UniqKey{(attn ? p.a : p.m)[row], p.n[row], has_k ? p.k[row] : 0u};
}

// Room for n new different records of family f: their first index among the
// family's (past its room, where unsorted steps make more pieces than steps: all
// its records are evaluated).
__device__ __forceinline__ uint32_t take_records(const UniqParams &p, int f, uint32_t n) {
  const uint32_t i = atomicAdd(p.count + f, n);
  if (i + n > p.cap[f]) no_room(p, f);
  return i;
}

// Workgroups 0 .. scan_off[KS_NFAM] - 1: 4096 slots each, the used ones' rows
// listed (one atomic addition per workgroup).  The others: entries, by one wave
// a quarter of a chunk with 1024 entry slots, else four chunks at 16 lanes each
// (with a record per layer a chunk has 10 to 50 entries: a wave per chunk took
// 26 us on the 70B batch where four took 21; with four entries a lane in flight
// 19.6, and 11.4 for 15.2 on the collapsed 70B trace).
__global__ __launch_bounds__(kUqThreads) void k_join(UniqParams p) {
  __shared__ uint32_t wave_sum[kUqThreads / 64], first;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  int b = (int)blockIdx.x;
  if (b < p.scan_off[KS_NFAM]) {
    int f = 0;
    while (b >= p.scan_off[f + 1]) ++f;
    const uint32_t s0 = (uint32_t)(b - p.scan_off[f]) * kUniqScan, n = min(kUniqScan, p.slots[f] - s0);
    const uint32_t *slot = p.slot_row + p.slot_off[f] + s0;
    uint32_t v[kUniqScan / kUqThreads], mine = 0;
#pragma unroll
    for (uint32_t i = 0; i < kUniqScan / kUqThreads; ++i) {
      const uint32_t s = i * kUqThreads + tid;
      v[i] = s < n ? slot[s] : 0u;
    }
#pragma unroll
    for (uint32_t i = 0; i < kUniqScan / kUqThreads; ++i) mine += v[i] ? 1u : 0u;
    const uint32_t incl = wave_prefix(mine);
    if (lane == 63) wave_sum[wave] = incl;
    __syncthreads();
    uint32_t all;
    uint32_t at = waves_before(wave_sum, all) + incl - mine;
    if (all == 0) return;
    if (tid == 0) first = take_records(p, f, all);
    __syncthreads();
    at += first;
#pragma unroll
    for (uint32_t i = 0; i < kUniqScan / kUqThreads; ++i) {
      if (!v[i]) continue;
      if (at < p.cap[f]) {
        p.list[p.base[f] + at] = v[i] - 1u;
        p.slot_id[p.slot_off[f] + s0 + i * kUqThreads + tid] = p.base[f] + at;
      }
      ++at;
    }
    return;
  }
  const int u = (b - p.scan_off[KS_NFAM]) * (kUqThreads / 64) + wave;
  if (u >= p.unit_off[KS_NFAM]) return;
  int f = 0;
  while (u >= p.unit_off[f + 1]) ++f;
  const bool flat = p.chunk_entries[f] == kUniqChunk;
  const int local = u - p.unit_off[f], c = flat ? local / 4 : 4 * local + (lane >> 4);
  if (p.over[f]) return;   // (a chunk without room wrote no count)
  const uint32_t e0 = flat ? (uint32_t)(local % 4) * (kUniqChunk / 4) : 0u, step = flat ? 64 : 16;
  const uint32_t ent0 = p.ent_off[f] + (uint32_t)c * p.chunk_entries[f];
  const uint32_t n = c < p.chunk_off[f + 1] - p.chunk_off[f] ? p.chunk_count[p.chunk_off[f] + c] : 0u;
  const uint32_t e1 = min(e0 + kUniqChunk / 4, n);
  // four entries a lane at a time, each load of the four before the next
  for (uint32_t e = e0 + (lane & (step - 1)); __any(e < e1); e += 4 * step) {
    uint32_t row[4], s[4], held[4], own = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const bool in = e + i * step < e1;
      row[i] = in ? p.ent[ent0 + e + i * step].id : kUniqNone;
      s[i] = in ? p.ent_slot[ent0 + e + i * step] : 0u;
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) held[i] = row[i] != kUniqNone ? p.slot_row[s[i]] - 1u : kUniqNone;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      if (held[i] == row[i]) continue;
      const UniqKey a = key_of(p, f, row[i]), h = key_of(p, f, held[i]);
      own |= (((h.x ^ a.x) | (h.n ^ a.n) | (h.k ^ a.k)) != 0 ? 1u : 0u) << i;
    }
    // one atomic addition per wave, at the family's one counter: one per entry
    // made a call of 220,000 records that seldom repeat (token counts up to
    // 4 million, 16 spec vectors) 633 us, this 164
    const uint32_t mine = (uint32_t)__popc(own), incl = wave_prefix(mine);
    const uint32_t all = (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
    uint32_t at = 0;
    if (all) {
      if (lane == 63) at = take_records(p, f, all);
      at = (uint32_t)__builtin_amdgcn_readlane((int)at, 63) + incl - mine;
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      if (row[i] == kUniqNone) continue;
      uint32_t id = s[i] | kUniqSlot;
      if ((own >> i) & 1u) {
        if (at < p.cap[f]) p.list[p.base[f] + at] = row[i];
        id = p.base[f] + min(at, p.cap[f] - 1u);
        ++at;
      }
      p.ent[ent0 + e + i * step].id = id;
    }
  }
}

// Per-pair outputs of a chunk's rows: its entries' records in LDS, then for each
// spec of the workgroup's range the rows' values, four consecutive rows per
// thread, gathered from the different records' (a wave's rows share few) and
// written as one 16-byte store.  Bound by the writes.
__global__ __launch_bounds__(kUqThreads) void k_spread(UniqParams u, const float *ut, size_t pair, int32_t n_specs,
                                                       int64_t n_rows, float *o_troof, float *o_eta, float *o_t,
                                                       uint32_t total, uint32_t all_slots, int per_range) {
  __shared__ uint32_t rec[kUniqChunk];
  typedef float f32x4_any __attribute__((ext_vector_type(4), aligned(4)));
  const int tid = threadIdx.x, c = (int)blockIdx.x;
  int f = 0;
  while (c >= u.chunk_off[f + 1]) ++f;
  if (u.over[f]) return;   // its every record was evaluated
  const int64_t row0 = u.fam_off[f] + (int64_t)(c - u.chunk_off[f]) * kUniqChunk;
  const int64_t left = u.fam_off[f + 1] - row0;
  const int n = left < kUniqChunk ? (int)left : kUniqChunk;
  const uint32_t ent0 = u.ent_off[f] + (uint32_t)(c - u.chunk_off[f]) * u.chunk_entries[f];
  const uint32_t n_ent = min(u.chunk_count[c], u.chunk_entries[f]);
  const ushort4 e = *reinterpret_cast<const ushort4 *>(u.row_entry + (size_t)c * kUniqChunk + 4 * tid);
  for (uint32_t i = tid; i < n_ent; i += kUqThreads) {
    const uint32_t id = u.ent[ent0 + i].id;
    uint32_t r = id & kUniqIndex;
    if (id & kUniqSlot) r = u.slot_id[min(r, all_slots - 1)];
    rec[i] = min(r, total - 1);
  }
  __syncthreads();
  if (4 * tid >= n) return;
  const size_t S = (size_t)n_specs;
  const float *src[4] = {ut + rec[e.x] * S, ut + rec[e.y] * S, ut + rec[e.z] * S, ut + rec[e.w] * S};
  const int s0 = (int)blockIdx.y * per_range, s1 = min(s0 + per_range, n_specs);
  auto copy = [&](float *out, size_t off) {
    for (int s = s0; s < s1; ++s) {
      float *q = out + (size_t)s * (size_t)n_rows + (size_t)row0 + 4 * tid;
      float v[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) v[j] = src[j][off + s];
      if (4 * tid + 3 < n) {
        __builtin_nontemporal_store(f32x4_any{v[0], v[1], v[2], v[3]}, reinterpret_cast<f32x4_any *>(q));
      } else {
        for (int j = 0; 4 * tid + j < n; ++j) q[j] = v[j];
      }
    }
  };
  if (o_t) copy(o_t, 0);
  if (o_troof) copy(o_troof, pair);
  if (o_eta) copy(o_eta, 2 * pair);
}

hipError_t launch_spread(const UniqParams &u, const EvalParams &p, hipStream_t s) {
  const int chunks = u.chunk_off[KS_NFAM];
  if (chunks == 0 || !(p.o_troof || p.o_eta || p.o_t)) return hipSuccess;
  // spec ranges until about eight workgroups per CU (256) are at work
  int ranges = 2048 / chunks;
  ranges = ranges < 1 ? 1 : ranges > p.n_specs ? p.n_specs : ranges;
  const int per = (p.n_specs + ranges - 1) / ranges;
  uint32_t total = 0, slots = 0;
  for (int f = 0; f < KS_NFAM; ++f) {
    total = u.base[f] + u.cap[f] > total ? u.base[f] + u.cap[f] : total;
    slots = u.slot_off[f] + u.slots[f] > slots ? u.slot_off[f] + u.slots[f] : slots;
  }
  hipLaunchKernelGGL(k_spread, dim3(chunks, (p.n_specs + per - 1) / per), dim3(kUqThreads), 0, s, u, p.u_t, p.u_pair,
                     p.n_specs, p.fam_off[KS_NFAM], p.o_troof, p.o_eta, p.o_t, total, slots, per);
  return hipGetLastError();
}

hipError_t launch_unique(const UniqParams &p, hipStream_t s) {
  const int chunks = p.chunk_off[KS_NFAM];
  if (chunks == 0) return hipSuccess;
  // the request sums' workgroups first: a step's chain of loads is the longest
  const int64_t steps_per = kUqThreads / kAggLanes;
  const int64_t aggs = (p.n_steps + steps_per - 1) / steps_per;
  const int n_agg = (int)(aggs < 8192 ? aggs : 8192);
  hipLaunchKernelGGL(k_unique, dim3(n_agg + chunks), dim3(kUqThreads), 0, s, p, n_agg);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const int waves = kUqThreads / 64;
  hipLaunchKernelGGL(k_join, dim3(p.scan_off[KS_NFAM] + (p.unit_off[KS_NFAM] + waves - 1) / waves), dim3(kUqThreads), 0,
                     s, p);
  return hipGetLastError();
}

}  // namespace ks
