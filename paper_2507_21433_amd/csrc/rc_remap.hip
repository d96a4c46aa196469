// rc_remap_block_table: zero-copy sharing applied to the PagedAttention block tables
// (ReasonCache Sec. IV-B: the kept block's reference count goes up, the table entry is
// rewritten, nothing is copied; a block is freed only at reference count 0).
//
// remap_layer_kernel, one launch: every workgroup of a layer counts the references of the whole table for itself and
// keeps its share of the layer's reference counts in LDS, so no workgroup needs anything from another one.  It
// serves what fits (see layer_kernel_fits); the rest goes through
//   gather  : table_out[e] = target of table_in[e], 16-byte loads and stores when the layout allows,
//             the next batch of entries in flight while the current one is worked on.  A workgroup
//             first builds what it needs to decide an entry without touching global memory again:
//             a 16-bit table "block id - lo -> slot + 1 of the matched query block" over the id
//             range of the query blocks and the target of every matched slot, both in LDS (when the
//             ids span at most 32768 blocks and Q <= 4096).  Otherwise every entry follows the chain
//             entry -> slot_of -> query_ids -> match_idx -> pool_ids through global memory;
//             slot_of[query_ids[q]] = q is written by every workgroup for itself and never cleared:
//             an entry s read for block b counts only if s < Q and query_ids[s] == b.
//             References to matched query blocks are counted per workgroup in an LDS histogram: the
//             hits of a batch are compacted into a list (prefix sums), then every wave adds up the
//             keys of its own residue class (equal keys merged with ballots).  The same workgroups
//             copy their share of refcount_in to refcount_out.  With one workgroup per layer (small
//             tables, or many layers) the workgroup goes on to finalize its layer from its histogram.
//   finalize: per layer, cnt[q] = sum of the workgroups' histograms; the query block loses cnt
//             references, its target gains them.  Queries that share a target take turns through
//             a small claim table in LDS, one winner per slot and round.  A launch of its own only
//             when a layer was gathered by several workgroups.
// No atomics on global memory anywhere; integer adds only, so the same counts on every run.
#include <hip/hip_runtime.h>

#include <mutex>

#include "rc_common.hpp"
#include "rc_remap_plan.hpp"

namespace rc {
namespace {

constexpr int kMaxQ = 8192;                                           // LDS histogram bins
constexpr int kLdsIds = 32768;                                        // id range the 16-bit slot table covers
constexpr int kLdsTargets = 4096;                                     // most query slots with their target in LDS
constexpr int kFinalThreads = 1024;
constexpr int kFinalPerThread = kMaxQ / kFinalThreads;
constexpr int kClaimSlots = 4096;
constexpr int kLayerCounts = 15872;                                   // reference counts a workgroup of remap_layer_kernel owns, at most
constexpr int64_t kLayerEntries = 131072;                             // entries of a table that several of its workgroups read, at most

// What remap_layer_kernel takes: query slots whose targets and counts fit beside a share of the reference counts in
// LDS; and, where several workgroups read a layer's table, a table that is short enough to be read by each and that is
// not rewritten in place.  Its lead shrinks with every entry, sooner where entries are loaded one by one (`vec` is false: the
// table's length or address is no multiple of 16 bytes), where there are few query blocks, whose histograms the gather launches
// add up in no time, and where the query blocks lie further apart than the 16-bit table reaches, which a pool of more
// than kLdsIds blocks allows.  Gather and finalize launches / this kernel, us, one layer:
//   16 bytes at a time  500 query blocks  131 072 entries 21.4 / 19.0   far apart 98 304 27.2 / 24.5, 131 072 28.5 / 30.4
//                       16                81 920 14.2 / 13.6, 114 688 15.6 / 16.8   4   81 920 13.6 / 13.8, 114 688 14.5 / 17.2
//   one by one          500               81 920 18.7 / 19.0, 98 304 19.9 / 21.4    64  49 152 14.9 / 13.5, 65 536 16.0 / 16.1
//                       16                49 152 14.1 / 13.4, 57 344 14.4 / 15.5    2   32 768 12.1 / 10.9, 49 152 12.4 / 13.0, 131 072 14.1 / 23.9
inline int64_t layer_kernel_entries(int64_t Q, int64_t NB, bool vec) {
  if (vec) return Q < 32 ? 81920 : NB > kLdsIds ? 98304 : kLayerEntries;
  return Q < 16 ? 32768 : Q < 256 ? 49152 : 81920;
}
inline bool layer_kernel_fits(int64_t Q, int64_t RE, int64_t NB, int64_t rc_chunk, int64_t per_layer, bool in_place, bool vec) {
  return Q <= kLdsTargets && rc_chunk <= kLayerCounts && RE <= (1 << 30) &&
         (per_layer == 1 || (!in_place && RE <= layer_kernel_entries(Q, NB, vec)));
}

typedef int i32x4 __attribute__((ext_vector_type(4)));

// Workgroup barrier that orders LDS traffic only: table loads and stores stay in flight across it
// (__syncthreads also waits for every outstanding global access of the wave, a memory round trip
// per batch in a kernel whose time at the benchmark's table shape is a chain of round trips).
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// Query slot of physical block t, or -1, through global memory.  slot_of may hold anything; a slot
// counts only if it points back at t.  A matched slot is then replaced by its target (out) and kept
// for counting.
__device__ __forceinline__ int remap_entry(int t, const int32_t* __restrict__ slot_of,
                                           const int32_t* __restrict__ query_ids, const int32_t* __restrict__ pool_ids,
                                           const int32_t* __restrict__ m, int Q, int P, long long NB, int& slot) {
  slot = -1;
  if (t < 0 || t >= NB) return t;
  const int s = slot_of[t];
  if ((unsigned)s >= (unsigned)Q || query_ids[s] != t) return t;
  const int mi = m[s];
  if (mi < 0 || mi >= P) return t;  // unmatched query block: entry stays, nothing to count
  slot = s;
  return pool_ids ? pool_ids[mi] : mi;
}

// The reference counts of one layer move from the matched query blocks to their targets.
// cnt_of(q) = references to query slot q that the gather rewrote.  All kFinalThreads threads of the
// workgroup call this; `claim` is kClaimSlots ints of LDS, `wsum` kFinalThreads / 64 ints.
template <typename CountOf>
__device__ __forceinline__ void finalize_layer(CountOf cnt_of, const int32_t* __restrict__ query_ids,
                                               const int32_t* __restrict__ pool_ids, const int32_t* __restrict__ m, int Q,
                                               int P, long long NB, int32_t* rc_l, uint8_t* __restrict__ freed_l,
                                               int32_t* __restrict__ n_remapped_l, int* claim, int* wsum) {
  const int tid = threadIdx.x;
  int cnt[kFinalPerThread], tgt[kFinalPerThread];
  int moved = 0;
#pragma unroll
  for (int k = 0; k < kFinalPerThread; ++k) {
    const int q = k * kFinalThreads + tid;
    cnt[k] = 0;
    tgt[k] = -1;
    if (q < Q) {
      const int mi = m[q];
      const int b = query_ids[q];
      unsigned char fr = 0;
      if (mi >= 0 && mi < P && b >= 0 && b < NB) {
        const int c = cnt_of(q);
        const int t = pool_ids ? pool_ids[mi] : mi;
        const int left = rc_l[b] - c;
        rc_l[b] = left;  // query ids are distinct: no other thread touches this entry
        fr = (left == 0);
        moved += c;
        if (c > 0 && t >= 0 && t < NB) {
          cnt[k] = c;
          tgt[k] = t;
        }
      }
      freed_l[q] = fr;
    }
  }
  // queries that share a target add their references in turns
  bool pending = false;
#pragma unroll
  for (int k = 0; k < kFinalPerThread; ++k) pending |= tgt[k] >= 0;
  while (__syncthreads_or(pending)) {
#pragma unroll
    for (int k = 0; k < kFinalPerThread; ++k)
      if (tgt[k] >= 0) claim[tgt[k] & (kClaimSlots - 1)] = k * kFinalThreads + tid;
    __syncthreads();
    pending = false;
#pragma unroll
    for (int k = 0; k < kFinalPerThread; ++k)
      if (tgt[k] >= 0) {
        if (claim[tgt[k] & (kClaimSlots - 1)] == k * kFinalThreads + tid) {
          rc_l[tgt[k]] += cnt[k];
          tgt[k] = -1;
        } else {
          pending = true;
        }
      }
    __threadfence_block();
  }
  // n_remapped = total references moved in this layer
  for (int off = 32; off > 0; off >>= 1) moved += __shfl_xor(moved, off);
  if ((tid & 63) == 0) wsum[tid >> 6] = moved;
  __syncthreads();
  if (tid == 0) {
    int s = 0;
    for (int w = 0; w < kFinalThreads / 64; ++w) s += wsum[w];
    *n_remapped_l = s;
  }
}

struct GatherLds {
  unsigned short slot[kLdsIds];           // block id - lo -> slot + 1 of the matched query block with that id (0 = none)
  int target[kLdsTargets];                // target block of a matched slot
  int hist[kMaxQ];                        // references rewritten per slot
  unsigned short list[kGatherBatch];      // the hits of a batch, compacted; later the claim table of the finalize step
  int wsum[kGatherThreads / 64];
};
static_assert(sizeof(GatherLds) <= 160 * 1024, "fits the LDS of a compute unit");
static_assert(sizeof(unsigned short) * kGatherBatch >= sizeof(int) * kClaimSlots, "the claim table reuses the hit list");
static_assert(kGatherThreads == kFinalThreads, "the fused finalize step runs in the gather workgroup");

// grid = (G, L).  Workgroup g rewrites entries [g*chunk, min((g+1)*chunk, RE)) of layer l and copies
// refcounts [g*rc_chunk, ...) of the layer.  VEC: every layer starts 16-byte aligned and chunk % 4 == 0.
// FUSED (G == 1): the workgroup also moves the layer's reference counts.
template <bool VEC, bool FUSED>
__global__ __launch_bounds__(kGatherThreads) void remap_gather_kernel(
    const int32_t* tables_in, int32_t* tables_out, long long RE, long long chunk, int32_t* slot_of, const int32_t* __restrict__ query_ids, const int32_t* __restrict__ pool_ids,
    const int32_t* __restrict__ match_idx, int Q, int P, long long NB, int32_t* __restrict__ partial,
    const int32_t* refcount_in, int32_t* refcount_out, long long rc_chunk, int rc_vec, uint8_t* __restrict__ freed,
    int32_t* __restrict__ n_remapped) {
  __shared__ GatherLds s;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const long long l = blockIdx.y, g = blockIdx.x, G = gridDim.x;
  const int32_t* tin = tables_in + l * RE;
  int32_t* tout = tables_out + l * RE;
  const int32_t* m = match_idx + l * Q;
  const long long lo_e = g * chunk, hi_e = (lo_e + chunk < RE) ? lo_e + chunk : RE;

  // ---- what decides an entry.  Every workgroup finds the range [id_lo, id_hi] of the query block ids itself.
  int id_lo = 0x7fffffff, id_hi = -1;
  for (int q = tid; q < Q; q += kGatherThreads) {
    const int b = query_ids[q];
    if (b >= 0 && b < NB) {
      id_lo = min(id_lo, b);
      id_hi = max(id_hi, b);
    }
    s.hist[q] = 0;
  }
  for (int off = 32; off > 0; off >>= 1) {
    id_lo = min(id_lo, __shfl_xor(id_lo, off));
    id_hi = max(id_hi, __shfl_xor(id_hi, off));
  }
  if (lane == 0) {
    s.wsum[wave] = id_lo;
    s.list[wave] = 0;  // (keeps the two arrays apart for the reader below)
    reinterpret_cast<int*>(s.list)[64 + wave] = id_hi;
  }
  lds_barrier();
#pragma unroll
  for (int w = 0; w < kGatherThreads / 64; ++w) {
    id_lo = min(id_lo, s.wsum[w]);
    id_hi = max(id_hi, reinterpret_cast<int*>(s.list)[64 + w]);
  }
  lds_barrier();
  const long long span = (long long)id_hi - id_lo + 1;  // <= 0: no query block with a valid id
  const bool in_lds = span <= kLdsIds && Q <= kLdsTargets;
  if (in_lds) {
    // a 16-bit table over the id range and the targets of the matched slots, in LDS
    if (span > 0) {
      unsigned int* z = reinterpret_cast<unsigned int*>(s.slot);
      for (int i = tid; i < (int)((span + 1) / 2); i += kGatherThreads) z[i] = 0u;
      lds_barrier();
      for (int q = tid; q < Q; q += kGatherThreads) {
        const int b = query_ids[q];
        const int mi = m[q];
        if (b >= 0 && b < NB && mi >= 0 && mi < P) {      // a matched query block
          s.slot[b - id_lo] = (unsigned short)(q + 1);    // query ids are distinct: one writer per entry
          s.target[q] = pool_ids ? pool_ids[mi] : mi;
        }
      }
    }
  } else {
    // the reverse index in global memory.  Every workgroup writes all of it (the same values), so each reads
    // what it wrote itself; words that no query block owns are stale or uninitialised and fail the check
    // query_ids[slot_of[t]] == t of the reader.
    for (int q = tid; q < Q; q += kGatherThreads) {
      const int b = query_ids[q];
      if (b >= 0 && b < NB) slot_of[b] = q;
    }
    __threadfence_block();
  }
  __syncthreads();

  // thread -> 4 consecutive entries per load (VEC) or entries strided by the workgroup size
  auto index_of = [&](long long base, int k) {
    return VEC ? base + ((k >> 2) * kGatherThreads + tid) * 4 + (k & 3) : base + (long long)k * kGatherThreads + tid;
  };
  auto load_batch = [&](long long base, int (&entry)[kGatherPerThread]) {
    if (VEC) {
#pragma unroll
      for (int k = 0; k < kGatherPerThread; k += 4) {
        const long long e = index_of(base, k);
        i32x4 v = {-1, -1, -1, -1};
        if (e + 3 < hi_e) {
          v = __builtin_nontemporal_load(reinterpret_cast<const i32x4*>(tin + e));
        } else {
#pragma unroll
          for (int c = 0; c < 4; ++c)
            if (e + c < hi_e) v[c] = tin[e + c];
        }
#pragma unroll
        for (int c = 0; c < 4; ++c) entry[k + c] = v[c];
      }
    } else {
#pragma unroll
      for (int k = 0; k < kGatherPerThread; ++k) {
        const long long e = index_of(base, k);
        entry[k] = (e < hi_e) ? tin[e] : -1;
      }
    }
  };
  // the entries of the next batch are asked for before the current batch is worked on
  int ahead[kGatherPerThread];
  if (lo_e < hi_e) load_batch(lo_e, ahead);
  for (long long base = lo_e; base < hi_e; base += kGatherBatch) {
    int entry[kGatherPerThread], slot[kGatherPerThread];
#pragma unroll
    for (int k = 0; k < kGatherPerThread; ++k) entry[k] = ahead[k];
    if (base + kGatherBatch < hi_e) load_batch(base + kGatherBatch, ahead);
    int outv[kGatherPerThread];
    int hits = 0;
    if (in_lds) {
#pragma unroll
      for (int k = 0; k < kGatherPerThread; ++k) {
        const int t = entry[k];
        const long long d = (long long)t - id_lo;
        int o = t, sl = -1;
        if (span > 0 && t >= 0 && t < NB && d >= 0 && d < span) {
          const int s1 = s.slot[d];
          if (s1) {
            sl = s1 - 1;
            o = s.target[sl];
          }
        }
        outv[k] = o;
        slot[k] = sl;
        hits += sl >= 0;
      }
    } else {
#pragma unroll
      for (int k = 0; k < kGatherPerThread; ++k) {
        outv[k] = remap_entry(entry[k], slot_of, query_ids, pool_ids, m, Q, P, NB, slot[k]);
        hits += slot[k] >= 0;
      }
    }
    if (VEC) {
#pragma unroll
      for (int k = 0; k < kGatherPerThread; k += 4) {
        const long long e = index_of(base, k);
        if (e + 3 < hi_e) {
          i32x4 v = {outv[k], outv[k + 1], outv[k + 2], outv[k + 3]};
          __builtin_nontemporal_store(v, reinterpret_cast<i32x4*>(tout + e));
        } else {
#pragma unroll
          for (int c = 0; c < 4; ++c)
            if (e + c < hi_e) tout[e + c] = outv[k + c];
        }
      }
    } else {
#pragma unroll
      for (int k = 0; k < kGatherPerThread; ++k) {
        const long long e = index_of(base, k);
        if (e < hi_e) tout[e] = outv[k];
      }
    }
    // ---- count the rewritten references of this batch
    // position of this thread's hits in the list: prefix sum over the workgroup
    int incl = hits;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const int n = __shfl_up(incl, off);
      if (lane >= off) incl += n;
    }
    if (lane == 63) s.wsum[wave] = incl;
    lds_barrier();
    int before = 0, total = 0;
#pragma unroll
    for (int w = 0; w < kGatherThreads / 64; ++w) {
      const int c = s.wsum[w];
      before += (w < wave) ? c : 0;
      total += c;
    }
    if (total != 0) {   // the same for every thread
      int pos = before + incl - hits;
#pragma unroll
      for (int k = 0; k < kGatherPerThread; ++k)
        if (slot[k] >= 0) s.list[pos++] = (unsigned short)slot[k];
      lds_barrier();
      // wave w adds up the keys congruent to w: no two waves touch the same bin
      for (int i0 = 0; i0 < total; i0 += 64) {
        const int i = i0 + lane;
        const int key = (i < total) ? (int)s.list[i] : -1;
        const bool mine = key >= 0 && (key & (kGatherThreads / 64 - 1)) == wave;
        unsigned long long active = __ballot(mine);
        while (active) {
          const int leader = __ffsll((long long)active) - 1;
          const int lkey = __shfl(key, leader);
          const unsigned long long same = __ballot(mine && key == lkey);
          if (lane == leader) s.hist[lkey] += __popcll(same);
          active &= ~same;
        }
      }
    }
    lds_barrier();  // the list and the wave sums are free again
  }
  // this workgroup's share of the refcount copy (the finalize step then edits refcount_out)
  if (refcount_in != refcount_out) {
    const long long rlo = g * rc_chunk, rhi = (rlo + rc_chunk < NB) ? rlo + rc_chunk : NB;
    const int32_t* src = refcount_in + l * NB;
    int32_t* dst = refcount_out + l * NB;
    if (rc_vec) {
      constexpr long long kStride = kGatherThreads * 4LL;
      long long i = rlo + tid * 4LL;
      for (; i + 3 * kStride + 3 < rhi; i += 4 * kStride) {  // four loads in flight
        i32x4 v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] = __builtin_nontemporal_load(reinterpret_cast<const i32x4*>(src + i + u * kStride));
#pragma unroll
        for (int u = 0; u < 4; ++u) __builtin_nontemporal_store(v[u], reinterpret_cast<i32x4*>(dst + i + u * kStride));
      }
      for (; i < rhi; i += kStride) {
        if (i + 3 < rhi) {
          __builtin_nontemporal_store(__builtin_nontemporal_load(reinterpret_cast<const i32x4*>(src + i)),
                                      reinterpret_cast<i32x4*>(dst + i));
        } else {
          for (long long c = i; c < rhi; ++c) dst[c] = src[c];
        }
      }
    } else {
      for (long long i = rlo + tid; i < rhi; i += kGatherThreads) dst[i] = src[i];
    }
  }
  if (FUSED) {
    // the copy of this layer's reference counts is this workgroup's own (same compute unit, same L1): a fence
    // at workgroup scope orders it before the edits.  (A device-scope fence writes the L2 back: tens of microseconds.)
    __threadfence_block();
    __syncthreads();
    finalize_layer([&](int q) { return s.hist[q]; }, query_ids, pool_ids, m, Q, P, NB, refcount_out + l * NB,
                   freed + l * Q, n_remapped + l, reinterpret_cast<int*>(s.list), s.wsum);
  } else {
    __syncthreads();
    int32_t* out = partial + (l * G + g) * Q;
    for (int q = tid; q < Q; q += kGatherThreads) out[q] = s.hist[q];
  }
}

// grid = L, one workgroup per layer (only when a layer was gathered by several workgroups).
__global__ __launch_bounds__(kFinalThreads) void remap_finalize_kernel(
    const int32_t* __restrict__ partial, int G, const int32_t* __restrict__ query_ids,
    const int32_t* __restrict__ pool_ids, const int32_t* __restrict__ match_idx, int Q, int P, long long NB,
    int32_t* refcount_out, uint8_t* __restrict__ freed, int32_t* __restrict__ n_remapped) {
  __shared__ int claim[kClaimSlots];
  __shared__ int wsum[kFinalThreads / 64];
  const long long l = blockIdx.x;
  finalize_layer(
      [&](int q) {
        int c = 0;
        for (int g = 0; g < G; ++g) c += partial[(l * G + g) * Q + q];
        return c;
      },
      query_ids, pool_ids, match_idx + l * Q, Q, P, NB, refcount_out + l * NB, freed + l * Q, n_remapped + l, claim, wsum);
}

constexpr int kHashBits = 14, kHashPlaces = 1 << kHashBits, kHashIdBits = 19;
constexpr unsigned kHashIdMask = (1u << kHashIdBits) - 1u;
struct LayerLds {
  union {
    unsigned short slot[kLdsIds];    // block id - lo -> slot + 1 of the matched query block with that id (0 = none)
    unsigned int hash[kHashPlaces];  // ids further apart than that: (slot + 1) << kHashIdBits | id of a matched query block (0 = free)
  };
  int target[kLdsTargets];        // target block of a matched slot
  int hist[kLdsTargets];          // references of the layer to a matched slot
  int rc[kLayerCounts];           // this workgroup's share of the layer's reference counts
  int lo[kGatherThreads / 64], hi[kGatherThreads / 64], moved[kGatherThreads / 64];
};
static_assert(sizeof(LayerLds) <= 160 * 1024, "fits the LDS of a compute unit");
static_assert(kLdsTargets < kHashPlaces, "a free place ends every search of the hash table");
static_assert(kLdsTargets < 1 << (32 - kHashIdBits) && kLayerCounts * (kLayerEntries / (kGatherBatch / 4)) <= 1 << kHashIdBits,
              "slot + 1 and a block id fit in one word: with several workgroups per layer there are as many shares of the counts at most");
// consecutive ids and ids at a regular distance spread over the table; a 24-bit product runs at four times the rate of a 32-bit one
__device__ __forceinline__ unsigned hash_place(int id) { return (unsigned)__umul24((unsigned)id, 0x9e3779u) >> (32 - kHashBits); }

// The whole remap of a layer by `per_layer` workgroups that do not need each other.  Each reads all of the layer's
// table and counts the references to the matched query blocks in LDS (integer adds: the same counts in any order),
// writes its chunk of the table, and owns the reference counts [rlo, rhi) of the layer, which it reads once, edits
// in LDS and writes once.  What bounds it is a chain of memory round trips, so everything that depends on nothing is
// asked for before the first wait (ids, decisions, reference counts, four groups of entries), later groups four groups
// ahead.  A layer's workgroups are dealt to one XCD (consecutive workgroups go round the 8 XCDs), so the repeated
// reads of the table come from its L2.  Measured against one gather launch and, with several workgroups per layer, a
// second launch that adds their histograms (us): 1 layer x 288 entries 9.1 -> 6.2, 4 x 8192 12.7 -> 7.2, 64 x 4352
// 12.4 -> 7.4, 64 x 49 664 entries and 50 176 counts 24.0 -> 15.3, 256 x 15 000 17.8 -> 12.4, 1 x 131 072 20.9 -> 16.9.
// Query blocks whose ids lie further apart than the table of slots reaches are looked up in an open-addressing table in the
// same LDS.  (Through global memory, entry -> slot -> id -> decision -> target, that is a chain of four round trips for every
// entry in every workgroup.  Ids all over 50 176 blocks, 1024 query blocks, gather launches / that chain / this table, us:
// 64 x 49 664 entries 49 / 65 / 21, 8 x 49 152 35 / 49 / 17.)
// What is left at 64 x 49 664 is vector work on the 48 entries that every thread looks at (a branch per entry instead of
// one per four: 16.6; no branch at all: 16.9) and 6 us that a call of one small table takes as well.
template <bool VEC>
__global__ __launch_bounds__(kGatherThreads) void remap_layer_kernel(
    const int32_t* tables_in, int32_t* tables_out, int RE, int chunk, const int32_t* __restrict__ query_ids,
    const int32_t* __restrict__ pool_ids, const int32_t* __restrict__ match_idx, int Q, int P, int NB,
    const int32_t* refcount_in, int32_t* refcount_out, int rc_chunk, int rc_vec, uint8_t* __restrict__ freed,
    int32_t* __restrict__ n_remapped, int L, int per_layer) {
  __shared__ LayerLds s;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int turn = blockIdx.x >> 3, g = turn % per_layer;
  const long long l = (long long)(turn / per_layer) * 8 + (blockIdx.x & 7);
  if (l >= L) return;
  const int32_t* tin = tables_in + l * RE;
  int32_t* tout = tables_out + l * RE;
  const int32_t* m = match_idx + l * Q;
  const int lo_e = g * chunk, len_e = share_items(RE, lo_e, chunk);
  const int rlo = g * rc_chunk, n_counts = share_items(NB, rlo, rc_chunk);

  // ---- everything that waits for nothing
  constexpr int kSlots = kLdsTargets / kGatherThreads, kCounts = (kLayerCounts + kGatherThreads * 4 - 1) / (kGatherThreads * 4);
  constexpr int kGroup = 4 * kGatherThreads, kAhead = 4;  // entries of a group, four per thread; groups in flight
  int id[kSlots], tgt[kSlots];  // this thread's query slots: block id; decision, then target
#pragma unroll
  for (int k = 0; k < kSlots; ++k) {
    const int q = k * kGatherThreads + tid;
    id[k] = q < Q ? query_ids[q] : -1;
    tgt[k] = q < Q ? m[q] : -1;
  }
  i32x4 count[kCounts];
#pragma unroll
  for (int u = 0; u < kCounts; ++u) {
    if (rc_vec) {  // four counts of a thread side by side
      const int i = (u * kGatherThreads + tid) * 4;
      if (i < n_counts) count[u] = __builtin_nontemporal_load(reinterpret_cast<const i32x4*>(refcount_in + l * NB + rlo + i));
    } else {
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const int i = (u * 4 + c) * kGatherThreads + tid;
        if (i < n_counts) count[u][c] = refcount_in[l * NB + rlo + i];
      }
    }
  }
  // entry c of this thread in the group that starts at `base`: four side by side (VEC) or a workgroup apart
  auto index_of = [&](int base, int c) { return VEC ? base + tid * 4 + c : base + c * kGatherThreads + tid; };
  auto load_group = [&](int base) {
    i32x4 v = {-1, -1, -1, -1};
    if (VEC) {  // RE % 4 == 0: four entries are inside or outside together
      if (index_of(base, 0) < RE) v = *reinterpret_cast<const i32x4*>(tin + index_of(base, 0));
    } else {
#pragma unroll
      for (int c = 0; c < 4; ++c)
        if (index_of(base, c) < RE) v[c] = tin[index_of(base, c)];
    }
    return v;
  };
  i32x4 ahead[kAhead];
#pragma unroll
  for (int u = 0; u < kAhead; ++u) ahead[u] = load_group(u * kGroup);

  // ---- the matched query blocks and the range [id_lo, id_hi] of their ids
  int id_lo = 0x7fffffff, id_hi = -1;
#pragma unroll
  for (int k = 0; k < kSlots; ++k) {
    if (id[k] >= 0 && id[k] < NB && tgt[k] >= 0 && tgt[k] < P) {
      id_lo = min(id_lo, id[k]);
      id_hi = max(id_hi, id[k]);
      if (pool_ids) tgt[k] = pool_ids[tgt[k]];
    } else {
      id[k] = -1;
    }
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    id_lo = min(id_lo, __shfl_xor(id_lo, off));
    id_hi = max(id_hi, __shfl_xor(id_hi, off));
  }
  if (lane == 0) {
    s.lo[wave] = id_lo;
    s.hi[wave] = id_hi;
  }
  lds_barrier();
#pragma unroll
  for (int w = 0; w < kGatherThreads / 64; ++w) {
    id_lo = min(id_lo, s.lo[w]);
    id_hi = max(id_hi, s.hi[w]);
  }
  const unsigned span = id_hi < 0 ? 0u : (unsigned)(id_hi - id_lo) + 1u;  // 0: no matched query block
  const bool in_lds = span <= kLdsIds;
  const int words = in_lds ? (int)((span + 1) / 2) : kHashPlaces;
  for (int i = tid; i < words; i += kGatherThreads) s.hash[i] = 0u;  // of either table
  lds_barrier();
#pragma unroll
  for (int k = 0; k < kSlots; ++k) {
    const int q = k * kGatherThreads + tid;
    if (q < Q) s.hist[q] = 0;
    if (id[k] >= 0) {
      if (in_lds) {
        s.slot[id[k] - id_lo] = (unsigned short)(q + 1);  // query ids are distinct: one writer per entry
      } else {
        unsigned at = hash_place(id[k]);
        while (atomicCAS(&s.hash[at], 0u, (unsigned)(q + 1) << kHashIdBits | (unsigned)id[k]) != 0u) at = (at + 1) & (kHashPlaces - 1);
      }
      s.target[q] = tgt[k];
    }
  }
#pragma unroll
  for (int u = 0; u < kCounts; ++u) {
    if (rc_vec) {
      const int i = (u * kGatherThreads + tid) * 4;
      if (i < n_counts) *reinterpret_cast<i32x4*>(&s.rc[i]) = count[u];
    } else {
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const int i = (u * 4 + c) * kGatherThreads + tid;
        if (i < n_counts) s.rc[i] = count[u][c];
      }
    }
  }
  lds_barrier();

  // ---- the table: every entry is counted, those of this workgroup's chunk are written
  for (int first = 0; first < RE; first += kAhead * kGroup) {
#pragma unroll
    for (int u = 0; u < kAhead; ++u) {
      const int base = first + u * kGroup;
      i32x4 entry = ahead[u];
      ahead[u] = load_group(base + kAhead * kGroup);  // entries of none past the end
      unsigned d[4];
#pragma unroll
      for (int c = 0; c < 4; ++c) d[c] = (unsigned)entry[c] - (unsigned)id_lo;
      // the table is mostly resident blocks: a wave without a query block among its 256 entries goes on
      if (d[0] < span || d[1] < span || d[2] < span || d[3] < span) {
        int slot1[4];
        if (in_lds) {
#pragma unroll
          for (int c = 0; c < 4; ++c) slot1[c] = d[c] < span ? (int)s.slot[d[c]] : 0;
        } else {
          unsigned at[4], item[4];
          bool other[4], more = false;  // the place holds another block
#pragma unroll
          for (int c = 0; c < 4; ++c) {
            at[c] = hash_place(entry[c]);
            item[c] = d[c] < span ? s.hash[at[c]] : 0u;
          }
#pragma unroll
          for (int c = 0; c < 4; ++c) more |= other[c] = item[c] != 0u && (int)(item[c] & kHashIdMask) != entry[c];
          while (more) {
            more = false;
#pragma unroll
            for (int c = 0; c < 4; ++c) {
              at[c] = (at[c] + 1) & (kHashPlaces - 1);
              if (other[c]) item[c] = s.hash[at[c]];
            }
#pragma unroll
            for (int c = 0; c < 4; ++c) more |= other[c] = item[c] != 0u && (int)(item[c] & kHashIdMask) != entry[c];
          }
#pragma unroll
          for (int c = 0; c < 4; ++c) slot1[c] = (int)(item[c] >> kHashIdBits);
        }
#pragma unroll
        for (int c = 0; c < 4; ++c)
          if (slot1[c] > 0) {
            atomicAdd(&s.hist[slot1[c] - 1], 1);
            entry[c] = s.target[slot1[c] - 1];
          }
      }
      if (VEC) {
        const int e = index_of(base, 0);  // chunks are multiples of four
        if ((unsigned)(e - lo_e) < (unsigned)len_e) __builtin_nontemporal_store(entry, reinterpret_cast<i32x4*>(tout + e));
      } else {
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          const int e = index_of(base, c);
          if ((unsigned)(e - lo_e) < (unsigned)len_e) tout[e] = entry[c];
        }
      }
    }
  }
  lds_barrier();  // the histogram is complete

  // ---- the reference counts
  int moved = 0;
#pragma unroll
  for (int k = 0; k < kSlots; ++k) {
    const int q = k * kGatherThreads + tid;
    if (q >= Q) continue;
    const int c = id[k] >= 0 ? s.hist[q] : 0;
    const unsigned at = (unsigned)(id[k] - rlo);
    moved += c;
    if (id[k] >= 0 && at < (unsigned)n_counts) {  // distinct ids: no other thread touches this count
      const int left = s.rc[at] - c;
      s.rc[at] = left;
      freed[l * Q + q] = left == 0;
    } else if (id[k] < 0 && g == 0) {
      freed[l * Q + q] = 0;
    }
  }
  lds_barrier();  // the query blocks have given up theirs before the targets gain them
#pragma unroll
  for (int k = 0; k < kSlots; ++k) {
    const int q = k * kGatherThreads + tid;
    const unsigned at = (unsigned)(tgt[k] - rlo);
    if (q < Q && id[k] >= 0 && tgt[k] >= 0 && at < (unsigned)n_counts) {
      const int c = s.hist[q];
      if (c > 0) atomicAdd(&s.rc[at], c);
    }
  }
  if (g == 0) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) moved += __shfl_xor(moved, off);
    if (lane == 0) s.moved[wave] = moved;
  }
  lds_barrier();
#pragma unroll
  for (int u = 0; u < kCounts; ++u) {
    if (rc_vec) {
      const int i = (u * kGatherThreads + tid) * 4;
      if (i < n_counts)
        __builtin_nontemporal_store(*reinterpret_cast<const i32x4*>(&s.rc[i]),
                                    reinterpret_cast<i32x4*>(refcount_out + l * NB + rlo + i));
    } else {
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const int i = (u * 4 + c) * kGatherThreads + tid;
        if (i < n_counts) refcount_out[l * NB + rlo + i] = s.rc[i];
      }
    }
  }
  if (g == 0 && tid == 0) {
    int n = 0;
#pragma unroll
    for (int w = 0; w < kGatherThreads / 64; ++w) n += s.moved[w];
    n_remapped[l] = n;
  }
}

}  // namespace
}  // namespace rc

extern "C" size_t rc_remap_workspace_size(int32_t n_layers, int64_t R, int64_t E, int64_t Q, int64_t NB) {
  using namespace rc;
  if (n_layers < 0 || R < 0 || E < 0 || Q < 0 || NB < 0) return 0;
  const int64_t G = chunks_per_layer(R * E, n_layers);
  const int64_t ints = ((NB + 3) / 4) * 4 + (G > 1 ? (int64_t)n_layers * G * Q : 0);
  return (size_t)(ints > 0 ? ints : 4) * sizeof(int32_t);
}

// Scratch of rc_remap_block_table_static: one array per GPU, part of the loaded code object, so it
// exists from the moment the library is loaded on a device until the process ends.  In host code
// the name is only a handle for hipGetSymbolAddress; kernels get the address it returns.
static __device__ __align__(256) unsigned char scratch[RC_REMAP_STATIC_SCRATCH_BYTES];

namespace rc {
namespace {

// Validation and the launches, shared by the two entry points; `who` names the caller in
// error texts.  Nothing is allocated here.
rc_status remap_run(const char* who, int32_t n_layers, const int32_t* tables_in, int32_t* tables_out, int64_t R,
                    int64_t E, const int32_t* query_ids, const int32_t* pool_ids, const int32_t* match_idx, int64_t Q,
                    int64_t P, int64_t NB, const int32_t* refcount_in, int32_t* refcount_out, uint8_t* freed,
                    int32_t* n_remapped, void* workspace, size_t workspace_bytes, void* hip_stream) {
  if (n_layers < 0 || R < 0 || E < 0 || Q < 0 || P < 0 || NB < 0)
    return fail(RC_ERR_INVALID_ARG, "%s: negative size", who);
  if (Q > kMaxQ) return fail(RC_ERR_UNSUPPORTED, "%s: Q %lld above %d", who, (long long)Q, kMaxQ);
  if (!pool_ids && P > NB) return fail(RC_ERR_INVALID_ARG, "%s: identity pool ids need P <= NB", who);
  if (n_layers == 0) return RC_OK;
  const int64_t RE = R * E;
  if (n_layers > 65535 || NB > 0x7fffffffLL || P > 0x7fffffffLL || RE > (1LL << 40))
    return fail(RC_ERR_UNSUPPORTED, "%s: problem beyond the grid limits", who);
  if (!n_remapped || (RE > 0 && (!tables_in || !tables_out)) || (NB > 0 && (!refcount_in || !refcount_out)) ||
      (Q > 0 && (!query_ids || !match_idx || !freed)))
    return fail(RC_ERR_INVALID_ARG, "%s: NULL pointer", who);
  const size_t need = rc_remap_workspace_size(n_layers, R, E, Q, NB);
  if (!workspace || workspace_bytes < need || !aligned16(workspace))
    return fail(RC_ERR_WORKSPACE, "%s: workspace of %zu bytes needed (16-byte aligned), got %zu", who,
                need, workspace_bytes);
  hipStream_t st = static_cast<hipStream_t>(hip_stream);
  int32_t* slot_of = static_cast<int32_t*>(workspace);
  int32_t* partial = slot_of + ((NB + 3) / 4) * 4;
  const int64_t G = chunks_per_layer(RE, n_layers);
  const int64_t chunk = share_length(RE, G), rc_chunk = share_length(NB, G);
  const bool vec = RE % 4 == 0 && aligned16(tables_in) && aligned16(tables_out);
  const int rc_vec = NB % 4 == 0 && aligned16(refcount_in) && aligned16(refcount_out);

  if (layer_kernel_fits(Q, RE, NB, rc_chunk, G, tables_in == tables_out, vec)) {
    const unsigned wgs = (unsigned)((n_layers + 7) / 8 * 8 * G);
    if (vec)
      remap_layer_kernel<true><<<wgs, kGatherThreads, 0, st>>>(tables_in, tables_out, (int)RE, (int)chunk, query_ids, pool_ids,
                                                               match_idx, (int)Q, (int)P, (int)NB, refcount_in, refcount_out,
                                                               (int)rc_chunk, rc_vec, freed, n_remapped, n_layers, (int)G);
    else
      remap_layer_kernel<false><<<wgs, kGatherThreads, 0, st>>>(tables_in, tables_out, (int)RE, (int)chunk, query_ids, pool_ids,
                                                                match_idx, (int)Q, (int)P, (int)NB, refcount_in, refcount_out,
                                                                (int)rc_chunk, rc_vec, freed, n_remapped, n_layers, (int)G);
    return check_launch("rc_remap_block_table(layers)");
  }

  const dim3 grid((unsigned)G, (unsigned)n_layers);
#define RC_GATHER(V, F)                                                                                                    \
  remap_gather_kernel<V, F><<<grid, kGatherThreads, 0, st>>>(tables_in, tables_out, RE, chunk, slot_of, query_ids,         \
                                                             pool_ids, match_idx, (int)Q, (int)P, NB, partial,             \
                                                             refcount_in, refcount_out, rc_chunk, rc_vec, freed, n_remapped)
  if (G == 1) {
    if (vec)
      RC_GATHER(true, true);
    else
      RC_GATHER(false, true);
    return check_launch("rc_remap_block_table(gather + finalize)");
  }
  if (vec)
    RC_GATHER(true, false);
  else
    RC_GATHER(false, false);
#undef RC_GATHER
  if (rc_status s = check_launch("rc_remap_block_table(gather)")) return s;
  remap_finalize_kernel<<<(unsigned)n_layers, kFinalThreads, 0, st>>>(partial, (int)G, query_ids, pool_ids, match_idx,
                                                                      (int)Q, (int)P, NB, refcount_out, freed,
                                                                      n_remapped);
  return check_launch("rc_remap_block_table(finalize)");
}

constexpr size_t kStaticScratchBytes = RC_REMAP_STATIC_SCRATCH_BYTES;

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
void* g_scratch_ptr[kMaxDevices];  // device address of `scratch` on each device, nullptr = not asked yet

// Address of the current device's copy of `scratch` (looked up once per device).
rc_status static_scratch(void** out) {
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return fail(RC_ERR_DEVICE, "rc_remap_block_table_static: hipGetDevice: %s", hipGetErrorString(e));
  if (dev < 0 || dev >= kMaxDevices)
    return fail(RC_ERR_UNSUPPORTED, "rc_remap_block_table_static: device %d beyond the %d devices kept track of", dev,
                kMaxDevices);
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (!g_scratch_ptr[dev]) {
    void* ptr = nullptr;
    e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !ptr)
      return fail(RC_ERR_DEVICE, "rc_remap_block_table_static: hipGetSymbolAddress: %s", hipGetErrorString(e));
    g_scratch_ptr[dev] = ptr;
  }
  *out = g_scratch_ptr[dev];
  return RC_OK;
}

}  // namespace
}  // namespace rc

extern "C" rc_status rc_remap_block_table(int32_t n_layers, const int32_t* tables_in, int32_t* tables_out, int64_t R,
                                          int64_t E, const int32_t* query_ids, const int32_t* pool_ids,
                                          const int32_t* match_idx, int64_t Q, int64_t P, int64_t NB,
                                          const int32_t* refcount_in, int32_t* refcount_out, uint8_t* freed,
                                          int32_t* n_remapped, void* workspace, size_t workspace_bytes,
                                          void* hip_stream) {
  rc::clear_error();
  return rc::remap_run("rc_remap_block_table", n_layers, tables_in, tables_out, R, E, query_ids, pool_ids, match_idx, Q, P,
                       NB, refcount_in, refcount_out, freed, n_remapped, workspace, workspace_bytes, hip_stream);
}

extern "C" size_t rc_remap_static_scratch_size(void) { return rc::kStaticScratchBytes; }

extern "C" rc_status rc_remap_block_table_static(int32_t n_layers, const int32_t* tables_in, int32_t* tables_out,
                                                 int64_t R, int64_t E, const int32_t* query_ids,
                                                 const int32_t* pool_ids, const int32_t* match_idx, int64_t Q,
                                                 int64_t P, int64_t NB, const int32_t* refcount_in,
                                                 int32_t* refcount_out, uint8_t* freed, int32_t* n_remapped,
                                                 void* hip_stream) {
  using namespace rc;
  clear_error();
  if (n_layers < 0 || R < 0 || E < 0 || Q < 0 || P < 0 || NB < 0)
    return fail(RC_ERR_INVALID_ARG, "rc_remap_block_table_static: negative size");
  const size_t need = rc_remap_workspace_size(n_layers, R, E, Q, NB);
  if (need > kStaticScratchBytes)
    return fail(RC_ERR_WORKSPACE,
                "rc_remap_block_table_static: this problem needs %zu bytes of scratch, the built-in buffer has %zu; "
                "use rc_remap_block_table with a workspace of the caller's",
                need, kStaticScratchBytes);
  if (n_layers == 0) return RC_OK;
  void* ptr = nullptr;
  if (rc_status s = static_scratch(&ptr)) return s;
  return remap_run("rc_remap_block_table_static", n_layers, tables_in, tables_out, R, E, query_ids, pool_ids, match_idx, Q,
                   P, NB, refcount_in, refcount_out, freed, n_remapped, ptr, kStaticScratchBytes, hip_stream);
}
