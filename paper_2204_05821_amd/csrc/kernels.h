// Device kernels of the k-bisimulation refinement step for gfx950 (CDNA4,
// 64-wide wavefronts).  One refinement step (Def. edge-labeled-fw-bisimulation)
// runs as:
//
//   signature   per vertex v: gather the pairs (edge label, previous block of
//               target) over v's CSR row, remove duplicates (the signature is a
//               SET, Def. signature), and fold the distinct pairs and v's own
//               previous block into a 64-bit key hash.  Degree tiers, fixed at
//               create time: runs of consecutive low-degree vertices share a
//               workgroup and an LDS hash set (range tier, at most 1024 or
//               2048 entries per run), a row of up to 4096 entries gets a
//               workgroup of its own, and hub rows are split into chunks that
//               are deduplicated in two passes (chunk, then partition), or,
//               beyond 4M entries, through a global hash set.
//   group       the minimum vertex per key hash becomes the candidate
//               representative of its vertices.  Few vertices insert (key
//               hash, v) into an open-addressing table and look theirs up;
//               many are partitioned by key hash into buckets that one
//               workgroup groups in LDS.
//   exact check every vertex whose representative is another vertex is
//               compared with it exactly: same previous block, same number of
//               distinct pairs, and every pair of v present in the
//               representative's set.  Hash collisions found here are
//               regrouped by a peeling round (min vertex per hash among the
//               collided vertices, exact check again) until none remain.
//   numbering   representatives are exactly the first vertex of each block;
//               an exclusive scan over "v is its own representative" in
//               vertex order gives dense ids numbered by first vertex, and
//               every other vertex copies its representative's id.
//
// The paper's own block ids are hash values and are only correct without
// collisions; here hashing only accelerates the grouping and every group is
// verified, so the ids are exact.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace kb {

typedef unsigned long long u64;
typedef uint32_t u32;

constexpr u64 EMPTY64 = ~0ULL;
constexpr int WAVE = 64;
constexpr int SMALL_MAX = 16;        // inline exact check limit (thread per vertex)
constexpr int RANGE_EDGES = 1024;    // CSR entries per multi-vertex range workgroup (or 2048)
constexpr int RANGE_VERTS = 256;     // vertices per range workgroup
constexpr int RANGE_DMAX = 4096;     // rows above RANGE_EDGES get a workgroup of 512 threads
constexpr int ROW_MAX = 8192;        // rows above RANGE_DMAX get one of 1024 threads; above this, hubs
constexpr int ROW_MAX_NARROW = 19456;  // with 32-bit keys rows up to this fit one workgroup's LDS (152 KB)
constexpr int BLOCK_MAX = ROW_MAX;
constexpr int BLOCK_SLOTS = 8192;    // LDS set slots for exact checks (64 KB)
constexpr int HUB_CHUNK_MAX = 4096;  // entries per hub staging workgroup: 2048 (default) or 4096
constexpr int HUB_PMAX = 1024;       // partitions per hub at most
constexpr int HUB_PART_TARGET = 2048;  // expected entries per hub partition
// LDS set slots per hub partition workgroup, and the largest staged hub (a
// larger one uses a global hash set): a partition then expects at most half
// as many distinct keys as its set has slots.  64-bit keys take half the
// slots (and half the staged hub size), so three workgroups fit a CU
// instead of two.
constexpr int HUB_PSLOTS = 8192;
constexpr int HUB_PSLOTS_WIDE = 4096;
constexpr int64_t HUB_STAGED_MAX = (int64_t)HUB_PMAX * HUB_PSLOTS / 2;
constexpr int64_t HUB_STAGED_MAX_WIDE = (int64_t)HUB_PMAX * HUB_PSLOTS_WIDE / 2;
constexpr int HUB_GCHUNK = 8192;     // entries per workgroup in the global-set path
constexpr int SCAN_ITEMS = 16;       // items per thread in the 64-bit offset scans (and the numbering, by default)
constexpr int SCAN_TILE = 256 * SCAN_ITEMS;
constexpr int SCAN_ITEMS_MIN = 8;    // smallest tunable items per thread of the numbering scan

// Device-resident epoch state (read by kernels at launch, advanced by
// k_advance), so a captured sequence of steps can be replayed.
constexpr int EP_TABLE = 0;    // grouping table epoch, 1..15
constexpr int EP_CTABLE = 1;   // peeling table epoch, 1..15
constexpr int EP_ZERO = 2;     // empty-signature epoch, increasing
constexpr int EP_HUB = 3;      // global hub set epoch, 1..3
constexpr int EP_CLR_TABLE = 4, EP_CLR_CTABLE = 5, EP_CLR_HUB = 6;
constexpr u32 ADV_TABLE = 1, ADV_CTABLE = 2, ADV_ZERO = 4, ADV_HUB = 8;

// Error bits reported through the workspace error word.
constexpr u32 ERR_LOOKUP_MISS = 1u;
constexpr u32 ERR_VERIFY_OVERFLOW = 4u;
constexpr u32 ERR_GRAPH_ROWPTR = 16u;
constexpr u32 ERR_GRAPH_COL = 32u;
constexpr u32 ERR_GRAPH_ELABEL = 64u;
constexpr u32 ERR_GRAPH_VPTR = 128u;
constexpr u32 ERR_GRAPH_VLABEL = 256u;
constexpr u32 ERR_BAD_PID = 512u;

// ---------------------------------------------------------------- hashing
// Murmur3's finalizers (Appleby, MurmurHash3, public domain) as the mixing
// functions.  The key hash of a vertex is
//   H = fmix64( sum_{k distinct} mix(k)  +  (own << 32 | dc) * odd )
// over the distinct set keys k of its pairs, with own = the vertex's previous
// block and dc = the number of distinct keys.  The sum makes the hash
// independent of the order in which a row's pairs are met, so no sort is
// needed to canonicalise.
__host__ __device__ inline u64 fmix64(u64 k) {
  k ^= k >> 33;
  k *= 0xff51afd7ed558ccdULL;
  k ^= k >> 33;
  k *= 0xc4ceb9fe1a85ec53ULL;
  k ^= k >> 33;
  return k;
}
__host__ __device__ inline u32 fmix32(u32 k) {
  k ^= k >> 16;
  k *= 0x85ebca6bu;
  k ^= k >> 13;
  k *= 0xc2b2ae35u;
  k ^= k >> 16;
  return k;
}
// What a distinct key adds to the sum.  64-bit keys are pairs and are mixed
// here; 32-bit keys are mixed already (fmix32), and one wide product of the
// key with a second form of itself spreads them over 64 bits without being
// linear in it.  Integer multiplies run at a quarter of the vector rate, and
// two 64-bit finalizers per entry (one of them on empty slots half the time)
// took a quarter of the range kernel.
__device__ inline u64 mix_pair(u64 p) { return fmix64(p ^ 0x9ae16a3b2f90404fULL); }
__device__ inline u64 mix_key32(u32 x) { return (u64)x * (u64)(x ^ 0x9E3779B9u) + ((u64)x << 32); }
// Slot position of 64-bit keys inside LDS hash sets: two 32-bit multiplies and
// a shift (the sets need spread, not collision resistance; equality is exact).
__device__ inline u32 set_hash(u64 p) {
  const u32 h = (u32)p * 0x9E3779B1u ^ ((u32)(p >> 32) + 0x7F4A7C15u) * 0x85EBCA77u;
  return h ^ (h >> 15);
}
__device__ inline u32 part_hash(u64 p) { return (u32)fmix64(p ^ 0x6a09e667f3bcc909ULL); }
__device__ inline u32 sub_hash(u64 p) { return (u32)(fmix64(p ^ 0xa0761d6478bd642fULL) >> 32); }
__device__ inline u64 finalize_key(u64 acc, u32 dc, u32 own) {
  return fmix64(acc + (((u64)own << 32) | (u64)dc) * 0x9E3779B97F4A7C15ULL);
}

// Where a key goes: into the grouping table, or (table NULL) to the partition
// (k_group_*): keys[i] for non-empty row i, EMPTY64 where another vertex of the
// range speaks for this one, and rep[v] = that vertex (or v itself).
struct KeySink {
  u64 *table;
  u64 tmask;
  int *rep;
  u64 *keys;
};

// ---------------------------------------------------------------- sources
// 32-bit set key of a pair (label l, reduced block b).  When every edge label
// and reduced block id fit together in 31 bits it is exact: fmix32 is one to
// one, and the one word it takes to 0xFFFFFFFF, the empty marker (0x331DA083),
// has the top bit clear, which is set here.  Otherwise (HK) it is a 32-bit hash
// of the pair, the label spread over the whole word by an odd multiplier: with
// the label merely rotated above the block, common labels met common blocks
// past 2^22 often enough that a graph of 2^28 vertices left more collided
// vertices than a step settles.  Deduplicating and summing hashed keys gives a
// function of the signature (equal pair sets give equal key sets), so equal signatures still get equal key hashes; the
// distinct count is then the number of distinct keys, and the exact check
// compares pair sets in both directions (a key collision inside a row could
// otherwise make a proper subset look equal).  kmask: the bits kept of hashed
// keys (all but for tests that make key collisions routine).
template <bool HK>
__device__ inline u32 narrow_key(u32 l, u32 b, u32 pb, u32 kmask) {
  if constexpr (HK) {
    const u32 k = fmix32(b ^ (l * 0x9E3779B1u)) & kmask;
    return k == 0xFFFFFFFFu ? 0xFFFFFFFEu : k;
  } else {
    return fmix32(0x80000000u | (l << pb) | b);
  }
}

// A source describes, for each vertex, a row of items and how an item maps
// to a 64-bit pair.  GraphSrc is one refinement step: item = CSR entry,
// pair = (edge label << 31) | previous block of the target.  LabelSrc builds
// P0: item = one vertex label, pair = the label.
// Gathers read the previous partition through a renumbered copy: gcol[e] =
// rank(col[e]) and gpid[rank(w)] = pid[w], where ranks order vertices by
// decreasing in-degree.  The targets most edges point to then share cache
// lines, which roughly halves the cost of the per-entry random gather.
// SEP: edge labels come from their own array (elabel); otherwise they sit
// above the rank in gcol (or there are none), and elabel is unused.
// HK: 32-bit set keys are a hash of the pair (used when the label and the
// reduced block do not fit 31 bits together); see key32_of.
template <bool SEP, bool HK = false>
struct GraphSrcT {
  static constexpr bool GRAPH = true;
  static constexpr bool HASHED = HK;
  const int64_t *row_ptr;
  const int32_t *gcol;    // targets renumbered by in-degree rank (and, packed, their labels)
  const int32_t *elabel;  // the labels when SEP
  const int32_t *gpid;    // previous partition in rank order
  const int32_t *pid;     // previous partition in vertex order
  __device__ inline int64_t begin(int v) const { return row_ptr[v]; }
  __device__ inline int64_t end(int v) const { return row_ptr[v + 1]; }
  // A pair keeps the target's block id modulo 2^pb.  The targets of one row
  // lie in one graph, whose block ids form an interval of at most 2^pb ids
  // (pb covers the largest graph; a single graph: all ids), so the reduction
  // is one-to-one within a row, and every kernel reduces the same way.
  u32 pb;
  // gcol[e] = (label << rbits) | rank when labels are packed (rbits < 31);
  // otherwise rbits = 31 and the label comes from elabel (SEP) or is 0.
  // Packing halves the streamed bytes per entry.
  u32 rbits;
  // bits kept of hashed keys (all but for tests that make key collisions routine)
  u32 kmask = 0xFFFFFFFFu;
  __device__ inline u32 pmask() const { return pb >= 31 ? 0x7FFFFFFFu : (1u << pb) - 1u; }
  // (label, rank of the target) of entry e; streamed arrays are read
  // non-temporally so they do not evict the gather targets from the L2
  __device__ inline void entry(int64_t e, u32 &l, u32 &r) const {
    const u32 g = (u32)__builtin_nontemporal_load(&gcol[e]);
    if constexpr (SEP) l = (u32)__builtin_nontemporal_load(&elabel[e]);
    else l = g >> rbits;
    r = g & ((1u << rbits) - 1u);
  }
  // entry() for first + min(t + u*STRIDE, count - 1), u < U: all the
  // streamed words are requested together, with no branch among them
  template <int U, int STRIDE>
  __device__ inline void entries(int64_t first, int t, int count, u32 (&l)[U], u32 (&r)[U]) const {
    const u32 rm = (1u << rbits) - 1u;
    if constexpr (SEP) {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int64_t e = first + min(t + u * STRIDE, count - 1);
        r[u] = (u32)__builtin_nontemporal_load(&gcol[e]);
        l[u] = (u32)__builtin_nontemporal_load(&elabel[e]);
      }
#pragma unroll
      for (int u = 0; u < U; ++u) r[u] &= rm;
    } else {
#pragma unroll
      for (int u = 0; u < U; ++u) r[u] = (u32)__builtin_nontemporal_load(&gcol[first + min(t + u * STRIDE, count - 1)]);
#pragma unroll
      for (int u = 0; u < U; ++u) {
        l[u] = r[u] >> rbits;
        r[u] &= rm;
      }
    }
  }
  // the pair of an entry whose (label, rank) entry() has read: one gather
  __device__ inline u64 pair_of(u32 l, u32 r) const { return ((u64)l << 31) | (u64)((u32)gpid[r] & pmask()); }
  __device__ inline u64 pair(int64_t e) const {
    u32 l, r;
    entry(e, l, r);
    return pair_of(l, r);
  }
  __device__ inline u32 own(int v) const { return (u32)pid[v]; }
  // Narrow form of a pair, used inside LDS sets (narrow_key).
  __device__ inline u32 key32_of(u32 l, u32 r) const {
    return narrow_key<HK>(l, (u32)gpid[r] & pmask(), pb, kmask);
  }
  __device__ inline u32 key32(int64_t e) const {
    u32 l, r;
    entry(e, l, r);
    return key32_of(l, r);
  }
};

struct LabelSrc {
  static constexpr bool GRAPH = false;
  static constexpr bool HASHED = false;
  const int64_t *ptr;  // may be null: one label per vertex
  const int32_t *lab;
  const int32_t *gid;  // may be null; in a batch, the graph of each vertex (P0 never joins graphs)
  __device__ inline int64_t begin(int v) const { return ptr ? ptr[v] : (int64_t)v; }
  __device__ inline int64_t end(int v) const { return ptr ? ptr[v + 1] : (int64_t)v + 1; }
  __device__ inline u64 pair(int64_t e) const { return (u64)(u32)lab[e]; }
  __device__ inline void entry(int64_t e, u32 &l, u32 &r) const {
    l = (u32)lab[e];
    r = 0;
  }
  template <int U, int STRIDE>
  __device__ inline void entries(int64_t first, int t, int count, u32 (&l)[U], u32 (&r)[U]) const {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      l[u] = (u32)lab[first + min(t + u * STRIDE, count - 1)];
      r[u] = 0;
    }
  }
  __device__ inline u64 pair_of(u32 l, u32) const { return (u64)l; }
  __device__ inline u32 own(int v) const { return gid ? (u32)gid[v] : 0u; }
};

// LDS set keys: the 64-bit pair itself, or the narrow 32-bit form.
template <class K>
struct Keys;
template <>
struct Keys<u64> {
  static constexpr u64 EMPTY = EMPTY64;
  template <class Src>
  __device__ static inline u64 load(const Src &s, int64_t e) { return s.pair(e); }
  template <class Src>
  __device__ static inline u64 from(const Src &s, u32 l, u32 r) { return s.pair_of(l, r); }
  __device__ static inline u64 mix(u64 p) { return mix_pair(p); }
  __device__ static inline u32 hash(u64 p) { return set_hash(p); }
};
template <>
struct Keys<u32> {
  static constexpr u32 EMPTY = 0xFFFFFFFFu;
  template <class Src>
  __device__ static inline u32 load(const Src &s, int64_t e) { return s.key32(e); }
  template <class Src>
  __device__ static inline u32 from(const Src &s, u32 l, u32 r) { return s.key32_of(l, r); }
  __device__ static inline u64 mix(u32 x) { return mix_key32(x); }
  __device__ static inline u32 hash(u32 x) { return x; }
};

// Load the keys of entries first + j*STRIDE (j = 0..U-1, only those below
// count are valid; the others become EMPTY).  All streamed words are
// requested before any gather, and no load sits under a branch, so a wave
// waits twice in all instead of twice per entry.  Invalid slots re-read the
// last valid entry (count >= 1 is required).
template <class K, int U, int STRIDE, class Src>
__device__ inline void load_keys(const Src &src, int64_t first, int t, int count, K (&out)[U]) {
  typedef Keys<K> KO;
  u32 l[U], r[U];
  src.template entries<U, STRIDE>(first, t, count, l, r);
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const K p = KO::from(src, l[u], r[u]);
    out[u] = t + u * STRIDE < count ? p : KO::EMPTY;
  }
}

// ---------------------------------------------------------------- LDS set overflow
// The overflow mark of an LDS set, set by the insertion that reaches the set's
// limit and read by all threads between their insertions.  Atomic accesses: a
// plain read is the compiler's to keep in a register over a whole loop without
// barriers, where the marks of other threads then go unseen, the set fills up
// and its probes never end.
__device__ inline bool set_full(const u32 *mark) {
  return __hip_atomic_load(mark, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) != 0u;
}
__device__ inline void mark_full(u32 *mark) {
  __hip_atomic_store(mark, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// ---------------------------------------------------------------- wave helpers
// Largest r in [lo, hi) with at(r) <= x, for a non-decreasing at() with
// at(lo) <= x; the whole wave searches, 64 probes at a time.
template <class At>
__device__ inline int64_t wave_last_le(int64_t lo, int64_t hi, int64_t x, At at) {
  const int lane = threadIdx.x & (WAVE - 1);
  while (hi - lo > 1) {
    const int64_t step = (hi - lo + WAVE - 1) / WAVE;
    const int64_t r = lo + lane * step;
    const int ok = __popcll(__ballot(r < hi && at(r) <= x));  // a prefix of the lanes, lane 0 among them
    lo += (ok - 1) * step;
    hi = min(hi, lo + step);
  }
  return lo;
}

__device__ inline u64 sink_form(u64 h) { return h == EMPTY64 ? EMPTY64 - 1ULL : h; }
__device__ inline void sink_key(const KeySink &s, int row, int v, u64 h) {
  s.rep[v] = v;
  s.keys[row] = sink_form(h);
}

__device__ inline u64 wave_sum_u64(u64 x) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o, WAVE);
  return x;
}
__device__ inline u32 wave_sum_u32(u32 x) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o, WAVE);
  return x;
}

// Append `item` to list[*counter] for every lane with pred set, one atomic
// per wave.  Works with any subset of active lanes.
__device__ inline void wave_append(int *counter, int *list, bool pred, int item) {
  u64 mask = __ballot(pred);
  if (mask == 0) return;
  int leader = __ffsll((long long)mask) - 1;
  int lane = threadIdx.x & (WAVE - 1);
  int base = 0;
  if (lane == leader) base = atomicAdd(counter, __popcll(mask));
  base = __shfl(base, leader, WAVE);
  if (pred) {
    u64 below = mask & ((1ULL << lane) - 1ULL);
    list[base + __popcll(below)] = item;
  }
}

// Append v0 + j for every bit j of each lane's mask to list[*counter], one
// atomic per wave.  Must be called by the whole wave.
__device__ inline void wave_append_mask(int *counter, int *list, u32 mask, int64_t v0) {
  const int lane = threadIdx.x & (WAVE - 1);
  const u32 c = (u32)__popc(mask);
  u32 x = c;
#pragma unroll
  for (int o = 1; o < WAVE; o <<= 1) {
    const u32 y = __shfl_up(x, o, WAVE);
    if (lane >= o) x += y;
  }
  const u32 total = __shfl(x, WAVE - 1, WAVE);
  if (total == 0) return;
  int base = 0;
  if (lane == WAVE - 1) base = atomicAdd(counter, (int)total);
  base = __shfl(base, WAVE - 1, WAVE);
  int at = base + (int)(x - c);
  while (mask) {
    const int j = __ffs(mask) - 1;
    list[at++] = (int)(v0 + j);
    mask &= mask - 1u;
  }
}

// ---------------------------------------------------------------- grouping table
// Open addressing with linear probing.  Slot = (tag << 32) | vertex, tag =
// 28 hash bits above bit 36 plus a 4-bit epoch (1..15).  A slot whose epoch is
// not the current one is free, so the table is reused across iterations
// without clearing (it is cleared once every 15 epochs).  Home slot = low
// hash bits.  Every vertex with the same (tag, home) ends in the same slot,
// which holds the minimum such vertex.  Two different keys can share a slot;
// the exact check separates them.
__device__ inline u32 slot_tag(u64 h, u32 epoch) { return ((u32)(h >> 36) << 4) | epoch; }

__device__ inline void table_insert(u64 *table, u64 tmask, u64 h, u32 v, u32 epoch) {
  const u32 tag = slot_tag(h, epoch);
  const u64 want = ((u64)tag << 32) | (u64)v;
  u64 s = h & tmask;
  while (true) {
    // A plain load may return an older value of the slot (empty, or a larger
    // minimum); every decision taken on it is re-validated by the atomics, so
    // hot keys are served from the L1 instead of serialising on one L2 line.
    u64 cur = table[s];
    while ((((u32)(cur >> 32)) & 15u) != epoch) {
      u64 old = atomicCAS(&table[s], cur, want);
      if (old == cur) return;
      cur = old;
    }
    if ((u32)(cur >> 32) == tag) {
      if ((u32)cur > v) atomicMin(&table[s], want);
      return;
    }
    s = (s + 1) & tmask;
  }
}

__device__ inline int table_lookup(const u64 *table, u64 tmask, u64 h, u32 epoch) {
  const u32 tag = slot_tag(h, epoch);
  u64 s = h & tmask;
  while (true) {
    u64 cur = table[s];
    u32 t = (u32)(cur >> 32);
    if (t == tag) return (int)(u32)cur;
    if ((t & 15u) != epoch) return -1;
    s = (s + 1) & tmask;
  }
}

// Vertices with an empty signature (no out-edges, or no labels in P0) are
// grouped exactly by their previous block alone: zrep[block] keeps
// (~epoch << 32 | min vertex), so entries of older epochs compare larger and
// are replaced, and no clearing is needed.  No hash and no check involved.
__device__ inline void zero_insert(u64 *zrep, u32 own, u32 v, u32 zep) {
  const u64 want = ((u64)(~zep) << 32) | (u64)v;
  // A plain load may be stale for the whole kernel (another XCD's atomics do
  // not reach this L2), and every wave would then queue at the few slots; the
  // device-scope load sees the current minimum, and atomicMin decides.
  if (zrep[own] > want && __hip_atomic_load(&zrep[own], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) > want)
    atomicMin(&zrep[own], want);
}

__device__ inline void key_insert(u64 *table, u64 tmask, u64 *zrep, u64 h, u32 dc, u32 own, u32 v, u32 epoch,
                                  u32 zep) {
  if (dc == 0) zero_insert(zrep, own, v, zep);
  else table_insert(table, tmask, h, v, epoch);
}

// Of the lanes with act set, all but one per key drop out before the table:
// where many vertices share a key (label classes, the first steps of
// unlabelled graphs) the lanes of a wave would otherwise queue at one table
// slot with device-wide atomics, which serialise beyond the L2.  Lanes meet
// in FIRST_SLOTS LDS words of their wave by hash bits; the lowest lane in a
// word speaks for every lane there with its key, and a lane whose word went
// to another key acts for itself, so there is no probing.  Lanes hold
// ascending vertices, so the lowest lane has the smallest vertex of its key.
// Measured: k_sig_range on an unlabelled graph of 1M vertices and 1.2M
// entries 169 -> 64 us; a graph with a key per vertex runs as before.
// Must be reached by the whole wave; slots is this wave's own region.
constexpr int FIRST_SLOTS = 256;
__device__ inline bool wave_first_of_key(u32 *slots, bool act, u64 h) {
  const int lane = threadIdx.x & (WAVE - 1);
#pragma unroll
  for (int i = 0; i < FIRST_SLOTS / WAVE; ++i) slots[lane + i * WAVE] = 0xFFFFFFFFu;
  __builtin_amdgcn_wave_barrier();
  const u32 at = (u32)(h >> 20) & (FIRST_SLOTS - 1);
  if (act) atomicMin(&slots[at], (u32)lane);
  __builtin_amdgcn_wave_barrier();
  const int m = act ? (int)slots[at] : lane;
  const u64 hm = __shfl(h, m, WAVE);
  return act && (m == lane || hm != h);
}

// The same for lanes whose vertices are in no order: the lane that goes on
// gets the smallest vertex of its key in v.  slots: 2 * FIRST_SLOTS words.
__device__ inline bool wave_min_of_key(u32 *slots, bool act, u64 h, u32 &v) {
  const int lane = threadIdx.x & (WAVE - 1);
  u32 *mins = slots + FIRST_SLOTS;
#pragma unroll
  for (int i = 0; i < FIRST_SLOTS / WAVE; ++i) mins[lane + i * WAVE] = 0xFFFFFFFFu;
  const u32 at = (u32)(h >> 20) & (FIRST_SLOTS - 1);
#pragma unroll
  for (int i = 0; i < FIRST_SLOTS / WAVE; ++i) slots[lane + i * WAVE] = 0xFFFFFFFFu;
  __builtin_amdgcn_wave_barrier();
  if (act) atomicMin(&slots[at], (u32)lane);
  __builtin_amdgcn_wave_barrier();
  const int m = act ? (int)slots[at] : lane;
  const u64 hm = __shfl(h, m, WAVE);
  const bool same = act && hm == h;
  if (same) atomicMin(&mins[at], v);
  __builtin_amdgcn_wave_barrier();
  if (same && m == lane) v = mins[at];
  return act && (m == lane || !same);
}

// zero_insert for the lanes with pred set, one per block met in the wave
// (empty signatures share few blocks).  A fixed number of LDS accesses, where
// a round of shuffles per distinct block cost up to a block count times that:
// the list inserts of an update on a 100M-edge graph 185 -> 92 us, a k = 10
// call on the 1B-edge graph 152.8 -> 148.3 ms (its first step).  Must be
// reached by the whole wave; slots: 2 * FIRST_SLOTS words of this wave.
__device__ inline void zero_insert_wave(u32 *slots, u64 *zrep, bool pred, u32 own, u32 v, u32 zep) {
  if (!__ballot(pred)) return;
  const u64 key = (u64)own * 0x9E3779B97F4A7C15ull;  // odd: one to one
  if (wave_min_of_key(slots, pred, key, v)) zero_insert(zrep, own, v, zep);
}

// ---------------------------------------------------------------- validation
__global__ void k_validate_rows(int64_t n, int64_t m, const int64_t *__restrict__ ptr, u32 *err, u32 bit) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i > n) return;
  int64_t a = ptr[i];
  bool bad = false;
  if (i == 0 && a != 0) bad = true;
  if (i == n && a != m) bad = true;
  if (i < n && ptr[i + 1] < a) bad = true;
  if (a < 0 || a > m) bad = true;
  if (bad) atomicOr(err, bit);
}

// Range check of cnt values: any value < 0, or >= upper when upper >= 0, sets
// `bit` in *err.  Grid-stride over the 16-byte-aligned body of the array (the
// few values before and after it one by one), 4 groups of 4 values in flight
// per thread, one atomic per wave that found a bad value.  MAX: the largest
// value too (as unsigned, into *max_out, which starts at 0) from the same
// read: one candidate per workgroup, and a workgroup whose candidate is not
// above the current maximum issues no atomic (one per wave, on one address,
// took 0.2 ms whatever the array's length).
constexpr int VALIDATE_GRID = 4096;
typedef u32 u32x4 __attribute__((ext_vector_type(4)));
template <bool MAX>
__global__ void __launch_bounds__(256) k_validate_vals(int64_t cnt, const int32_t *__restrict__ vals, int64_t upper,
                                                       u32 *err, u32 bit, u32 *max_out) {
  // negative values become >= 2^31 as unsigned: one compare covers both ends
  const u32 lim = (upper >= 0 && upper < 0x80000000ll) ? (u32)upper : 0x80000000u;
  const uintptr_t a = reinterpret_cast<uintptr_t>(vals);
  const int64_t head = (a & 3) ? cnt : std::min<int64_t>(cnt, (int64_t)(((16 - (a & 15)) & 15) >> 2));
  const int64_t ng = (cnt - head) >> 2;
  const u32x4 *__restrict__ g4 = reinterpret_cast<const u32x4 *>(vals + head);
  const int64_t stride = (int64_t)gridDim.x * 256;
  const int64_t gt = (int64_t)blockIdx.x * 256 + threadIdx.x;
  bool bad = false;
  u32 mx = 0;
  int64_t i = gt;
  for (; i + 3 * stride < ng; i += 4 * stride) {
    u32x4 q[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) q[j] = __builtin_nontemporal_load(&g4[i + j * stride]);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      bad |= (q[j].x >= lim) | (q[j].y >= lim) | (q[j].z >= lim) | (q[j].w >= lim);
      if constexpr (MAX) mx = max(max(max(mx, q[j].x), max(q[j].y, q[j].z)), q[j].w);
    }
  }
  for (; i < ng; i += stride) {
    const u32x4 q = __builtin_nontemporal_load(&g4[i]);
    bad |= (q.x >= lim) | (q.y >= lim) | (q.z >= lim) | (q.w >= lim);
    if constexpr (MAX) mx = max(max(max(mx, q.x), max(q.y, q.z)), q.w);
  }
  auto one = [&](int64_t t) {
    const u32 x = (u32)vals[t];
    bad |= x >= lim;
    if constexpr (MAX) mx = max(mx, x);
  };
  for (int64_t t = gt; t < head; t += stride) one(t);
  for (int64_t t = head + (ng << 2) + gt; t < cnt; t += stride) one(t);
  if (__ballot(bad) && (threadIdx.x & (WAVE - 1)) == 0) atomicOr(err, bit);
  if constexpr (MAX) {
    __shared__ u32 sh_m[4];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) mx = max(mx, (u32)__shfl_xor(mx, o, WAVE));
    if ((threadIdx.x & (WAVE - 1)) == 0) sh_m[threadIdx.x >> 6] = mx;
    __syncthreads();
    if (threadIdx.x == 0) {
      mx = max(max(sh_m[0], sh_m[1]), max(sh_m[2], sh_m[3]));
      if (mx > __hip_atomic_load(max_out, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicMax(max_out, mx);
    }
  }
}

// ---------------------------------------------------------------- signature tiers
// A run of consecutive non-empty rows [v0, v1) (indices into the list of
// non-empty rows; vertices in a single-row range of the row tiers) handled by
// one workgroup, with the run's first entry e0 and its entry count ne, so that
// a workgroup requests its entries without waiting for the row offsets.
struct Range {
  int v0, v1;
  int ne;
  int row;  // single-row ranges: the row's index among the non-empty rows
  int64_t e0;
};

// a scaled to [0, n)
__device__ inline u64 scale_to(u32 a, u64 n) { return __umul64hi(((u64)a) << 32, n); }
__device__ inline u32 scale_to(u32 a, u32 n) { return __umulhi(a, n); }

// Exclusive block scan (256 threads) of one u32 per thread; returns the
// thread's prefix and writes the block total to *total.
__device__ inline u32 block_exclusive_scan(u32 mine, u32 *sh_w, u32 *total) {
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  u32 x = mine;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const u32 y = __shfl_up(x, o, WAVE);
    if (lane >= o) x += y;
  }
  if (lane == 63) sh_w[w] = x;
  __syncthreads();
  u32 base = 0;
  for (int i = 0; i < w; ++i) base += sh_w[i];
  *total = sh_w[0] + sh_w[1] + sh_w[2] + sh_w[3];
  __syncthreads();
  return base + x - mine;
}

// Sum over the workgroup; the result is valid in thread 0.  sh_acc and
// sh_cnt hold one slot per wave.
__device__ inline void block_reduce_2(u64 &acc, u32 &cnt, u64 *sh_acc, u32 *sh_cnt) {
  acc = wave_sum_u64(acc);
  cnt = wave_sum_u32(cnt);
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  if (lane == 0) { sh_acc[w] = acc; sh_cnt[w] = cnt; }
  __syncthreads();
  if (threadIdx.x == 0) {
    const int nw = blockDim.x >> 6;
    for (int i = 1; i < nw; ++i) { acc += sh_acc[i]; cnt += sh_cnt[i]; }
  }
}

// Range tier: a workgroup takes a run of consecutive non-empty rows holding at
// most EMAX entries (the range capacity, 1024 or 2048), RANGE_VERTS rows;
// longer rows go to the row tier.  All entries are gathered at once (EMAX/256
// per thread, loads issued before dependent work, consecutive entries on
// consecutive lanes), then inserted into their vertex's region of an LDS hash
// set (2*deg slots at offset 2*row offset); sums are formed from the set.
// SKIP (work-efficient mode): rows of vertices flagged in skip[] (singleton
// blocks, which cannot split) are left out; the remaining rows are packed,
// so their entries are gathered only after the owner scan.
// NT: 256 threads keep the most ranges in flight where ranges are many; where
// they are few (FEW_RANGES) the chip has room, and 1024 threads walk a range's
// chain of loads, LDS passes and barriers with 2 entries a thread instead of 8.
template <class Src, int EMAX, class K = u64, bool SKIP = false, int NT = 256>
__global__ void __launch_bounds__(NT) k_sig_range(Src src, const Range *__restrict__ ranges, u64 *__restrict__ H,
                                                   u32 *__restrict__ DC, KeySink sink,
                                                   const u32 *__restrict__ dep, u64 hmask,
                                                   const int *__restrict__ nzv, const u32 *__restrict__ nzrow,
                                                   const unsigned char *__restrict__ skip) {
  typedef Keys<K> KO;
  static_assert(NT >= RANGE_VERTS && (!SKIP || NT == 256), "a thread per vertex; the packing scan has four waves");
  constexpr int U = EMAX / NT;
  const u32 epoch = dep[EP_TABLE];
  __shared__ K set[2 * EMAX];
  __shared__ u64 acc[RANGE_VERTS];
  __shared__ u32 cnt[RANGE_VERTS];
  __shared__ int roff[RANGE_VERTS + 1];  // CSR row offsets, relative to the range
  __shared__ int coff[SKIP ? RANGE_VERTS + 1 : 1];  // packed offsets (skipped rows empty)
  __shared__ unsigned char owner[EMAX];
  __shared__ u32 wmax[NT / WAVE];
  __shared__ u64 sh_acc[NT / WAVE];
  __shared__ u32 sh_cnt[NT / WAVE];
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  const Range rg = ranges[blockIdx.x];
  const int V = rg.v1 - rg.v0;
  const bool single = V == 1;
  const int64_t eb = rg.e0;
  // The addresses of the row offsets, this thread's vertex (V <= blockDim)
  // and the streamed words need only the range, so all three are requested
  // together; the gathers follow (the vertex's previous block among them), and
  // the offsets reach LDS last.
  const u32 b0 = t < V ? nzrow[rg.v0 + t] : 0u;
  const int v = t < V ? nzv[rg.v0 + t] : 0;
  u32 el[U], er[U];
  if constexpr (!SKIP) src.template entries<U, NT>(eb, t, rg.ne, el, er);
  K pr[U];
  if constexpr (!SKIP) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const K p = KO::from(src, el[u], er[u]);
      pr[u] = t + u * NT < rg.ne ? p : KO::EMPTY;
    }
  }
  const u32 own_t = t < V ? src.own(v) : 0u;
  if (t < V) roff[t] = (int)(b0 - (u32)eb);
  if (t == 0) roff[V] = rg.ne;
  for (int i = t; i < V; i += NT) {
    acc[i] = 0;
    cnt[i] = 0;
  }
  if (!single)
    for (int i = t; i < EMAX; i += NT) owner[i] = 0;
  __syncthreads();
  const int *off = roff;  // offsets that place entries and set regions
  bool skipped = false;   // this thread's vertex (t < V) is left out
  if constexpr (SKIP) {
    skipped = t < V && skip[v];
    const u32 d = (t < V && !skipped) ? (u32)(roff[t + 1] - roff[t]) : 0u;
    u32 total;
    const u32 ex = block_exclusive_scan(d, wmax, &total);
    if (t < V) coff[t] = (int)ex;
    if (t == 0) coff[V] = (int)total;
    __syncthreads();
    off = coff;
  }
  const int E = off[V];
  for (int i = t; i < 2 * E; i += NT) set[i] = KO::EMPTY;
  // the row start of every non-empty vertex marks its index; a max-scan then
  // gives the owner of every entry
  if (!single)
    for (int i = t; i < V; i += NT)
      if (off[i + 1] > off[i]) owner[off[i]] = (unsigned char)i;
  __syncthreads();
  if (!single) {
    constexpr int PER = EMAX / NT;
    u32 run = 0;
    const int j0 = t * PER;
#pragma unroll
    for (int k = 0; k < PER; ++k) run = max(run, (u32)owner[j0 + k]);
    u32 x = run;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const u32 y = __shfl_up(x, o, WAVE);
      if (lane >= o) x = max(x, y);
    }
    if (lane == 63) wmax[w] = x;
    __syncthreads();
    u32 carry = __shfl_up(x, 1, WAVE);
    if (lane == 0) carry = 0;
    for (int i = 0; i < w; ++i) carry = max(carry, wmax[i]);
#pragma unroll
    for (int k = 0; k < PER; ++k) {
      carry = max(carry, (u32)owner[j0 + k]);
      owner[j0 + k] = (unsigned char)carry;
    }
    __syncthreads();
  }
  if constexpr (SKIP) {
    // packed entry j of row lo sits at CSR offset roff[lo] + (j - coff[lo])
    u32 l[U], r[U];
    if (E > 0) {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int j = min(t + u * NT, E - 1);
        const int lo = single ? 0 : owner[j];
        src.entry(eb + roff[lo] + (j - coff[lo]), l[u], r[u]);
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      K p = KO::EMPTY;
      if (E > 0) p = KO::from(src, l[u], r[u]);
      pr[u] = t + u * NT < E ? p : KO::EMPTY;
    }
  }
  if (single) {
    // one row: thread-local sums, one block reduction
    u64 a = 0;
    u32 c = 0;
    const u32 sz = 2u * (u32)E;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const K p = pr[u];
      if (p == KO::EMPTY) continue;
      u32 sl = scale_to(KO::hash(p), sz);
      while (true) {
        const K old = atomicCAS(&set[sl], KO::EMPTY, p);
        if (old == KO::EMPTY) { a += KO::mix(p); ++c; break; }
        if (old == p) break;
        sl = (sl + 1 == sz) ? 0u : sl + 1;
      }
    }
    block_reduce_2(a, c, sh_acc, sh_cnt);
    if (t == 0 && !skipped) {
      const u64 h = finalize_key(a, c, own_t) & hmask;
      H[v] = h;
      DC[v] = c;
      if (sink.table) table_insert(sink.table, sink.tmask, h, (u32)v, epoch);
      else sink_key(sink, rg.v0, v, h);
    }
    return;
  }
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int j = t + u * NT;
    if (j < E) {
      const int lo = owner[j];
      const K p = pr[u];
      const int base = 2 * off[lo];
      const u32 sz = 2u * (u32)(off[lo + 1] - off[lo]);
      u32 sl = scale_to(KO::hash(p), sz);
      while (true) {
        const K old = atomicCAS(&set[base + sl], KO::EMPTY, p);
        if (old == KO::EMPTY || old == p) break;
        sl = (sl + 1 == sz) ? 0u : sl + 1;
      }
    }
  }
  __syncthreads();
  // Sums from the set: thread t reads the 2U consecutive slots from 2Ut on;
  // slot s lies in the region of vertex owner[s / 2].  Runs of one vertex are
  // summed in registers and added to the vertex once per run, so the shared
  // accumulators see a few atomics per vertex instead of one per pair.  Each
  // lane starts at a different slot of its 2U (rotation by lane / (64 / 2U)),
  // so the lanes of one read fall in different LDS banks instead of the few
  // that a stride of 2U words allows; the order of a sum does not matter,
  // and the rotation breaks at most one run.
  {
    constexpr int SL = 2 * U, GRP = WAVE / SL > 0 ? WAVE / SL : 1;
    const int rot = (lane / GRP) & (SL - 1);
    u64 a = 0;
    u32 c = 0;
    int cur = -1;
#pragma unroll
    for (int q = 0; q < SL; ++q) {
      const int sidx = SL * t + ((q + rot) & (SL - 1));
      if (sidx < 2 * E) {
        const int lo = owner[sidx >> 1];
        if (lo != cur) {
          if (c) {
            atomicAdd(&acc[cur], a);
            atomicAdd(&cnt[cur], c);
          }
          cur = lo;
          a = 0;
          c = 0;
        }
        const K p = set[sidx];
        if (p != KO::EMPTY) {
          a += KO::mix(p);
          ++c;
        }
      }
    }
    if (c) {
      atomicAdd(&acc[cur], a);
      atomicAdd(&cnt[cur], c);
    }
  }
  __syncthreads();
  // V <= RANGE_VERTS <= NT: one vertex per thread.
  const bool keyed = t < V && !skipped;
  u64 h = 0;
  if (keyed) {
    const u32 c = cnt[t];
    h = finalize_key(acc[t], c, own_t) & hmask;
    H[v] = h;
    DC[v] = c;
  }
  // One key of the workgroup goes on, as in wave_first_of_key: two barriers more
  // than per wave, but a quarter of the pairs or device-wide atomics of keys that
  // many vertices share (unlabelled graphs, ten steps: table, 1M vertices 1.09 ->
  // 1.00 ms; partition, 4.8M entries 3.32 -> 3.27, 72M 49.0 -> 47.9).  The set is no
  // longer read: its space holds the slots.
  constexpr int NS = 4 * FIRST_SLOTS;
  static_assert(sizeof(set) >= NS * sizeof(u32), "key slots of the workgroup");
  u32 *slots = reinterpret_cast<u32 *>(set);
  if (keyed) {
    acc[t] = h;
    cnt[t] = (u32)v;
  }
#pragma unroll
  for (int i = 0; i < NS / NT; ++i) slots[t + i * NT] = 0xFFFFFFFFu;
  __syncthreads();
  const u32 at = (u32)(h >> 20) & (NS - 1);
  if (keyed) atomicMin(&slots[at], (u32)t);
  __syncthreads();
  if (!keyed) return;
  u32 m = slots[at];
  if (acc[m] != h) m = (u32)t;
  if (!sink.table) {
    sink.rep[v] = (int)cnt[m];
    sink.keys[rg.v0 + t] = m == (u32)t ? sink_form(h) : EMPTY64;
  } else if (m == (u32)t) {
    table_insert(sink.table, sink.tmask, h, (u32)v, epoch);
  }
}

// Vertices with an empty signature, which are in no range: no distinct pair,
// and grouped by their previous block alone.  Launched where representatives
// of empty signatures are formed: the first step of a call (their classes
// never change within a call), P0, and updates (skip: all but the flagged).
// A workgroup inserts each block of its EMPTY_VERTS vertices once (they meet in
// LDS as in wave_first_of_key): where blocks are few, waves queue at their slots in
// zrep, each for as long as chance has it (one insert per wave of 64, the same code
// in two libraries: RMAT graph of 23M entries 41 / 85 us, 40M 52 / 145; now 38 and,
// 72M entries of one block, 241 -> 209).  Graphs of many blocks pay for the LDS:
// 94M vertices without entries 0.89 -> 0.97 ms of a call of 129.
constexpr int EMPTY_THREADS = 1024, EMPTY_ITEMS = 4, EMPTY_VERTS = EMPTY_THREADS * EMPTY_ITEMS;
template <class Src>
__global__ void __launch_bounds__(EMPTY_THREADS) k_sig_empty(Src src, int n, u32 *__restrict__ DC, u64 *zrep,
                                                             const u32 *__restrict__ dep,
                                                             const unsigned char *__restrict__ skip) {
  constexpr int NS = 2 * EMPTY_VERTS;
  __shared__ u32 block[EMPTY_VERTS];
  __shared__ u32 slots[NS];
  const u32 zep = dep[EP_ZERO];
  const int64_t v0 = (int64_t)blockIdx.x * EMPTY_VERTS;
#pragma unroll
  for (int j = 0; j < NS / EMPTY_THREADS; ++j) slots[threadIdx.x + j * EMPTY_THREADS] = 0xFFFFFFFFu;
  bool zero[EMPTY_ITEMS];
#pragma unroll
  for (int j = 0; j < EMPTY_ITEMS; ++j) {
    const int64_t v = v0 + threadIdx.x + j * EMPTY_THREADS;
    zero[j] = v < n && src.begin((int)v) == src.end((int)v) && !(skip && skip[v]);
  }
  u32 own[EMPTY_ITEMS];
#pragma unroll
  for (int j = 0; j < EMPTY_ITEMS; ++j) {
    const int i = threadIdx.x + j * EMPTY_THREADS;
    own[j] = zero[j] ? src.own((int)(v0 + i)) : 0u;
    if (zero[j]) DC[v0 + i] = 0;
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < EMPTY_ITEMS; ++j) {
    const int i = threadIdx.x + j * EMPTY_THREADS;
    if (!zero[j]) continue;
    block[i] = own[j];
    atomicMin(&slots[own[j] * 0x9E3779B1u >> 19], (u32)i);  // 13 bits: NS
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < EMPTY_ITEMS; ++j) {
    const int i = threadIdx.x + j * EMPTY_THREADS;
    if (!zero[j]) continue;
    const u32 m = slots[own[j] * 0x9E3779B1u >> 19];
    if (m == (u32)i || block[m] != own[j]) zero_insert(zrep, own[j], (u32)(v0 + i), zep);
  }
}

// Representatives of the vertices with an empty signature (DC = 0) in a call's
// first step: the minimum vertex of their previous block.
template <class Src>
__global__ void __launch_bounds__(256) k_rep_empty(Src src, int n, const u32 *__restrict__ DC,
                                                   const u64 *__restrict__ zrep, const u32 *__restrict__ dep,
                                                   int *__restrict__ rep, u32 *err,
                                                   const unsigned char *__restrict__ skip) {
  const u32 zep = dep[EP_ZERO];
  const int v = blockIdx.x * 256 + threadIdx.x;
  if (v >= n || DC[v] != 0 || (skip && skip[v])) return;
  const u64 z = zrep[src.own(v)];
  if ((u32)(z >> 32) != ~zep) {
    atomicOr(err, ERR_LOOKUP_MISS);
    rep[v] = v;
  } else {
    rep[v] = (int)(u32)z;
  }
}

// Rows of exactly one item (P0 with one label per vertex): no set, no row
// offsets.  A workgroup inserts each key of its ONE_VERTS vertices once (they
// meet in LDS as in wave_first_of_key): labels are few, and their slots were
// where all waves queued (2M vertices, 32 labels: 180 -> 24 us).
constexpr int ONE_THREADS = 1024, ONE_ITEMS = 4, ONE_VERTS = ONE_THREADS * ONE_ITEMS;
template <class Src>
__global__ void __launch_bounds__(ONE_THREADS) k_sig_one(Src src, int n, u64 *__restrict__ H, u32 *__restrict__ DC,
                                                         u64 *table, u64 tmask, const u32 *__restrict__ dep,
                                                         u64 hmask) {
  constexpr int NS = 2 * ONE_VERTS;
  __shared__ u64 key[ONE_VERTS];
  __shared__ u32 slots[NS];
  const u32 epoch = dep[EP_TABLE];
  const int64_t v0 = (int64_t)blockIdx.x * ONE_VERTS;
#pragma unroll
  for (int j = 0; j < NS / ONE_THREADS; ++j) slots[threadIdx.x + j * ONE_THREADS] = 0xFFFFFFFFu;
  __syncthreads();
  u64 h[ONE_ITEMS];
#pragma unroll
  for (int j = 0; j < ONE_ITEMS; ++j) {
    const int i = threadIdx.x + j * ONE_THREADS;
    const int64_t v = v0 + i;
    h[j] = 0;
    if (v >= n) continue;
    h[j] = finalize_key(mix_pair(src.pair(v)), 1u, src.own((int)v)) & hmask;
    H[v] = h[j];
    DC[v] = 1u;
    key[i] = h[j];
    atomicMin(&slots[(u32)(h[j] >> 20) & (NS - 1)], (u32)i);
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < ONE_ITEMS; ++j) {
    const int i = threadIdx.x + j * ONE_THREADS;
    if (v0 + i >= n) continue;
    const u32 m = slots[(u32)(h[j] >> 20) & (NS - 1)];
    if (m == (u32)i || key[m] != h[j]) table_insert(table, tmask, h[j], (u32)(v0 + i), epoch);
  }
}

// Row tier: one workgroup of NT threads per row of more entries than the
// range capacity and at most EMAX.  All entries are gathered at once (EMAX / NT per thread), then
// inserted into an LDS hash set of 2 * deg slots; first insertions add to
// thread-local sums, reduced over the workgroup at the end.
template <class Src, int EMAX, int NT, class K = u64>
__global__ void __launch_bounds__(NT) k_sig_row(Src src, const Range *__restrict__ rows, u64 *__restrict__ H,
                                                u32 *__restrict__ DC, KeySink sink,
                                                const u32 *__restrict__ dep, u64 hmask, u64 *zrep,
                                                const unsigned char *__restrict__ skip) {
  typedef Keys<K> KO;
  constexpr int U = EMAX / NT;
  __shared__ K set[2 * EMAX];
  __shared__ u64 sh_acc[NT / WAVE];
  __shared__ u32 sh_cnt[NT / WAVE];
  const int t = threadIdx.x;
  const Range rw = rows[blockIdx.x];
  const int v = rw.v0;
  if (skip && skip[v]) return;  // singleton block (work-efficient mode)
  const int64_t eb = rw.e0;
  const u32 own0 = t == 0 ? src.own(v) : 0u;  // fetched early, used by thread 0 at the end
  const int E = rw.ne;
  for (int i = t; i < 2 * E; i += NT) set[i] = KO::EMPTY;
  K pr[U];
  if (E > 0) {
    load_keys<K, U, NT>(src, eb, t, E, pr);
  } else {
#pragma unroll
    for (int u = 0; u < U; ++u) pr[u] = KO::EMPTY;
  }
  __syncthreads();
  u64 a = 0;
  u32 c = 0;
  const u32 sz = 2u * (u32)E;
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const K p = pr[u];
    if (p == KO::EMPTY) continue;
    u32 sl = scale_to(KO::hash(p), sz);
    while (true) {
      const K old = atomicCAS(&set[sl], KO::EMPTY, p);
      if (old == KO::EMPTY) { a += KO::mix(p); ++c; break; }
      if (old == p) break;
      sl = (sl + 1 == sz) ? 0u : sl + 1;
    }
  }
  block_reduce_2(a, c, sh_acc, sh_cnt);
  if (t == 0) {
    const u64 h = finalize_key(a, c, own0) & hmask;
    H[v] = h;
    DC[v] = c;
    if (sink.table) key_insert(sink.table, sink.tmask, zrep, h, c, own0, (u32)v, dep[EP_TABLE], dep[EP_ZERO]);
    else sink_key(sink, rw.row, v, h);
  }
}

// Hub tier (deg > BLOCK_MAX), two passes without per-entry global atomics.
//  stage:  a workgroup per chunk of hub_chunk entries removes duplicates
//          inside the chunk (LDS set), splits the chunk's distinct pairs into
//          the hub's P partitions by a partition hash and writes them,
//          grouped by partition, to the chunk's staging area together with
//          the P+1 partition offsets.
//  reduce: a workgroup per (hub, partition) reads that partition's segment
//          of every chunk of the hub, removes duplicates across chunks (LDS
//          set) and adds its distinct count and mix sum to the hub's totals.
struct HubChunk {
  int hub;          // index into the hub arrays
  int parts;        // partitions of this hub (power of two)
  int64_t b, e;     // entry range relative to the start of the hub's row
  int64_t stage;    // offset of the chunk's staging area (hub_chunk slots)
  int64_t poff;     // offset of the chunk's parts+1 partition offsets
};

struct HubPart {
  int hub;
  int part;
  int chunk0;       // first chunk of the hub
  int nchunks;
};

template <class Src, int CHUNK, class K = u64>
__global__ void __launch_bounds__(256) k_hub_stage(Src src, const HubChunk *__restrict__ chunks,
                                                   const int *__restrict__ hubs, K *__restrict__ stage,
                                                   int *__restrict__ poff, u32 *err,
                                                   const unsigned char *__restrict__ skip) {
  typedef Keys<K> KO;
  constexpr int HUB_U = CHUNK / 256;
  __shared__ K set[2 * CHUNK];
  __shared__ int hist[HUB_PMAX + 1];
  __shared__ int wtot[4];
  const HubChunk c = chunks[blockIdx.x];
  if (skip && skip[hubs[c.hub]]) return;  // singleton block (work-efficient mode)
  const int P = c.parts;
  const int64_t row = src.begin(hubs[c.hub]);
  const int E = (int)(c.e - c.b);
  for (int i = threadIdx.x; i < 2 * CHUNK; i += 256) set[i] = KO::EMPTY;
  for (int i = threadIdx.x; i <= P; i += 256) hist[i] = 0;
  K pr[HUB_U];
  if (E > 0) {
    load_keys<K, HUB_U, 256>(src, row + c.b, (int)threadIdx.x, E, pr);
  } else {
#pragma unroll
    for (int u = 0; u < HUB_U; ++u) pr[u] = KO::EMPTY;
  }
  __syncthreads();
  int rank[HUB_U];
#pragma unroll
  for (int u = 0; u < HUB_U; ++u) {
    rank[u] = -1;
    const K p = pr[u];
    if (p == KO::EMPTY) continue;
    u32 sl = KO::hash(p) & (2 * CHUNK - 1);
    while (true) {
      const K old = atomicCAS(&set[sl], KO::EMPTY, p);
      if (old == KO::EMPTY) {
        rank[u] = atomicAdd(&hist[part_hash(p) & (P - 1)], 1);
        break;
      }
      if (old == p) break;
      sl = (sl + 1) & (2 * CHUNK - 1);
    }
  }
  __syncthreads();
  // exclusive scan of hist[0..P) by the whole workgroup (P <= 1024: 4 per thread)
  {
    const int t = threadIdx.x, lane = t & 63, w = t >> 6;
    int v4[4];
    int sum = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int idx = t * 4 + k;
      v4[k] = idx < P ? hist[idx] : 0;
      sum += v4[k];
    }
    int x = sum;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int y = __shfl_up(x, o, WAVE);
      if (lane >= o) x += y;
    }
    if (lane == 63) wtot[w] = x;
    __syncthreads();
    int off = x - sum;
    for (int i = 0; i < w; ++i) off += wtot[i];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int idx = t * 4 + k;
      if (idx < P) {
        hist[idx] = off;
        poff[c.poff + idx] = off;
      }
      off += v4[k];
    }
    if (t == 255) poff[c.poff + P] = off;
    __syncthreads();
  }
#pragma unroll
  for (int u = 0; u < HUB_U; ++u) {
    if (rank[u] >= 0) {
      const K p = pr[u];
      stage[c.stage + hist[part_hash(p) & (P - 1)] + rank[u]] = p;
    }
  }
}

template <class Src, class K = u64>
__global__ void __launch_bounds__(256) k_hub_reduce(Src src, const HubPart *__restrict__ parts,
                                                    const HubChunk *__restrict__ chunks,
                                                    const K *__restrict__ stage, const int *__restrict__ poff,
                                                    u64 *hub_acc, u32 *hub_cnt, u32 *err, const int *__restrict__ hubs,
                                                    const unsigned char *__restrict__ skip) {
  typedef Keys<K> KO;
  constexpr int PS = sizeof(K) == 8 ? HUB_PSLOTS_WIDE : HUB_PSLOTS;
  __shared__ K set[PS];
  __shared__ int64_t sbase[HUB_PMAX]; // per chunk: staging position of this partition's segment
  __shared__ int pre[HUB_PMAX + 1];    // exclusive prefix of segment lengths
  __shared__ int wtot[4];
  __shared__ u64 sh_acc[4];
  __shared__ u32 sh_cnt[4];
  __shared__ u32 sh_fill[2];  // distinct keys in the set, overflow flag
  const HubPart hp = parts[blockIdx.x];
  if (skip && skip[hubs[hp.hub]]) return;  // singleton block (work-efficient mode)
  const int C = hp.nchunks;
  for (int i = threadIdx.x; i < PS; i += 256) set[i] = KO::EMPTY;
  // segment lengths, then an exclusive scan over the (at most 1024) chunks
  {
    const int t = threadIdx.x, lane = t & 63, w = t >> 6;
    int len4[4];
    int sum = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int ci = t * 4 + k;
      len4[k] = 0;
      if (ci < C) {
        const HubChunk c = chunks[hp.chunk0 + ci];
        const int a = poff[c.poff + hp.part], b = poff[c.poff + hp.part + 1];
        sbase[ci] = c.stage + a;
        len4[k] = b - a;
      }
      sum += len4[k];
    }
    int x = sum;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int y = __shfl_up(x, o, WAVE);
      if (lane >= o) x += y;
    }
    if (lane == 63) wtot[w] = x;
    __syncthreads();
    int off = x - sum;
    for (int i = 0; i < w; ++i) off += wtot[i];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int ci = t * 4 + k;
      if (ci < C) pre[ci] = off;
      off += len4[k];
    }
    if (t == 255) pre[C] = off;
    __syncthreads();
  }
  const int T = pre[C];
  // Distinct keys of this partition, PS slots at a time.  A partition is
  // planned to hold at most PS / 2 of them, but a skewed hub can put more in
  // one partition: then the set stops filling at 3/4 (so probes always end),
  // and the partition is redone in Q sub-passes, each taking the keys whose
  // sub-partition hash (independent of the partition and slot hashes) is q,
  // with Q doubled until every sub-pass fits.  Sub-passes hold disjoint key
  // sets, so their sums and counts add up to the partition's.
  u64 acc = 0;
  u32 cnt = 0;
  u32 Q = 1;
  for (u32 q = 0; q < Q;) {
    if (threadIdx.x == 0) { sh_fill[0] = 0; sh_fill[1] = 0; }
    __syncthreads();
    u64 pacc = 0;
    u32 pcnt = 0;
    for (int t0 = 0; t0 < T; t0 += 4 * 256) {
      // One read per batch: the barrier after each batch shows the marks of the
      // one before, and an unmarked set has room for a whole batch beyond 3/4.
      static_assert(PS / 4 * 3 - 1 + 4 * 256 < PS, "an empty slot ends every probe");
      const bool full = set_full(&sh_fill[1]);
      K pr[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int t = t0 + threadIdx.x + u * 256;
        pr[u] = KO::EMPTY;
        if (t < T) {
          int lo = 0, hi = C - 1;
          while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (pre[mid] <= t) lo = mid; else hi = mid - 1;
          }
          pr[u] = stage[sbase[lo] + (t - pre[lo])];
        }
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const K p = pr[u];
        if (p == KO::EMPTY) continue;
        if (Q > 1 && (sub_hash((u64)p) & (Q - 1)) != q) continue;
        u32 sl = KO::hash(p) & (PS - 1);
        while (true) {
          const K cur = set[sl];
          if (cur == p) break;
          if (cur == KO::EMPTY) {
            // once the pass has overflowed nothing more is inserted (it is redone)
            if (full) break;
            const K old = atomicCAS(&set[sl], KO::EMPTY, p);
            if (old == KO::EMPTY) {
              pacc += KO::mix(p);
              ++pcnt;
              if (atomicAdd(&sh_fill[0], 1u) + 1u >= (u32)(PS / 4 * 3)) mark_full(&sh_fill[1]);
              break;
            }
            if (old == p) break;
          }
          sl = (sl + 1) & (PS - 1);
        }
      }
      __syncthreads();
    }
    __syncthreads();
    const bool over = sh_fill[1] != 0;
    __syncthreads();
    for (int i = threadIdx.x; i < PS; i += 256) set[i] = KO::EMPTY;
    if (over) {
      if (Q >= 4096) {  // 4096 * PS * 3/4 slots exceed any staged hub; not reached
        if (threadIdx.x == 0) atomicOr(err, ERR_VERIFY_OVERFLOW);
        return;
      }
      Q <<= 1;
      q = 0;
      acc = 0;
      cnt = 0;
    } else {
      acc += pacc;
      cnt += pcnt;
      ++q;
    }
    __syncthreads();
  }
  block_reduce_2(acc, cnt, sh_acc, sh_cnt);
  if (threadIdx.x == 0) {
    if (acc) atomicAdd(&hub_acc[hp.hub], acc);
    if (cnt) atomicAdd(&hub_cnt[hp.hub], cnt);
  }
}

// Very large hubs (deg > HUB_STAGED_MAX, or HUB_STAGED_MAX_WIDE with 64-bit
// keys): workgroups of one hub share a
// global hash set of 2*deg slots; slot = pair | (epoch << 62), 0 = unused,
// epochs 1..3.  Pairs are < 2^62.
struct HubGChunk {
  int hub;
  int pad;
  int64_t b, e;      // entry range relative to the start of the hub's row
  int64_t set_off;   // the hub's global set
  int64_t set_size;
};

// Set slots hold key | epoch << 62 and count as empty unless their epoch is
// the current one, so dep[EP_HUB] must be 1..3 (advanced at least once; a
// zeroed set with epoch 0 would have no empty slot) and each set must hold
// more slots than its row has entries.
template <class Src, class K>
__global__ void __launch_bounds__(256) k_sig_hub_global(Src src, const HubGChunk *__restrict__ chunks,
                                                        const int *__restrict__ hubs, u64 *sets, u64 *hub_acc,
                                                        u32 *hub_cnt, const u32 *__restrict__ dep,
                                                        const unsigned char *__restrict__ skip) {
  const u32 hepoch = dep[EP_HUB];
  __shared__ u64 sh_acc[4];
  __shared__ u32 sh_cnt[4];
  const HubGChunk c = chunks[blockIdx.x];
  if (skip && skip[hubs[c.hub]]) return;  // singleton block (work-efficient mode)
  u64 *set = sets + c.set_off;
  const u64 size = (u64)c.set_size;
  const int64_t row = src.begin(hubs[c.hub]);
  u64 acc = 0;
  u32 cnt = 0;
  for (int64_t i = row + c.b + threadIdx.x; i < row + c.e; i += 256) {
    const K key = Keys<K>::load(src, i);  // the tiers of one graph dedupe the same keys
    const u64 want = (u64)key | ((u64)hepoch << 62);
    u64 sl = scale_to(set_hash((u64)key), size);
    while (true) {
      u64 cur = __hip_atomic_load(&set[sl], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      bool done = false;
      while ((cur >> 62) != (u64)hepoch) {
        const u64 old = atomicCAS(&set[sl], cur, want);
        if (old == cur) { acc += Keys<K>::mix(key); ++cnt; done = true; break; }
        cur = old;
      }
      if (done || cur == want) break;
      sl = (sl + 1 == size) ? 0 : sl + 1;
    }
  }
  block_reduce_2(acc, cnt, sh_acc, sh_cnt);
  if (threadIdx.x == 0) {
    if (acc) atomicAdd(&hub_acc[c.hub], acc);
    if (cnt) atomicAdd(&hub_cnt[c.hub], cnt);
  }
}

template <class Src>
__global__ void k_hub_final(Src src, const int *__restrict__ hubs, int nhub, u64 *hub_acc, u32 *hub_cnt,
                            u64 *__restrict__ H, u32 *__restrict__ DC, KeySink sink,
                            const u32 *__restrict__ dep, u64 hmask, u64 *zrep,
                            const unsigned char *__restrict__ skip, const int *__restrict__ nzv, int nonempty) {
  const u32 epoch = dep[EP_TABLE], zep = dep[EP_ZERO];
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= nhub) return;
  const int v = hubs[i];
  const u64 acc = hub_acc[i];
  const u32 cnt = hub_cnt[i];
  hub_acc[i] = 0;
  hub_cnt[i] = 0;
  if (skip && skip[v]) return;  // singleton block (work-efficient mode)
  const u32 own = src.own(v);
  const u64 h = finalize_key(acc, cnt, own) & hmask;
  H[v] = h;
  DC[v] = cnt;
  if (sink.table) {
    key_insert(sink.table, sink.tmask, zrep, h, cnt, own, (u32)v, epoch, zep);
  } else {
    int lo = 0, hi = nonempty;  // the hub's place among the non-empty rows
    while (hi - lo > 1) {
      const int mid = lo + ((hi - lo) >> 1);
      if (nzv[mid] <= v) lo = mid;
      else hi = mid;
    }
    sink_key(sink, lo, v, h);
  }
}

constexpr int XCDS = 8;  // workgroups go to the XCDs in turn
// Tile of this workgroup (>= ntiles: none; grids are padded to a multiple of
// XCDS): each XCD takes a contiguous share of the tiles in order, so that the
// runs that neighbouring tiles write side by side meet in one L2 and leave it
// as whole lines (9.25 -> 7.6 ms per summary graph of 125M entries).
__device__ inline int64_t radix_tile(int64_t ntiles) {
  return (int64_t)(blockIdx.x % XCDS) * ((ntiles + XCDS - 1) / XCDS) + blockIdx.x / XCDS;
}

// ---------------------------------------------------------------- grouping by partition
// The table's inserts are device-wide atomics on random lines (about 25 G/s
// here) and every vertex probes a random line again to find its minimum.
// Large steps group without it: the signature kernels leave H, and rep[v] = v
// for one vertex per key of a workgroup (rep = that vertex for its others,
// which go no further); (H, v) pairs are partitioned by 16 hash bits in two
// stable radix passes; workgroups then find the minimum vertex of each key of
// whole buckets in LDS, and write rep[v] only where the minimum is another
// vertex (few, once most blocks are single vertices).  On the 1B-edge graph (40M
// keys per step) the passes and buckets take 0.9 ms; the table's inserts cost the
// range kernel 1.3 ms (9.49 -> 8.17) and its lookups 1.7 (k_resolve: 0.39).
constexpr int GROUP_THREADS = 512, GROUP_ITEMS = 8;
constexpr int GROUP_TILE = GROUP_THREADS * GROUP_ITEMS;  // pairs per radix tile
static_assert(GROUP_TILE == 4096, "12-bit slots");
constexpr int GROUP_BITS = 16;                           // bucket bits, the low ones of H
constexpr u32 GROUP_MASK = (1u << GROUP_BITS) - 1u;      // (the kernels take the mask: a test keeps fewer)
constexpr int GROUP_SLOTS = 4096;  // slots of the set of k_group_buckets (32 KB)
// Digit of a pass: 8 bits of the bucket.
__device__ inline u32 group_digit(u64 h, u32 mask, int shift) { return ((u32)h & mask) >> shift & 255u; }

// Pairs of a pass (the first: all rows; the second: what the first left), and
// this workgroup's tile of them (>= the number of tiles: none).  The tiles that
// hold pairs are dealt to the XCDs as in radix_tile, and their histograms lie
// together: dealt out over the rows, the pairs of a step with few keys all fell
// to the first XCD (unlabelled graph of 120M rows: the second histogram 415 -> 134
// us, the scatters 241 -> 201 on average).
__device__ inline int64_t group_tiles(int64_t count, const int64_t *total, int64_t &pairs, int64_t &tile) {
  pairs = total ? *total : count;
  const int64_t nt = (pairs + GROUP_TILE - 1) / GROUP_TILE;
  tile = (int64_t)(blockIdx.x / XCDS) < (nt + XCDS - 1) / XCDS ? radix_tile(nt) : nt;
  return nt;
}

// Pair `at` of a pass: its key (EMPTY64: none) and, with vals, its vertex.
__device__ inline void group_load(int64_t at, int64_t count, const u64 *__restrict__ keys,
                                  const int *__restrict__ vals, bool &valid, u64 &key, int &v) {
  const bool in = at < count;
  key = in ? __builtin_nontemporal_load(&keys[at]) : EMPTY64;
  v = in && vals ? __builtin_nontemporal_load(&vals[at]) : 0;
  valid = key != EMPTY64;
}

// Digit histogram of each tile (tiles dealt to the XCDs as radix_tile).
// DROP (second pass): keys that many rows share drop out, all but one per tile,
// which a single workgroup would otherwise walk in the key's bucket.  A tile now
// holds one digit or two of the first pass, so the pairs of such a key (one per
// range of rows) lie together: where a digit has more than GROUP_HOT keys of a tile
// (16 are there by chance, more than 40 once in 30,000 tiles), its equal keys meet
// in an LDS table and all but the minimum vertex of each drop out (rep = that
// vertex).  A bucket gets at most about n / 26,000 pairs of one key (dropped in the
// first pass, by the same mark, where rows lie as they come: n / 100).  Unlabelled
// graphs, per step, k_group_buckets with drops in the first pass and in the second:
// 4.8M entries 38 / 14 us, 24M 173 / 37; both histograms together 22 / 27, 82 / 108.
constexpr int GROUP_HOT = 40;
template <bool DROP>
__global__ void __launch_bounds__(GROUP_THREADS) k_group_hist(int64_t count, const int64_t *__restrict__ total,
                                                              const int *__restrict__ vals, int *rep, u64 *keys,
                                                              u32 mask, int shift, int64_t max_tiles,
                                                              int *__restrict__ hist) {
  __shared__ int h[256];
  __shared__ u64 slot[DROP ? GROUP_TILE : 1];
  __shared__ u32 mins[DROP ? GROUP_TILE : 1];
  int64_t cnt, tile;
  const int64_t ntiles = group_tiles(count, total, cnt, tile);
  // (the scan goes over the counters of max_tiles tiles: zeros past those used)
  if (blockIdx.x >= ntiles && blockIdx.x < max_tiles && threadIdx.x < 256)
    hist[(int64_t)blockIdx.x * 256 + threadIdx.x] = 0;
  if (tile >= ntiles) return;
  if (threadIdx.x < 256) h[threadIdx.x] = 0;
  __syncthreads();
  u64 key[GROUP_ITEMS];
  bool valid[GROUP_ITEMS];
  const int64_t i0 = tile * GROUP_TILE + threadIdx.x;
#pragma unroll
  for (int j = 0; j < GROUP_ITEMS; ++j) {
    int none;
    group_load(i0 + j * GROUP_THREADS, cnt, keys, nullptr, valid[j], key[j], none);
  }
#pragma unroll
  for (int j = 0; j < GROUP_ITEMS; ++j)
    if (valid[j]) atomicAdd(&h[group_digit(key[j], mask, shift)], 1);
  __syncthreads();
  if constexpr (DROP) {
    if (__syncthreads_or(threadIdx.x < 256 && h[threadIdx.x] > GROUP_HOT)) {
#pragma unroll
      for (int j = 0; j < GROUP_ITEMS; ++j)  // (keys of the other digits take no part)
        valid[j] = valid[j] && h[group_digit(key[j], mask, shift)] > GROUP_HOT;
      for (int i = threadIdx.x; i < GROUP_TILE; i += GROUP_THREADS) {
        slot[i] = EMPTY64;
        mins[i] = 0xFFFFFFFFu;
      }
      __syncthreads();
      int at[GROUP_ITEMS], v[GROUP_ITEMS];
#pragma unroll
      for (int j = 0; j < GROUP_ITEMS; ++j) v[j] = valid[j] ? vals[i0 + j * GROUP_THREADS] : 0;
#pragma unroll
      for (int j = 0; j < GROUP_ITEMS; ++j) {
        if (!valid[j]) continue;
        u32 s = (u32)(key[j] >> GROUP_BITS) * 0x9E3779B1u >> 20;  // 12 bits: no fewer slots than keys
        while (true) {
          u64 old = slot[s];
          if (old == EMPTY64) old = atomicCAS(&slot[s], EMPTY64, key[j]);
          if (old == EMPTY64 || old == key[j]) break;
          s = (s + 1) & (GROUP_TILE - 1);
        }
        at[j] = (int)s;
        if (mins[s] > (u32)v[j]) atomicMin(&mins[s], (u32)v[j]);
      }
      __syncthreads();
#pragma unroll
      for (int j = 0; j < GROUP_ITEMS; ++j) {
        if (!valid[j]) continue;
        const int first = (int)mins[at[j]];
        if (first != v[j]) {
          rep[v[j]] = first;
          keys[i0 + j * GROUP_THREADS] = EMPTY64;
          atomicSub(&h[group_digit(key[j], mask, shift)], 1);
        }
      }
      __syncthreads();
    }
  }
  if (threadIdx.x < 256) hist[(int64_t)threadIdx.x * ntiles + tile] = h[threadIdx.x];
}

// Stable scatter of a tile's pairs by their digit (as k_radix_scatter).
__global__ void __launch_bounds__(GROUP_THREADS) k_group_scatter(int64_t count, const int64_t *__restrict__ total,
                                                                 const u64 *__restrict__ keys,
                                                                 const int *__restrict__ vals, u32 mask, int shift,
                                                                 const int64_t *__restrict__ offs,
                                                                 u64 *__restrict__ out_keys,
                                                                 int *__restrict__ out_vals) {
  constexpr int NW = GROUP_THREADS / WAVE;
  __shared__ u64 sk[GROUP_TILE];
  __shared__ int sv[GROUP_TILE];
  __shared__ int64_t gpos[256];
  __shared__ int wcnt[NW][256];
  __shared__ u32 sh_w[4];
  __shared__ int sh_n;
  int64_t cnt, tile;
  const int64_t ntiles = group_tiles(count, total, cnt, tile);
  if (tile >= ntiles) return;
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  const int64_t goff = t < 256 ? offs[(int64_t)t * ntiles + tile] : 0;
  const u64 lt = (1ULL << lane) - 1ULL;
  u64 key[GROUP_ITEMS];
  int val[GROUP_ITEMS];
  bool valid[GROUP_ITEMS];
  const int64_t i0 = tile * GROUP_TILE + w * (WAVE * GROUP_ITEMS) + lane;
#pragma unroll
  for (int j = 0; j < GROUP_ITEMS; ++j)
    group_load(i0 + j * WAVE, cnt, keys, vals, valid[j], key[j], val[j]);
#pragma unroll
  for (int q = 0; q < 256 / WAVE; ++q) wcnt[w][q * WAVE + lane] = 0;
  __builtin_amdgcn_wave_barrier();
  int rank[GROUP_ITEMS];
#pragma unroll
  for (int j = 0; j < GROUP_ITEMS; ++j) {
    const u32 d = group_digit(key[j], mask, shift);
    u64 peers = __ballot(valid[j]);
#pragma unroll
    for (int b = 0; b < 8; ++b) {
      const u64 ones = __ballot((d >> b) & 1u);
      peers &= ((d >> b) & 1u) ? ones : ~ones;
    }
    const int below = __popcll(peers & lt);
    const int before = wcnt[w][d];
    __builtin_amdgcn_wave_barrier();
    if (valid[j] && below == 0) wcnt[w][d] = before + __popcll(peers);
    __builtin_amdgcn_wave_barrier();
    rank[j] = before + below;
  }
  __syncthreads();
  {
    u32 c = 0;
    if (t < 256)
#pragma unroll
      for (int q = 0; q < NW; ++q) c += (u32)wcnt[q][t];
    u32 x = c;
#pragma unroll
    for (int o = 1; o < WAVE; o <<= 1) {
      const u32 y = __shfl_up(x, o, WAVE);
      if (lane >= o) x += y;
    }
    if (t < 256 && lane == WAVE - 1) sh_w[w] = x;
    __syncthreads();
    if (t < 256) {
      int at = (int)(x - c);
      for (int i = 0; i < w; ++i) at += (int)sh_w[i];
      gpos[t] = goff - at;
#pragma unroll
      for (int q = 0; q < NW; ++q) {
        const int m = wcnt[q][t];
        wcnt[q][t] = at;
        at += m;
      }
      if (t == 255) sh_n = at;
    }
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < GROUP_ITEMS; ++j) {
    if (!valid[j]) continue;
    const int at = wcnt[w][group_digit(key[j], mask, shift)] + rank[j];
    sk[at] = key[j];
    sv[at] = val[j];
  }
  __syncthreads();
  const int n = sh_n;
#pragma unroll
  for (int j = 0; j < GROUP_ITEMS; ++j) {
    const int i = j * GROUP_THREADS + t;
    if (i < n) {
      const u64 k = sk[i];
      const int64_t o = gpos[group_digit(k, mask, shift)] + i;
      out_keys[o] = k;
      out_vals[o] = sv[i];
    }
  }
}

// Links the vertices of every key of the buckets that start in this workgroup's
// chunk.  Equal keys share a bucket, so the LDS table sees all of them; it
// holds the distinct keys of about a chunk (stretches end at bucket starts).
// Slots are (high hash word << 32 | vertex), the smallest vertex so far: of two
// vertices that meet, the larger gets a link (rep) to the smaller, so every
// vertex but the minimum is linked once, along a chain that ends there, and
// one look at each pair is enough.  Two keys that share bucket, slot run and
// high word meet in one group; the exact check separates them.  A stretch with
// more than 3/4 of the slots distinct is redone in Q sub-passes by other hash
// bits, Q doubled until each fits.  From about 185M pairs on the mean bucket is
// longer than that by itself and says how many sub-passes to begin with, so that
// none is walked in vain (mean_bits: bucket bits of that estimate).
// U: pairs in flight per thread; a chunk is one round of them.  With 2 (chunks of
// 1,024) a stretch holds one bucket of up to 2,048 pairs; two in a stretch of 2,048
// overflow from 100M rows on.  From BUCKET_WIDE pairs a bucket, of which every
// stretch holds one at most, 4 in flight read it faster.  Distinct keys, U = 2 / 4,
// ms per step: 4M rows 0.036 / 0.052, 40M 0.34 / 0.39, 90M 0.81 / 1.03, 110M 1.05 /
// 2.03, 130M 1.38 / 2.06, 160M 2.02 / 1.72, 200M 2.70 / 2.21.
constexpr int64_t BUCKET_WIDE = 2048;
constexpr int BUCKET_GROUP = 512;
constexpr u32 BUCKET_FIT = GROUP_SLOTS / 16 * 11;  // mean pairs of a planned pass: 3/4 less 5 standard deviations
template <int U>
__global__ void __launch_bounds__(BUCKET_GROUP) k_group_buckets(const int64_t *__restrict__ total_p,
                                                       const u64 *__restrict__ keys, const int *__restrict__ vals,
                                                       u32 mask, int mean_bits, int *__restrict__ rep,
                                                       u32 *err) {
  constexpr int BATCH = BUCKET_GROUP * U;  // a chunk, and the pairs in flight (launched with BUCKET_GROUP threads)
  static_assert(GROUP_SLOTS / 4 > BUCKET_GROUP, "an empty slot ends every probe");
  __shared__ u64 slot[GROUP_SLOTS];
  __shared__ u32 sh[2];
  __shared__ u32 fill[2];
  const int t = threadIdx.x;
  const int64_t total = *total_p;
  const int64_t c0 = (int64_t)blockIdx.x * BATCH;
  if (c0 >= total) return;
  u32 Q = 1;
  while ((u32)(total >> mean_bits) / Q > BUCKET_FIT) Q <<= 1;
  for (int i = t; i < GROUP_SLOTS; i += BUCKET_GROUP) slot[i] = EMPTY64;
  if (t < 2) fill[t] = 0;
  auto put = [&](u64 key, int x) {
    const u32 tag = (u32)(key >> 32);
    const u64 want = (key & 0xFFFFFFFF00000000ULL) | (u64)(u32)x;
    u32 s = (u32)(key >> GROUP_BITS) * 0x9E3779B1u >> 20;  // 12 bits: GROUP_SLOTS
    const bool full = set_full(&fill[1]);
    while (true) {
      u64 cur = slot[s];
      if (cur == EMPTY64) {
        // overflowed: nothing more goes in, the stretch is redone (free slots
        // remain: at most one insertion per thread lands after the mark)
        if (full) return;
        cur = atomicCAS(&slot[s], EMPTY64, want);
        if (cur == EMPTY64) {
          if (atomicAdd(&fill[0], 1u) + 1u >= (u32)(GROUP_SLOTS / 4 * 3)) mark_full(&fill[1]);
          return;
        }
      }
      if ((u32)(cur >> 32) == tag) {
        cur = atomicMin(&slot[s], want);
        if ((u32)cur < (u32)x) rep[x] = (int)(u32)cur;
        else if ((u32)cur > (u32)x) rep[(u32)cur] = x;
        return;
      }
      s = (s + 1) & (GROUP_SLOTS - 1);
    }
  };
  // from the first bucket start in the chunk to the first one past it
  int64_t b0 = -1, e = total;
  for (int64_t at = c0;; at += BATCH) {
    u64 k[U];
    int v[U];
    u32 edge = BATCH;  // first bucket start of the batch (the end counts as one)
#pragma unroll
    for (int j = 0; j < U; ++j) {
      const int64_t i = at + j * BUCKET_GROUP + t;
      k[j] = i < total ? keys[i] : 0ULL;
      v[j] = i < total ? vals[i] : 0;
    }
#pragma unroll
    for (int j = U - 1; j >= 0; --j) {
      const int64_t i = at + j * BUCKET_GROUP + t;
      if (i == 0 || i >= total || (((u32)keys[i - 1] ^ (u32)k[j]) & mask) != 0) edge = j * BUCKET_GROUP + t;
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) edge = min(edge, (u32)__shfl_xor(edge, o, WAVE));
    __syncthreads();
    if (t == 0) sh[0] = BATCH;
    __syncthreads();
    if ((t & (WAVE - 1)) == 0) atomicMin(&sh[0], edge);
    __syncthreads();
    edge = sh[0];
    u32 lo = 0, hi = BATCH;
    const bool past = at >= c0 + BATCH;
    if (past) {
      hi = edge;
    } else if (b0 < 0) {
      lo = edge;
      if (edge < BATCH && at + edge < total) b0 = at + edge;
    }
#pragma unroll
    for (int j = 0; j < U; ++j) {
      const u32 p = (u32)(j * BUCKET_GROUP + t);
      if (p >= lo && p < hi && at + p < total && (Q == 1 || (sub_hash(k[j]) & (Q - 1)) == 0)) put(k[j], v[j]);
    }
    if (past && edge < BATCH) {
      e = at + edge;
      break;
    }
    if (at + BATCH >= total) break;
    if (b0 < 0 && at + BATCH >= c0 + BATCH) return;  // no bucket starts in this chunk
  }
  if (b0 < 0) return;
  __syncthreads();
  u32 q = 1;
  if (fill[1]) {
    Q <<= 1;
    q = 0;
  }
  while (q < Q) {
    __syncthreads();
    for (int i = t; i < GROUP_SLOTS; i += BUCKET_GROUP) slot[i] = EMPTY64;
    if (t < 2) fill[t] = 0;
    __syncthreads();
    for (int64_t at = b0 + t; at < e; at += BATCH) {
      u64 k[U];
      int v[U];
#pragma unroll
      for (int j = 0; j < U; ++j) {
        const int64_t i = min(at + j * BUCKET_GROUP, e - 1);
        k[j] = keys[i];
        v[j] = vals[i];
      }
#pragma unroll
      for (int j = 0; j < U; ++j)
        if (at + j * BUCKET_GROUP < e && (sub_hash(k[j]) & (Q - 1)) == q) put(k[j], v[j]);
    }
    __syncthreads();
    if (!fill[1]) {
      ++q;
    } else if (Q < (1u << 24)) {
      Q <<= 1;
      q = 0;
    } else {  // more distinct keys than a stretch has pairs; not reached
      if (t == 0) atomicOr(err, ERR_VERIFY_OVERFLOW);
      return;
    }
  }
}

// ---------------------------------------------------------------- lookup + exact check
// Pairs of the entries first + u, u < 4, EMPTY64 from u = count on.  The words and
// then the gathers of all four are requested together; lanes without an entry
// read the first of all rows and the first target, which they share.
template <class Src>
__device__ inline void four_pairs(const Src &src, int64_t first, int count, u64 *p) {
  u32 l[4][1], r[4][1];
#pragma unroll
  for (int u = 0; u < 4; ++u) src.template entries<1, 1>(u < count ? first + u : 0, 0, 1, l[u], r[u]);
#pragma unroll
  for (int u = 0; u < 4; ++u) p[u] = src.pair_of(l[u][0], u < count ? r[u][0] : 0u);
#pragma unroll
  for (int u = 0; u < 4; ++u) p[u] = u < count ? p[u] : EMPTY64;
}

// 1 or 0: the rows of v and r hold the same pairs or not; -1: one of them has
// more than SMALL_MAX entries.  Every pair of v must occur in r and every pair of
// r in v (set equality in both directions, so it does not rest on the distinct
// counts).  Loads are what bounds it, so four entries of a row are in flight at a
// time, and RU pairs of v are held, r (the row that many lanes may share) being read
// again for each RU of them: with all 16 held, lookups of mostly heads have too few
// waves in flight.  Ten steps, entry by entry / 16 pairs of r held / 8 of r / 8 of v:
// unlabelled graphs of 20M vertices and 160M entries 64.3 / 59.6 / 63.3 / 60.6 ms,
// 60M and 72M 47.9 / 46.5 / 46.4 / 46.4, 1M and 1.2M (k_lookup) 0.99 / 0.94 / 0.91 /
// 0.91; work-efficient calls on 250M entries 8.3 / 8.4 / 8.3 / 8.3, on 50M entries of
// 9 a row that share their keys 3.48 / - / 3.61 / 3.37.
template <class Src>
__device__ inline int same_small_rows(const Src &src, int v, int r) {
  constexpr int RU = Src::GRAPH ? 8 : 4;  // (label sets are short)
  const int64_t bv = src.begin(v), lv = src.end(v) - bv;
  const int64_t br = src.begin(r), lr = src.end(r) - br;
  if (lv > SMALL_MAX || lr > SMALL_MAX) return -1;
  const int dv = (int)lv, dr = (int)lr;
  u32 in_r = 0, in_v = 0;  // entries of v found in r, and of r found in v
  for (int g = 0; g < dv; g += RU) {
    u64 vp[RU];
#pragma unroll
    for (int q = 0; q < RU; q += 4) {
      if (q == 0 || g + q < dv) four_pairs(src, bv + g + q, dv - g - q, vp + q);
      else vp[q] = vp[q + 1] = vp[q + 2] = vp[q + 3] = EMPTY64;
    }
    for (int i = 0; i < dr; i += 4) {
      u64 p[4];
      four_pairs(src, br + i, dr - i, p);
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        u32 hit = 0;
#pragma unroll
        for (int q = 0; q < RU; ++q) hit |= (vp[q] == p[u] ? 1u : 0u) << q;
        in_r |= hit << g;
        in_v |= (hit != 0 ? 1u : 0u) << (i + u);
      }
    }
  }
  const u32 all_v = (1u << dv) - 1u, all_r = (1u << dr) - 1u;
  return (in_r & all_v) == all_v && (in_v & all_r) == all_r ? 1 : 0;
}

// From the vertex that spoke for v, if any, to the minimum of its key.  Links
// only ever point on to that minimum (a collided vertex keeps its link, so that
// others can walk over it; peeling gives it its representative).
__device__ inline int key_minimum(const int *rep, int v) {
  int r = rep[v];
  for (int nx = rep[r]; nx != r; nx = rep[r]) r = nx;
  return r;
}

// k_lookup's work after a partition, over the list of non-empty vertices: a wave
// takes RESOLVE_V of them and looks only at those whose representative is another
// vertex, so that a wave of heads ends after two loads.  These are packed and
// taken 64 at a time: neighbouring lanes then read neighbouring rows, and long
// rows are listed with one atomic per wave.  A thread that walked the up to four
// of its own read rows at a stride, which cost more than the table's lookups where
// most rows share their keys: unlabelled graphs of 20M vertices, 160M entries
// 5.49 -> 3.69 ms a step (k_lookup 3.68), 24M entries 0.90 -> 0.66 (0.68).
constexpr int RESOLVE_V = 256;
template <class Src>
__global__ void __launch_bounds__(256) k_resolve(Src src, int count, const int *__restrict__ list,
                                                 const u32 *__restrict__ DC, int *rep, int *vcount, int *vlist,
                                                 int *ccount, int *clist) {
  constexpr int U = RESOLVE_V / WAVE;
  __shared__ int held[4][RESOLVE_V];  // per wave: vertices to look at, then those with long rows
  const int lane = threadIdx.x & (WAVE - 1), w = threadIdx.x >> 6;
  const int64_t base = ((int64_t)blockIdx.x * 4 + w) * RESOLVE_V;
  const u64 lt = (1ULL << lane) - 1ULL;
  int v[U], c[U];
#pragma unroll
  for (int j = 0; j < U; ++j) v[j] = base + j * WAVE + lane < count ? list[base + j * WAVE + lane] : -1;
#pragma unroll
  for (int j = 0; j < U; ++j) c[j] = v[j] >= 0 ? rep[v[j]] : -1;
  int pending = 0;  // uniform in the wave
#pragma unroll
  for (int j = 0; j < U; ++j) {
    const u64 mask = __ballot(c[j] != v[j]);
    if (c[j] != v[j]) held[w][pending + __popcll(mask & lt)] = v[j];
    pending += __popcll(mask);
  }
  __builtin_amdgcn_wave_barrier();
  int longs = 0;
  for (int b = 0; b < pending; b += WAVE) {
    const bool act = b + lane < pending;
    const int x = act ? held[w][b + lane] : 0;
    int eq = 0;
    if (act) {
      const int r = key_minimum(rep, x);
      if (src.own(x) == src.own(r)) eq = same_small_rows(src, x, r);
      if (eq < 0 && DC[x] != DC[r]) eq = 0;  // (equal short rows need no look at their counts)
      if (eq != 0) rep[x] = r;
    }
    __builtin_amdgcn_wave_barrier();  // (places up to b + 63 have been read)
    const u64 mask = __ballot(act && eq < 0);
    if (act && eq < 0) held[w][longs + __popcll(mask & lt)] = x;
    longs += __popcll(mask);
    wave_append(ccount, clist, act && eq == 0, x);
  }
  if (longs == 0) return;
  __builtin_amdgcn_wave_barrier();
  int at = 0;
  if (lane == 0) at = atomicAdd(vcount, longs);
  at = __shfl(at, 0, WAVE);
  for (int i = lane; i < longs; i += WAVE) vlist[at + i] = held[w][i];
}

// For each vertex: representative r = minimum vertex stored under its key.
// r == v: v heads its block.  Otherwise v joins r's block once the keys are
// shown equal exactly: the previous block, the number of distinct pairs and,
// for rows of at most SMALL_MAX entries, the pair sets here; larger rows go
// to a verification list (k_verify).  Mismatches (hash collisions) go to the
// collision list with rep = -1.  Lists are appended with one atomic per
// wave; they stay short, since device-wide atomics on one counter serialise.
// Updates (dirty != NULL): a vertex and its candidate that are both clean
// (key inputs unchanged) and shared a block in the cached chain (same cached
// name mvc) still have equal keys, so they are accepted without the check.
template <class Src>
__global__ void __launch_bounds__(256) k_lookup(Src src, int count, const int *__restrict__ list,
                                                const u64 *__restrict__ H, const u32 *__restrict__ DC,
                                                const u64 *table, u64 tmask, const u32 *__restrict__ dep,
                                                int *__restrict__ rep, int *vcount, int *vlist, int *ccount,
                                                int *clist, u32 *err, const u64 *zrep, int zfresh,
                                                const unsigned char *__restrict__ skip,
                                                const unsigned char *__restrict__ dirty,
                                                const int32_t *__restrict__ mvc) {
  const u32 epoch = dep[EP_TABLE], zep = dep[EP_ZERO];
  const int i = blockIdx.x * 256 + threadIdx.x;
  const bool act = i < count;
  const int v = act ? (list ? list[i] : i) : 0;
  bool to_verify = false, collided = false;
  if (act && skip && skip[v]) {
    rep[v] = v;  // a singleton block stays a singleton
  } else if (act) {
    const u32 dcv = DC[v];
    if (dcv == 0) {
      // empty signature: exact grouping by previous block (without zfresh the
      // representative is kept from the call's first step)
      if (zfresh) {
        const u64 z = zrep[src.own(v)];
        if ((u32)(z >> 32) != ~zep) {
          atomicOr(err, ERR_LOOKUP_MISS);
          rep[v] = v;
        } else {
          rep[v] = (int)(u32)z;
        }
      }
    } else {
      const int r = table_lookup(table, tmask, H[v], epoch);
      if (r < 0) {
        atomicOr(err, ERR_LOOKUP_MISS);
        rep[v] = v;
      } else if (r == v) {
        rep[v] = v;
      } else if (src.own(v) != src.own(r) || dcv != DC[r]) {
        rep[v] = -1;
        collided = true;
      } else if (dirty && !dirty[v] && !dirty[r] && mvc[v] == mvc[r]) {
        rep[v] = r;
      } else {
        const int eq = same_small_rows(src, v, r);
        if (eq != 0) rep[v] = r;  // (long rows: confirmed or rejected by k_verify)
        else rep[v] = -1;
        to_verify = eq < 0;
        collided = eq == 0;
      }
    }
  }
  wave_append(vcount, vlist, to_verify, v);
  wave_append(ccount, clist, collided, v);
}

// Exact set check of v against r with one workgroup: the distinct pairs of r
// go into an LDS hash set (in several passes, split by a partition hash, when
// they do not fit), and every pair of v is looked up.  Result: 1 if every pair
// of v occurs in r's row, 0 if not, -1 if a pass overflowed the LDS set (the
// caller retries with more passes).  Must be called by the whole workgroup.
template <class Src>
__device__ int wg_subset_pass(const Src &src, int v, int r, u32 parts, u64 *set, int *sh_flag) {
  const int64_t bv = src.begin(v), ev = src.end(v);
  const int64_t br = src.begin(r), er = src.end(r);
  for (u32 q = 0; q < parts; ++q) {
    for (int i = threadIdx.x; i < BLOCK_SLOTS; i += blockDim.x) set[i] = EMPTY64;
    if (threadIdx.x == 0) { sh_flag[0] = 1; sh_flag[1] = 0; }
    __syncthreads();
    for (int64_t i = br + threadIdx.x; i < er; i += blockDim.x) {
      const u64 p = src.pair(i);
      if (parts > 1 && (part_hash(p) & (parts - 1)) != q) continue;
      u32 s = set_hash(p) & (BLOCK_SLOTS - 1);
      for (int probes = 0;; ++probes) {
        if (probes >= BLOCK_SLOTS) { sh_flag[1] = 1; break; }
        const u64 old = atomicCAS(&set[s], EMPTY64, p);
        if (old == EMPTY64 || old == p) break;
        s = (s + 1) & (BLOCK_SLOTS - 1);
      }
    }
    __syncthreads();
    const bool overflow = sh_flag[1] != 0;
    if (!overflow) {
      for (int64_t i = bv + threadIdx.x; i < ev; i += blockDim.x) {
        const u64 p = src.pair(i);
        if (parts > 1 && (part_hash(p) & (parts - 1)) != q) continue;
        u32 s = set_hash(p) & (BLOCK_SLOTS - 1);
        bool found = false;
        for (int probes = 0; probes < BLOCK_SLOTS; ++probes) {
          const u64 x = set[s];
          if (x == p) { found = true; break; }
          if (x == EMPTY64) break;
          s = (s + 1) & (BLOCK_SLOTS - 1);
        }
        if (!found) sh_flag[0] = 0;
      }
    }
    __syncthreads();
    const int res = overflow ? -1 : (sh_flag[0] != 0 ? 1 : 0);
    __syncthreads();
    if (res != 1) return res;
  }
  return 1;
}

template <class Src>
__device__ bool wg_subset_one(const Src &src, int v, int r, u32 dcr, u64 *set, int *sh_flag, u32 *err) {
  u32 parts = 1;
  while ((u64)parts * (BLOCK_SLOTS / 2) < (u64)dcr) parts <<= 1;
  while (true) {
    const int res = wg_subset_pass(src, v, r, parts, set, sh_flag);
    if (res >= 0) return res == 1;
    if (parts >= (1u << 24)) {
      if (threadIdx.x == 0) atomicOr(err, ERR_VERIFY_OVERFLOW);
      return false;
    }
    parts <<= 1;
  }
}

// Equal signatures of v and r, given equal distinct counts.  With exact keys
// the counts are the pair counts and one inclusion decides; with hashed keys
// they count distinct keys, so both inclusions are checked.
template <class Src>
__device__ bool wg_subset(const Src &src, int v, int r, u32 dcr, u64 *set, int *sh_flag, u32 *err) {
  if (!wg_subset_one(src, v, r, dcr, set, sh_flag, err)) return false;
  if constexpr (Src::HASHED) return wg_subset_one(src, r, v, dcr, set, sh_flag, err);
  return true;
}

// Persistent: grid-strides over the verification list (count read on device).
template <class Src>
__global__ void __launch_bounds__(256) k_verify(Src src, const int *__restrict__ vcount, const int *__restrict__ vlist,
                                                const u32 *__restrict__ DC, int *__restrict__ rep, int *ccount,
                                                int *clist, u32 *err) {
  __shared__ u64 set[BLOCK_SLOTS];
  __shared__ int sh_flag[2];
  const int total = *vcount;
  for (int item = blockIdx.x; item < total; item += gridDim.x) {
    const int v = vlist[item];
    const int r = rep[v];
    const bool ok = wg_subset(src, v, r, DC[r], set, sh_flag, err);
    if (threadIdx.x == 0 && !ok) {
      rep[v] = -1;
      const int at = atomicAdd(ccount, 1);
      clist[at] = v;
    }
    __syncthreads();
  }
}

// ---------------------------------------------------------------- collision peeling
// One peeling round over a list of collided vertices: insert (hash, v) into a
// second table (minimum vertex per hash), then check every vertex exactly
// against that minimum.  The minimum itself heads its block; matches join it;
// the rest go to the next round's list.  Every round settles at least one
// block per hash value, so rounds end.
__global__ void k_res_insert(const int *__restrict__ count, const int *__restrict__ list, const u64 *__restrict__ H,
                             u64 *ctable, u64 tmask, const u32 *__restrict__ dep) {
  const u32 epoch = dep[EP_CTABLE];
  const int total = *count;
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < total; i += gridDim.x * blockDim.x) {
    const int v = list[i];
    table_insert(ctable, tmask, H[v], (u32)v, epoch);
  }
}

template <class Src>
__global__ void __launch_bounds__(256) k_res_verify(Src src, const int *__restrict__ count, const int *__restrict__ list,
                                                    const u64 *__restrict__ H, const u32 *__restrict__ DC,
                                                    const u64 *ctable, u64 tmask, const u32 *__restrict__ dep,
                                                    int *__restrict__ rep, int *next_count, int *next_list, u32 *err) {
  const u32 epoch = dep[EP_CTABLE];
  __shared__ u64 set[BLOCK_SLOTS];
  __shared__ int sh_flag[2];
  const int total = *count;
  for (int item = blockIdx.x; item < total; item += gridDim.x) {
    const int v = list[item];
    const int r = table_lookup(ctable, tmask, H[v], epoch);
    bool ok;
    if (r < 0) {
      if (threadIdx.x == 0) atomicOr(err, ERR_LOOKUP_MISS);
      ok = true;  // leave v as its own block; the error is reported
    } else if (r == v) {
      ok = true;
    } else if (src.own(v) != src.own(r) || DC[v] != DC[r]) {
      ok = false;
    } else if (DC[v] == 0) {
      ok = true;
    } else {
      ok = wg_subset(src, v, r, DC[r], set, sh_flag, err);
    }
    if (threadIdx.x == 0) {
      if (ok) {
        rep[v] = r < 0 ? v : r;
      } else {
        const int at = atomicAdd(next_count, 1);
        next_list[at] = v;
      }
    }
    __syncthreads();
  }
}

// The one peeling round inside a step, by one workgroup: tags and home slots of
// 10^8 exact keys leave a handful of collided vertices; 32-bit hashes of pairs
// some hundred to a few thousand on the largest graphs.  The vertices of one hash
// meet in an LDS table that keeps the smallest; then a thread each compares rows
// of at most SMALL_MAX entries, and only longer ones go through the workgroup's
// check one after another (all of them that way: ten steps on 40,000 vertices of
// one or two entries, hashes cut to 20 bits, 84.9 ms; now 2.6).  With more than
// PEEL_MAX of them, or some left over, the host redoes the step with k_res_insert
// and k_res_verify rounds over the whole grid, which costs a call on a large graph
// as much again: here they are only counted.
constexpr int PEEL_MAX = 4096;
static_assert(2 * PEEL_MAX <= BLOCK_SLOTS && PEEL_MAX <= 65536, "slots for twice the hashes, 16-bit places");
template <class Src>
__global__ void __launch_bounds__(256) k_peel_few(Src src, const int *__restrict__ count, const int *__restrict__ list,
                                                  const u64 *__restrict__ H, const u32 *__restrict__ DC,
                                                  int *__restrict__ rep, int *next_count, u32 *err) {
  const int total = *count;
  if (total == 0) return;
  if (total > PEEL_MAX) {
    if (threadIdx.x == 0) *next_count = total;
    return;
  }
  __shared__ u64 set[BLOCK_SLOTS];
  __shared__ u32 mins[BLOCK_SLOTS];
  __shared__ int vs[PEEL_MAX];
  __shared__ unsigned short at[PEEL_MAX];     // slot of the vertex's hash
  __shared__ unsigned short longs[PEEL_MAX];  // places of the vertices whose rows are too long for a thread
  __shared__ int sh_flag[2];
  __shared__ int sh_long, sh_left;
  for (int i = threadIdx.x; i < BLOCK_SLOTS; i += 256) {
    set[i] = EMPTY64;
    mins[i] = 0xFFFFFFFFu;
  }
  if (threadIdx.x == 0) sh_long = sh_left = 0;
  __syncthreads();
  for (int i = threadIdx.x; i < total; i += 256) {
    const int v = list[i];
    const u64 h = sink_form(H[v]);
    u32 s = ((u32)h ^ (u32)(h >> 32)) * 0x9E3779B1u >> 19;  // 13 bits: BLOCK_SLOTS
    while (true) {
      const u64 old = atomicCAS(&set[s], EMPTY64, h);
      if (old == EMPTY64 || old == h) break;
      s = (s + 1) & (BLOCK_SLOTS - 1);
    }
    atomicMin(&mins[s], (u32)v);
    vs[i] = v;
    at[i] = (unsigned short)s;
  }
  __syncthreads();
  for (int i = threadIdx.x; i < total; i += 256) {
    const int v = vs[i], r = (int)mins[at[i]];
    int eq = 1;
    if (r != v) {
      if (src.own(v) != src.own(r) || DC[v] != DC[r]) eq = 0;
      else if (DC[v] != 0) eq = same_small_rows(src, v, r);
    }
    if (eq > 0) rep[v] = r;
    else if (eq == 0) atomicAdd(&sh_left, 1);
    else longs[atomicAdd(&sh_long, 1)] = (unsigned short)i;
  }
  __syncthreads();
  const int nlong = sh_long;
  for (int i = 0; i < nlong; ++i) {
    const int v = vs[longs[i]], r = (int)mins[at[longs[i]]];
    const bool ok = wg_subset(src, v, r, DC[r], set, sh_flag, err);
    if (threadIdx.x == 0) {
      if (ok) rep[v] = r;
      else ++sh_left;
    }
  }
  __syncthreads();
  if (threadIdx.x == 0) *next_count = sh_left;
}

// ---------------------------------------------------------------- numbering
// Flags "rep[v] == v" in vertex order (tiles of 256 * ITEMS vertices, ITEMS =
// 8 or 16 per thread).  A head's exclusive prefix is its dense id, so blocks
// are numbered by their first vertex.
template <int ITEMS>
__device__ inline u32 tile_flags(int n, const int *__restrict__ rep, int64_t base) {
  int r[ITEMS];
  if (base + ITEMS <= n) {
    const int4 *p4 = reinterpret_cast<const int4 *>(rep + base);
#pragma unroll
    for (int q = 0; q < ITEMS / 4; ++q) {
      const int4 x = p4[q];
      r[4 * q] = x.x;
      r[4 * q + 1] = x.y;
      r[4 * q + 2] = x.z;
      r[4 * q + 3] = x.w;
    }
  } else {
#pragma unroll
    for (int j = 0; j < ITEMS; ++j) r[j] = (base + j < n) ? rep[base + j] : -1;
  }
  u32 bits = 0;
#pragma unroll
  for (int j = 0; j < ITEMS; ++j)
    if (r[j] == (int)(base + j)) bits |= 1u << j;
  return bits;
}


// One workgroup of 1024 threads: in-place exclusive scan of ntiles counts.
__global__ void __launch_bounds__(1024) k_tile_scan(int ntiles, u32 *tile_sum, int64_t *count_out) {
  __shared__ u32 sh_w[16];
  __shared__ u32 carry;
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  if (t == 0) carry = 0;
  __syncthreads();
  for (int b0 = 0; b0 < ntiles; b0 += 1024 * 8) {
    u32 v8[8];
    u32 sum = 0;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const int i = b0 + t * 8 + k;
      v8[k] = i < ntiles ? tile_sum[i] : 0u;
      sum += v8[k];
    }
    u32 x = sum;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const u32 y = __shfl_up(x, o, WAVE);
      if (lane >= o) x += y;
    }
    if (lane == 63) sh_w[w] = x;
    __syncthreads();
    u32 off = carry + x - sum;
    for (int i = 0; i < w; ++i) off += sh_w[i];
    u32 all = 0;
    for (int i = 0; i < 16; ++i) all += sh_w[i];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const int i = b0 + t * 8 + k;
      if (i < ntiles) tile_sum[i] = off;
      off += v8[k];
    }
    __syncthreads();
    if (t == 0) carry += all;
    __syncthreads();
  }
  if (t == 0) *count_out = (int64_t)carry;
}

// Head words: the numbering of a step without the scattered write of every
// head's id.  Word w holds one bit per vertex 64w..64w+63 (set for a head,
// rep[v] == v) and the number of heads before the word in its tile (the
// tile counts go to tile_sum for k_tile_scan).  A vertex then reads its dense
// id from its representative's word: tile prefix + word prefix + heads below
// it in the word.  The words (n / 4 bytes) and tile prefixes stay in the
// caches, unlike a gather of every representative's id from the output.
struct HeadWord {
  u64 bits;
  u32 pre;
  u32 pad;
};
struct HeadIds {
  const HeadWord *hw;
  const u32 *tile_pre;  // exclusive prefix of head counts per tile
  int tile_shift;       // log2 of the tile's vertex count
};
__device__ inline int head_id(const HeadIds &h, int r) {
  const u32x4 q = *reinterpret_cast<const u32x4 *>(&h.hw[r >> 6]);
  const u64 bits = (u64)q.x | ((u64)q.y << 32);
  const u64 below = bits & ((1ull << (r & 63)) - 1ull);
  return (int)(h.tile_pre[r >> h.tile_shift] + q.z + (u32)__popcll(below));
}

template <int ITEMS>
__global__ void __launch_bounds__(256) k_head_words(int n, const int *__restrict__ rep, HeadWord *__restrict__ hw,
                                                    u32 *__restrict__ tile_sum) {
  static_assert(64 % ITEMS == 0, "a word spans whole threads");
  constexpr int TPW = 64 / ITEMS;  // threads per word (consecutive lanes of one wave)
  __shared__ u32 sh_w[4];
  const int64_t base = (int64_t)blockIdx.x * (256 * ITEMS) + (int64_t)threadIdx.x * ITEMS;
  const u32 bits = tile_flags<ITEMS>(n, rep, base);
  u32 total;
  const u32 pre = block_exclusive_scan(__popc(bits), sh_w, &total);
  u64 word = 0;
#pragma unroll
  for (int q = 0; q < TPW; ++q) word |= (u64)__shfl_down(bits, q, WAVE) << (q * ITEMS);
  if ((threadIdx.x % TPW) == 0 && base < n)
    *reinterpret_cast<u32x4 *>(&hw[base >> 6]) = u32x4{(u32)word, (u32)(word >> 32), pre, 0u};
  if (threadIdx.x == 0) tile_sum[blockIdx.x] = total;
}

// Every vertex takes its representative's dense id (head words), and the
// new partition is also written in rank order for the next gather (vertices
// no entry names have rank -1 and are left out).
// Work-efficient mode (multi != NULL): every non-head marks its head with the
// step's stamp, so a head left unmarked is a singleton block (k_singletons).
// ASSIGN_V consecutive vertices per thread: representatives, ranks and ids
// move 16 bytes at a time where the arrays' starts allow.
// SCAN (at most 256 tiles): the tile counts are still to be scanned, which
// every workgroup does for itself (one launch less; with more tiles the loads
// of every workgroup would cost more than it); the total goes to *count_out.
// LOCAL (batches): the ids inside each graph are written as well.  A graph's
// first vertex heads its block, so the graph's first id is one more read of
// the head words; a kernel of its own read every id and graph again (1024
// graphs, 57M vertices: 306 -> 273 us a step).
constexpr int ASSIGN_V = 4;
struct LocalIds {
  const int *gid;        // graph of every vertex
  const int64_t *first;  // first vertex of every graph
  int *out;
};
template <bool SCAN, bool LOCAL>
__global__ void __launch_bounds__(256) k_assign(int n, const int *__restrict__ rep, HeadIds ids,
                                                int *__restrict__ out, const int *__restrict__ rank,
                                                int *__restrict__ gpid_next, u32 *multi,
                                                const u32 *__restrict__ dep, int ntiles, int64_t *count_out,
                                                LocalIds loc) {
  __shared__ u32 tp[SCAN ? 256 : 1];
  if constexpr (SCAN) {
    __shared__ u32 sh_w[4];
    u32 total;
    const u32 mine = (int)threadIdx.x < ntiles ? ids.tile_pre[threadIdx.x] : 0u;
    tp[threadIdx.x] = block_exclusive_scan(mine, sh_w, &total);
    if (blockIdx.x == 0 && threadIdx.x == 0) *count_out = (int64_t)total;
    __syncthreads();
    ids.tile_pre = tp;
  }
  const int64_t v0 = ((int64_t)blockIdx.x * 256 + threadIdx.x) * ASSIGN_V;
  if (v0 >= n) return;
  const bool vec = v0 + ASSIGN_V <= n && ((reinterpret_cast<uintptr_t>(rep) | reinterpret_cast<uintptr_t>(out) |
                                           reinterpret_cast<uintptr_t>(rank)) & 15) == 0;
  int r[ASSIGN_V], rk[ASSIGN_V], val[ASSIGN_V];
  if (vec) {
    const int4 r4 = *reinterpret_cast<const int4 *>(rep + v0);
    r[0] = r4.x; r[1] = r4.y; r[2] = r4.z; r[3] = r4.w;
    if (rank) {
      const int4 k4 = *reinterpret_cast<const int4 *>(rank + v0);
      rk[0] = k4.x; rk[1] = k4.y; rk[2] = k4.z; rk[3] = k4.w;
    }
  } else {
#pragma unroll
    for (int j = 0; j < ASSIGN_V; ++j) {
      r[j] = v0 + j < n ? rep[v0 + j] : -1;
      if (rank) rk[j] = v0 + j < n ? rank[v0 + j] : -1;
    }
  }
#pragma unroll
  for (int j = 0; j < ASSIGN_V; ++j) val[j] = r[j] >= 0 ? head_id(ids, r[j]) : -1;
  if (vec) {
    *reinterpret_cast<int4 *>(out + v0) = make_int4(val[0], val[1], val[2], val[3]);
  } else {
#pragma unroll
    for (int j = 0; j < ASSIGN_V; ++j)
      if (v0 + j < n) out[v0 + j] = val[j];
  }
  if constexpr (LOCAL) {
    int g[ASSIGN_V], id[ASSIGN_V];
    if (vec && (reinterpret_cast<uintptr_t>(loc.gid) & 15) == 0) {
      const int4 g4 = *reinterpret_cast<const int4 *>(loc.gid + v0);
      g[0] = g4.x; g[1] = g4.y; g[2] = g4.z; g[3] = g4.w;
    } else {
#pragma unroll
      for (int j = 0; j < ASSIGN_V; ++j) g[j] = loc.gid[v0 + j < n ? v0 + j : v0];
    }
    int base = head_id(ids, (int)loc.first[g[0]]);
#pragma unroll
    for (int j = 0; j < ASSIGN_V; ++j) {
      if (j && g[j] != g[j - 1]) base = head_id(ids, (int)loc.first[g[j]]);
      id[j] = val[j] - base;
    }
    if (vec && (reinterpret_cast<uintptr_t>(loc.out) & 15) == 0) {
      *reinterpret_cast<int4 *>(loc.out + v0) = make_int4(id[0], id[1], id[2], id[3]);
    } else {
#pragma unroll
      for (int j = 0; j < ASSIGN_V; ++j)
        if (v0 + j < n) loc.out[v0 + j] = id[j];
    }
  }
#pragma unroll
  for (int j = 0; j < ASSIGN_V; ++j) {
    if (v0 + j >= n) break;
    if (multi && r[j] >= 0 && r[j] != (int)(v0 + j)) multi[r[j]] = dep[EP_ZERO];
    if (rank && rk[j] >= 0) gpid_next[rk[j]] = val[j];
  }
}

// single[v] = 1 iff v is alone in its block of the partition just computed.
// A singleton block never splits, so the next step can skip its vertex.
__global__ void k_singletons(int n, const int *__restrict__ rep, const u32 *__restrict__ multi,
                             const u32 *__restrict__ dep, unsigned char *single) {
  const int v = blockIdx.x * blockDim.x + threadIdx.x;
  if (v >= n) return;
  single[v] = (rep[v] == v && multi[v] != dep[EP_ZERO]) ? 1 : 0;
}

// In-degree histogram, target renumbering and rank-order scatter (create time
// and the start of each call).
// ---------------------------------------------------------------- transpose
// Backward refinement is forward refinement of the transposed graph
// (Def. inverse-schema-element).  Transpose = count entries per target,
// exclusive scan into row offsets, scatter each entry (v, l, w) to row w.

// Exclusive scan of 64-bit values over a 256-thread workgroup.
__device__ inline int64_t block_exclusive_scan64(int64_t mine, int64_t *sh_w, int64_t *total) {
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  int64_t x = mine;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int64_t y = __shfl_up(x, o, WAVE);
    if (lane >= o) x += y;
  }
  if (lane == 63) sh_w[w] = x;
  __syncthreads();
  int64_t base = 0;
  for (int i = 0; i < w; ++i) base += sh_w[i];
  *total = sh_w[0] + sh_w[1] + sh_w[2] + sh_w[3];
  __syncthreads();
  return base + x - mine;
}

// The SCAN_ITEMS counts from base on (zeros past n), 16 bytes per load where
// the array allows.
__device__ inline void scan_items(int64_t n, const int *__restrict__ cnt, int64_t base, int (&c)[SCAN_ITEMS]) {
  if (base + SCAN_ITEMS <= n && (reinterpret_cast<uintptr_t>(cnt) & 15) == 0) {
    const int4 *p4 = reinterpret_cast<const int4 *>(cnt + base);
#pragma unroll
    for (int q = 0; q < SCAN_ITEMS / 4; ++q) {
      const int4 x = p4[q];
      c[4 * q] = x.x;
      c[4 * q + 1] = x.y;
      c[4 * q + 2] = x.z;
      c[4 * q + 3] = x.w;
    }
  } else {
#pragma unroll
    for (int j = 0; j < SCAN_ITEMS; ++j) c[j] = base + j < n ? cnt[base + j] : 0;
  }
}

__global__ void __launch_bounds__(256) k_sum_tiles64(int64_t n, const int *__restrict__ cnt, int64_t *tile_sum) {
  __shared__ int64_t sh_w[4];
  const int64_t base = (int64_t)blockIdx.x * SCAN_TILE + (int64_t)threadIdx.x * SCAN_ITEMS;
  int c[SCAN_ITEMS];
  scan_items(n, cnt, base, c);
  int64_t mine = 0;
#pragma unroll
  for (int j = 0; j < SCAN_ITEMS; ++j) mine += c[j];
  int64_t total;
  block_exclusive_scan64(mine, sh_w, &total);
  if (threadIdx.x == 0) tile_sum[blockIdx.x] = total;
}

// One workgroup of 256 threads: in-place exclusive scan of ntiles sums.
__global__ void __launch_bounds__(256) k_scan_tiles64(int64_t ntiles, int64_t *tile_sum) {
  __shared__ int64_t sh_w[4];
  __shared__ int64_t carry;
  if (threadIdx.x == 0) carry = 0;
  __syncthreads();
  constexpr int PER = 8;  // consecutive sums per thread and round
  for (int64_t b0 = 0; b0 < ntiles; b0 += 256 * PER) {
    const int64_t i0 = b0 + (int64_t)threadIdx.x * PER;
    int64_t c[PER];
    int64_t mine = 0;
#pragma unroll
    for (int j = 0; j < PER; ++j) {
      c[j] = i0 + j < ntiles ? tile_sum[i0 + j] : 0;
      mine += c[j];
    }
    int64_t total;
    int64_t at = carry + block_exclusive_scan64(mine, sh_w, &total);
#pragma unroll
    for (int j = 0; j < PER; ++j) {
      if (i0 + j < ntiles) tile_sum[i0 + j] = at;
      at += c[j];
    }
    __syncthreads();
    if (threadIdx.x == 0) carry += total;
    __syncthreads();
  }
}

// out_ptr[i] = sum of cnt[0..i), out_ptr[n] = total; cursor[i] = out_ptr[i] (cursor may be NULL).
// SUMS (at most 256 tiles): tile_pre holds the tile sums, which every workgroup
// adds up to its own tile, instead of a launch that scans them.
template <bool SUMS>
__global__ void __launch_bounds__(256) k_write_ptr64(int64_t n, const int *__restrict__ cnt,
                                                     const int64_t *__restrict__ tile_pre, int64_t *out_ptr,
                                                     unsigned long long *cursor) {
  __shared__ int64_t sh_w[4];
  const int64_t base = (int64_t)blockIdx.x * SCAN_TILE + (int64_t)threadIdx.x * SCAN_ITEMS;
  int c[SCAN_ITEMS];
  scan_items(n, cnt, base, c);
  int64_t mine = 0;
#pragma unroll
  for (int j = 0; j < SCAN_ITEMS; ++j) mine += c[j];
  int64_t total, before;
  if constexpr (SUMS) block_exclusive_scan64(threadIdx.x < blockIdx.x ? tile_pre[threadIdx.x] : 0, sh_w, &before);
  else before = tile_pre[blockIdx.x];
  int64_t off = before + block_exclusive_scan64(mine, sh_w, &total);
  const bool vec = base + SCAN_ITEMS < n && ((reinterpret_cast<uintptr_t>(out_ptr) |
                                              reinterpret_cast<uintptr_t>(cursor)) & 15) == 0;
  if (vec) {
#pragma unroll
    for (int j = 0; j < SCAN_ITEMS; j += 2) {
      const longlong2 two = make_longlong2(off, off + c[j]);
      reinterpret_cast<longlong2 *>(out_ptr + base)[j / 2] = two;
      if (cursor) reinterpret_cast<longlong2 *>(cursor + base)[j / 2] = two;
      off += c[j] + (int64_t)c[j + 1];
    }
    return;
  }
#pragma unroll
  for (int j = 0; j < SCAN_ITEMS; ++j) {
    if (base + j < n) {
      out_ptr[base + j] = off;
      if (cursor) cursor[base + j] = (unsigned long long)off;
    }
    off += c[j];
    if (base + j + 1 == n) out_ptr[n] = off;
  }
}

// One wave per source row: every entry (v, l, w) takes the next free
// position of row w.  The order inside a transposed row depends on timing;
// signatures are sets, so refinement results do not.
__global__ void __launch_bounds__(256) k_transpose_scatter(int64_t n, const int64_t *__restrict__ row_ptr,
                                                           const int32_t *__restrict__ col,
                                                           const int32_t *__restrict__ elabel,
                                                           unsigned long long *cursor, int32_t *out_col,
                                                           int32_t *out_elabel) {
  const int lane = threadIdx.x & (WAVE - 1);
  const int64_t waves = ((int64_t)gridDim.x * blockDim.x) >> 6;
  for (int64_t v = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6; v < n; v += waves) {
    const int64_t b = row_ptr[v], e = row_ptr[v + 1];
    for (int64_t i = b + lane; i < e; i += WAVE) {
      const unsigned long long pos = atomicAdd(&cursor[col[i]], 1ULL);
      out_col[pos] = (int32_t)v;
      if (out_elabel) out_elabel[pos] = elabel ? elabel[i] : 0;
    }
  }
}

// Entries per target.  A workgroup counts a chunk of INDEG_CHUNK entries in
// an LDS table (target -> count), then adds one device atomic per distinct
// target, so the many entries of a hot target do not serialise on one
// address across the device.  indeg starts at zero; 256 threads.
constexpr int INDEG_CHUNK = 2048, INDEG_SLOTS = 4096;
__global__ void __launch_bounds__(256) k_indegree(int64_t m, const int *__restrict__ col, int *indeg) {
  __shared__ int key[INDEG_SLOTS];
  __shared__ int val[INDEG_SLOTS];
  for (int64_t base = (int64_t)blockIdx.x * INDEG_CHUNK; base < m; base += (int64_t)gridDim.x * INDEG_CHUNK) {
    for (int i = threadIdx.x; i < INDEG_SLOTS; i += 256) {
      key[i] = -1;
      val[i] = 0;
    }
    __syncthreads();
    const int cnt = (int)min<int64_t>(m - base, INDEG_CHUNK);
    for (int i = threadIdx.x; i < cnt; i += 256) {
      const int c = col[base + i];
      u32 sl = ((u32)c * 0x9E3779B1u) >> 20;  // 12 bits: INDEG_SLOTS
      while (true) {
        const int old = atomicCAS(&key[sl], -1, c);
        if (old == -1 || old == c) {
          atomicAdd(&val[sl], 1);
          break;
        }
        sl = (sl + 1) & (INDEG_SLOTS - 1);
      }
    }
    __syncthreads();
    for (int i = threadIdx.x; i < INDEG_SLOTS; i += 256)
      if (key[i] >= 0) atomicAdd(&indeg[key[i]], val[i]);
    __syncthreads();
  }
}
// gcol[e] = rank[col[e]], with the entry's label in the bits above rbits
// when elabel is given (packed form).
__global__ void k_remap(int64_t m, const int *__restrict__ col, const int *__restrict__ rank, int *__restrict__ gcol,
                        const int *__restrict__ elabel, u32 rbits) {
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < m; e += (int64_t)gridDim.x * blockDim.x) {
    u32 g = (u32)rank[col[e]];
    if (elabel) g |= (u32)elabel[e] << rbits;
    gcol[e] = (int)g;
  }
}
// Order of the entries inside a row.  A signature is a set, so the kernels
// may read a row's entries in any order; with the entries of a row in order of
// their targets' ranks, the lanes of a wave gather from fewer cache lines
// (ranks put the targets of most edges together).  What matters is that the
// hot low ranks meet, so ranks are put into buckets of whole lines on a
// logarithmic scale (8 per octave, at most ORDER_BUCKETS) and rows ordered by
// bucket with a counting sort in LDS, instead of a full sort: the bitonic
// networks that did that took 66 barriers per range, 0.9 ms on a graph of 23M
// entries (now 0.15), and calls are as fast (100M-edge graph 8.73 / 8.78 ms).
constexpr int ORDER_BUCKETS = 256;
__device__ inline u32 order_bucket(u32 rank) {
  const u32 x = (rank >> 5) + 8u;  // lines of 32 ids; the first 8 exactly
  const int e = 28 - __clz(x);     // x in [8, 16) << e
  return ((u32)e << 3) + ((x >> e) & 7u);
}
static_assert((29 - 4) * 8 < ORDER_BUCKETS, "ranks are below 2^31");

// Entries words[0, len) (len <= N) ordered by bucket, by a workgroup of NT
// threads.  PAY: labels[0, len) (separate edge labels) move with their words.
template <int N, int NT, bool PAY>
struct OrderSpace {
  u32 w[N];
  u32 l[PAY ? N : 1];
  u32 at[ORDER_BUCKETS];
  u32 wsum[ORDER_BUCKETS / WAVE];
};
template <int N, int NT, bool PAY>
__device__ inline void order_row(u32 *words, u32 *labels, int len, u32 rbits, OrderSpace<N, NT, PAY> &sp) {
  constexpr int U = N / NT;
  const int t = threadIdx.x;
  const u32 rm = (1u << rbits) - 1u;
  if (t < ORDER_BUCKETS) sp.at[t] = 0;
  u32 w[U], l[U], b[U], pos[U];
#pragma unroll
  for (int j = 0; j < U; ++j) {
    const int i = t + j * NT;
    w[j] = i < len ? words[i] : 0u;
    if constexpr (PAY) l[j] = i < len ? labels[i] : 0u;
    b[j] = order_bucket(w[j] & rm);
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < U; ++j) pos[j] = t + j * NT < len ? atomicAdd(&sp.at[b[j]], 1u) : 0u;
  __syncthreads();
  u32 mine = 0, x = 0;
  if (t < ORDER_BUCKETS) {
    mine = x = sp.at[t];
#pragma unroll
    for (int o = 1; o < WAVE; o <<= 1) {
      const u32 y = __shfl_up(x, o, WAVE);
      if ((t & (WAVE - 1)) >= o) x += y;
    }
    if ((t & (WAVE - 1)) == WAVE - 1) sp.wsum[t / WAVE] = x;
  }
  __syncthreads();
  if (t < ORDER_BUCKETS) {
    u32 base = x - mine;
    for (int i = 0; i < t / WAVE; ++i) base += sp.wsum[i];
    sp.at[t] = base;
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < U; ++j) {
    if (t + j * NT >= len) continue;
    const u32 p = sp.at[b[j]] + pos[j];
    sp.w[p] = w[j];
    if constexpr (PAY) sp.l[p] = l[j];
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < U; ++j) {
    const int i = t + j * NT;
    if (i >= len) continue;
    words[i] = sp.w[i];
    if constexpr (PAY) labels[i] = sp.l[i];
  }
}

static_assert(RANGE_DMAX <= 4096 && ROW_MAX <= 8192 && ROW_MAX_NARROW <= 19 * 1024 && HUB_CHUNK_MAX <= 4096,
              "row order sizes");

// One workgroup of 256 threads per range of at most N entries: every row of
// the range ordered in place.  The range's entries go by bucket first, then
// stably by row: each wave ranks the entries of its share of the bucket order
// by row with ballots (as k_radix_scatter), and a row's places are known from
// its offset.
template <int N, bool PAY>
__global__ void __launch_bounds__(256) k_sort_ranges(u32 *gcol, u32 *labels, const Range *__restrict__ ranges,
                                                     const u32 *__restrict__ nzrow, u32 rbits) {
  constexpr int U = N / 256;
  static_assert(RANGE_VERTS == 256 && ORDER_BUCKETS == 256, "a thread per row and per bucket");
  __shared__ u32 sw[N];
  __shared__ u32 sl[PAY ? N : 1];
  __shared__ unsigned char row[N];   // row of entry i, then of the entry at place i
  __shared__ u32 at[256];
  __shared__ int wcnt[4][256];
  __shared__ u32 sh_w[4];
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  const Range rg = ranges[blockIdx.x];
  const int V = rg.v1 - rg.v0, E = rg.ne;
  const u32 rm = (1u << rbits) - 1u;
  u32 *words = gcol + rg.e0;
  u32 *labs = PAY ? labels + rg.e0 : nullptr;
  const int off = t < V ? (int)(nzrow[rg.v0 + t] - (u32)rg.e0) : E;  // this thread's row starts here
  u32 x[U], l[U];
#pragma unroll
  for (int j = 0; j < U; ++j) {
    const int i = t + j * 256;
    x[j] = i < E ? words[i] : 0u;
    if constexpr (PAY) l[j] = i < E ? labs[i] : 0u;
  }
#pragma unroll
  for (int j = 0; j < U; ++j) row[t + j * 256] = 0;
  at[t] = 0;
#pragma unroll
  for (int q = 0; q < 4; ++q) wcnt[q][t] = 0;
  __syncthreads();
  if (t < V) row[off] = (unsigned char)t;
  __syncthreads();
  // the row of every entry: a max-scan over the row starts
  {
    u32 run = 0;
#pragma unroll
    for (int k = 0; k < U; ++k) run = max(run, (u32)row[t * U + k]);
    u32 y = run;
#pragma unroll
    for (int o = 1; o < WAVE; o <<= 1) {
      const u32 z = __shfl_up(y, o, WAVE);
      if (lane >= o) y = max(y, z);
    }
    if (lane == WAVE - 1) sh_w[w] = y;
    __syncthreads();
    u32 carry = __shfl_up(y, 1, WAVE);
    if (lane == 0) carry = 0;
    for (int i = 0; i < w; ++i) carry = max(carry, sh_w[i]);
#pragma unroll
    for (int k = 0; k < U; ++k) {
      carry = max(carry, (u32)row[t * U + k]);
      row[t * U + k] = (unsigned char)carry;
    }
    __syncthreads();
  }
  // by bucket
  u32 b[U], pos[U], rw[U];
#pragma unroll
  for (int j = 0; j < U; ++j) {
    b[j] = order_bucket(x[j] & rm);
    pos[j] = t + j * 256 < E ? atomicAdd(&at[b[j]], 1u) : 0u;
    rw[j] = row[t + j * 256];
  }
  __syncthreads();
  u32 total;
  const u32 base = block_exclusive_scan(at[t], sh_w, &total);
  at[t] = base;
  __syncthreads();
#pragma unroll
  for (int j = 0; j < U; ++j) {
    if (t + j * 256 >= E) continue;
    const u32 p = at[b[j]] + pos[j];
    sw[p] = x[j];
    row[p] = (unsigned char)rw[j];
    if constexpr (PAY) sl[p] = l[j];
  }
  __syncthreads();
  // then by row
  const u64 lt = (1ULL << lane) - 1ULL;
#pragma unroll
  for (int j = 0; j < U; ++j) {
    const int p = w * (N / 4) + j * WAVE + lane;
    const bool valid = p < E;
    const u32 r = row[p];
    x[j] = sw[p];
    if constexpr (PAY) l[j] = sl[p];
    u64 peers = __ballot(valid);
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const u64 ones = __ballot((r >> q) & 1u);
      peers &= ((r >> q) & 1u) ? ones : ~ones;
    }
    const int below = __popcll(peers & lt);
    const int before = wcnt[w][r];
    __builtin_amdgcn_wave_barrier();
    if (valid && below == 0) wcnt[w][r] = before + __popcll(peers);
    __builtin_amdgcn_wave_barrier();
    pos[j] = (u32)(before + below);
    rw[j] = r;
  }
  __syncthreads();
  {
    int a = off;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int c = wcnt[q][t];
      wcnt[q][t] = a;
      a += c;
    }
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < U; ++j) {
    if (w * (N / 4) + j * WAVE + lane >= E) continue;
    const u32 p = (u32)wcnt[w][rw[j]] + pos[j];
    sw[p] = x[j];
    if constexpr (PAY) sl[p] = l[j];
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < U; ++j) {
    const int i = t + j * 256;
    if (i >= E) continue;
    words[i] = sw[i];
    if constexpr (PAY) labs[i] = sl[i];
  }
}

// One workgroup per single-row range of at most N entries.
template <int N, bool PAY>
__global__ void __launch_bounds__(1024) k_sort_rows(u32 *gcol, u32 *labels, const Range *__restrict__ rows,
                                                    u32 rbits) {
  __shared__ OrderSpace<N, 1024, PAY> sp;
  const Range r = rows[blockIdx.x];
  order_row<N, 1024, PAY>(gcol + r.e0, PAY ? labels + r.e0 : nullptr, r.ne, rbits, sp);
}

// One workgroup per staged hub chunk (entries [b, e) of the hub's row, e - b <= N).
template <int N, bool PAY>
__global__ void __launch_bounds__(1024) k_sort_hub_chunks(u32 *gcol, u32 *labels, const int64_t *__restrict__ row_ptr,
                                                          const int *__restrict__ hubs,
                                                          const HubChunk *__restrict__ chunks, u32 rbits) {
  __shared__ OrderSpace<N, 1024, PAY> sp;
  const HubChunk c = chunks[blockIdx.x];
  const int64_t e0 = row_ptr[hubs[c.hub]] + c.b;
  order_row<N, 1024, PAY>(gcol + e0, PAY ? labels + e0 : nullptr, (int)(c.e - c.b), rbits, sp);
}

// gpid[rank[v]] = pid[v] for every vertex some entry names (rank >= 0).
__global__ void k_scatter_rank(int n, const int *__restrict__ pid, const int *__restrict__ rank, int *__restrict__ gpid) {
  const int v = blockIdx.x * blockDim.x + threadIdx.x;
  if (v >= n) return;
  const int r = rank[v];
  if (r >= 0) gpid[r] = pid[v];
}

// ---------------------------------------------------------------- batches
// A batch is the disjoint union of G graphs (vertex ranges [first[g],
// first[g+1])).  Blocks never span graphs, so each graph's first vertex heads
// a block and its global id is the number of blocks in earlier graphs:
// per-graph ids are global ids minus that base.

// The graph of every vertex (gid), and the check that every CSR entry stays
// inside its row's graph.  Rows being in vertex order, the entries of a graph
// are consecutive too, so vertices and entries are both cut into chunks of
// GRAPH_CHUNK, whatever the sizes of the graphs (the first `vchunks` workgroups
// take vertices, the others entries): the graphs of a chunk's ends come from
// two searches, those between mark their starts, and a max-scan gives every
// item its graph.  A share of the grid per graph left a large graph among
// thousands of small ones to a single workgroup: 40M entries beside 9,000 graphs
// of two vertices took 68 ms to create, now 1.75 (2 graphs of the same entries:
// 1.57).
constexpr int GRAPH_CHUNK = 4096;
__global__ void __launch_bounds__(256) k_graph_ids(int64_t G, int64_t n, int64_t m, u32 vchunks,
                                                   const int64_t *__restrict__ first,
                                                   const int64_t *__restrict__ row_ptr,
                                                   const int32_t *__restrict__ col, int *__restrict__ gid, u32 *err) {
  constexpr int PER = GRAPH_CHUNK / 256;
  __shared__ u32 own[GRAPH_CHUNK];
  __shared__ int64_t ends[2];
  __shared__ u32 wmax[4];
  // (row offsets out of order, which k_validate_rows has reported, cannot be searched)
  if (*err & ERR_GRAPH_ROWPTR) return;
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  const bool entries = blockIdx.x >= vchunks;
  const int64_t c0 = (int64_t)(entries ? blockIdx.x - vchunks : blockIdx.x) * GRAPH_CHUNK;
  const int cnt = (int)min<int64_t>((entries ? m : n) - c0, GRAPH_CHUNK);
  auto start = [&](int64_t g) { return entries ? row_ptr[first[g]] : first[g]; };
  if (w < 2) {
    const int64_t g = wave_last_le(0, G, w == 0 ? c0 : c0 + cnt - 1, start);
    if (lane == 0) ends[w] = g;
  }
  __syncthreads();
  const int g0 = (int)ends[0], more = (int)(ends[1] - ends[0]);
  bool bad = false;
  int c[PER];
  if (entries)
#pragma unroll
    for (int j = 0; j < PER; ++j) {
      const int i = t + j * 256;
      c[j] = __builtin_nontemporal_load(&col[c0 + min(i, cnt - 1)]);
    }
  if (more == 0) {  // one graph
    if (entries) {
      const int v0 = (int)first[g0], v1 = (int)first[g0 + 1];
#pragma unroll
      for (int j = 0; j < PER; ++j) bad |= c[j] < v0 || c[j] >= v1;
    } else {
      for (int i = t; i < cnt; i += 256) gid[c0 + i] = g0;
    }
  } else {
    for (int i = t; i < GRAPH_CHUNK; i += 256) own[i] = 0;
    __syncthreads();
    // of the graphs that start at one position the last is not empty
    for (int i = 1 + t; i <= more; i += 256) atomicMax(&own[start(g0 + i) - c0], (u32)i);
    __syncthreads();
    u32 run = 0;
#pragma unroll
    for (int k = 0; k < PER; ++k) run = max(run, own[t * PER + k]);
    u32 x = run;
#pragma unroll
    for (int o = 1; o < WAVE; o <<= 1) {
      const u32 y = __shfl_up(x, o, WAVE);
      if (lane >= o) x = max(x, y);
    }
    if (lane == WAVE - 1) wmax[w] = x;
    u32 carry = __shfl_up(x, 1, WAVE);
    if (lane == 0) carry = 0;
    __syncthreads();
    for (int i = 0; i < w; ++i) carry = max(carry, wmax[i]);
#pragma unroll
    for (int k = 0; k < PER; ++k) {
      carry = max(carry, own[t * PER + k]);
      own[t * PER + k] = carry;
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < PER; ++j) {
      const int i = min(t + j * 256, cnt - 1);
      const int g = g0 + (int)own[i];
      if (entries) bad |= c[j] < (int)first[g] || c[j] >= (int)first[g + 1];
      else gid[c0 + i] = g;
    }
  }
  if (__ballot(bad) && lane == 0) atomicOr(err, ERR_GRAPH_COL);
}

// counts[g * k + i] for step i; `next[g]` is the first vertex of the next
// non-empty graph after g, or -1 (then the total count closes the range).
__global__ void k_batch_counts(int G, const int64_t *__restrict__ first, const int64_t *__restrict__ next,
                               const int *__restrict__ global_ids, const int64_t *__restrict__ total, int k, int i,
                               int64_t *__restrict__ counts) {
  const int g = blockIdx.x * blockDim.x + threadIdx.x;
  if (g >= G) return;
  int64_t c = 0;
  if (first[g + 1] > first[g]) {
    const int64_t base = global_ids[first[g]];
    const int64_t end = next[g] >= 0 ? (int64_t)global_ids[next[g]] : *total;
    c = end - base;
  }
  counts[(int64_t)g * k + i] = c;
}

// ---------------------------------------------------------------- summary graph
// The summary (quotient) graph of a refinement chain has one vertex per block
// of P_k and an edge (B, l, C) when the members of B have an l-edge into block
// C of P_{k-1} (Sec. "Graph Summaries for Bisimulation": connected when all
// represented vertices have such an edge; members of one P_k block share
// their (label, P_{k-1} block) sets, so "all" and "some" coincide).  Built by
// packing each CSR entry into one 64-bit key (source block, label, target
// block), sorting the keys (LSD radix, 8-bit digits) and keeping the first of
// every run of equal keys.

struct QKey {
  u32 lb, db;  // bits of the label and target-block fields
};

// Keys are built from the context's gather layout: the target's rank (and
// packed or sorted label) per entry, and the target blocks copied into rank
// order, so the per-entry gather runs over the hot-first array of the
// signature kernels.  One workgroup per range of the degree schedule (owner
// of each entry by a max-scan over row starts, as in k_sig_range), one per
// single-row range, and one per hub chunk; consecutive entries give
// consecutive keys.
template <class Src>
__device__ inline u64 quotient_key(const Src &src, const int32_t *__restrict__ tgt, QKey q, u64 sb, int64_t e) {
  u32 l, r;
  src.entry(e, l, r);
  return sb | ((u64)l << q.db) | (u64)(u32)tgt[r];
}

template <class Src, int EMAX>
__global__ void __launch_bounds__(256) k_quotient_range(Src src, const Range *__restrict__ ranges,
                                                        const int *__restrict__ nzv, const u32 *__restrict__ nzrow,
                                                        const int32_t *__restrict__ src_pid,
                                                        const int32_t *__restrict__ tgt, QKey q, u64 *keys) {
  __shared__ int roff[RANGE_VERTS + 1];
  __shared__ unsigned char owner[EMAX];
  __shared__ u64 sbk[RANGE_VERTS];
  __shared__ u32 wmax[4];
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  const Range rg = ranges[blockIdx.x];
  const int V = rg.v1 - rg.v0;
  if (t < V) {
    roff[t] = (int)(nzrow[rg.v0 + t] - (u32)rg.e0);
    sbk[t] = (u64)(u32)src_pid[nzv[rg.v0 + t]] << (q.lb + q.db);
  }
  if (t == 0) roff[V] = rg.ne;
  for (int i = t; i < EMAX; i += 256) owner[i] = 0;
  __syncthreads();
  for (int i = t; i < V; i += 256)
    if (roff[i + 1] > roff[i]) owner[roff[i]] = (unsigned char)i;
  __syncthreads();
  {
    constexpr int PER = EMAX / 256;
    u32 run = 0;
    const int j0 = t * PER;
#pragma unroll
    for (int k = 0; k < PER; ++k) run = max(run, (u32)owner[j0 + k]);
    u32 x = run;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const u32 y = __shfl_up(x, o, WAVE);
      if (lane >= o) x = max(x, y);
    }
    if (lane == 63) wmax[w] = x;
    __syncthreads();
    u32 carry = __shfl_up(x, 1, WAVE);
    if (lane == 0) carry = 0;
    for (int i = 0; i < w; ++i) carry = max(carry, wmax[i]);
#pragma unroll
    for (int k = 0; k < PER; ++k) {
      carry = max(carry, (u32)owner[j0 + k]);
      owner[j0 + k] = (unsigned char)carry;
    }
    __syncthreads();
  }
  for (int j = t; j < rg.ne; j += 256) keys[rg.e0 + j] = quotient_key(src, tgt, q, sbk[owner[j]], rg.e0 + j);
}

// Entry segments of one row each: single-row ranges (v0, e0, ne) ...
template <class Src>
__global__ void __launch_bounds__(256) k_quotient_rows(Src src, const Range *__restrict__ rows,
                                                       const int32_t *__restrict__ src_pid,
                                                       const int32_t *__restrict__ tgt, QKey q, u64 *keys) {
  const Range rw = rows[blockIdx.x];
  const u64 sb = (u64)(u32)src_pid[rw.v0] << (q.lb + q.db);
  for (int j = threadIdx.x; j < rw.ne; j += 256) keys[rw.e0 + j] = quotient_key(src, tgt, q, sb, rw.e0 + j);
}

// ... and hub chunks (entries [b, e) of the hub's row).
template <class Src, class Chunk>
__global__ void __launch_bounds__(256) k_quotient_hubs(Src src, const Chunk *__restrict__ chunks,
                                                       const int *__restrict__ hubs,
                                                       const int32_t *__restrict__ src_pid,
                                                       const int32_t *__restrict__ tgt, QKey q, u64 *keys) {
  const Chunk c = chunks[blockIdx.x];
  const int v = hubs[c.hub];
  const u64 sb = (u64)(u32)src_pid[v] << (q.lb + q.db);
  const int64_t row = src.begin(v);
  for (int64_t e = row + c.b + threadIdx.x; e < row + c.e; e += 256) keys[e] = quotient_key(src, tgt, q, sb, e);
}

// Tiles of 8192 keys: the 32 keys a digit gets on average leave as whole
// lines.  A summary graph of 125M entries (7 passes): 8.5 ms with 8192-key
// tiles against 9.25 with 4096; 16384 leave one workgroup per CU (8.6
// against 7.6 ms, both with the mapping of radix_tile).
constexpr int RADIX_ITEMS = 16;  // keys per thread per tile
constexpr int RADIX_THREADS = 512;
constexpr int RADIX_TILE = RADIX_THREADS * RADIX_ITEMS;
// Digit histogram of each tile: hist[digit * ntiles + tile].
template <class K>
__global__ void __launch_bounds__(RADIX_THREADS) k_radix_hist(int64_t m, const K *__restrict__ keys, int shift, int64_t ntiles,
                                                    int *__restrict__ hist) {
  __shared__ int h[256];
  const int64_t tile = radix_tile(ntiles);
  if (tile >= ntiles) return;
  if (threadIdx.x < 256) h[threadIdx.x] = 0;
  __syncthreads();
  const int64_t base = tile * RADIX_TILE;
  // every key of the thread is requested before the first count
  K kk[RADIX_ITEMS];
#pragma unroll
  for (int j = 0; j < RADIX_ITEMS; ++j) {
    const int64_t i = base + j * RADIX_THREADS + threadIdx.x;
    kk[j] = i < m ? __builtin_nontemporal_load(&keys[i]) : (K)0;
  }
#pragma unroll
  for (int j = 0; j < RADIX_ITEMS; ++j)
    if (base + j * RADIX_THREADS + threadIdx.x < m) atomicAdd(&h[(u32)(kk[j] >> shift) & 255u], 1);
  __syncthreads();
  if (threadIdx.x < 256) hist[(int64_t)threadIdx.x * ntiles + tile] = h[threadIdx.x];
}

// Stable scatter of a tile.  Each wave ranks its own 1024 consecutive keys by
// itself: per 64 keys, the lanes with equal digits are found with one ballot
// per digit bit, and a wave-private count per digit carries on (LDS accesses
// of one wave stay in order, so the loop has no workgroup barrier; ranking
// the tile in chunks of 256 keys took three barriers per chunk).  A scan over
// digits and waves then gives every key its place in the tile, the tile is
// put in digit order in LDS and written out in that order, so the keys of one
// digit leave as one run of consecutive addresses (whole lines).
// Bound by the ranking's LDS round trips and HBM (16 bytes per 64-bit key).
template <class K>
__global__ void __launch_bounds__(RADIX_THREADS) k_radix_scatter(int64_t m, const K *__restrict__ keys, int shift,
                                                       int64_t ntiles, const int64_t *__restrict__ offs,
                                                       K *__restrict__ out) {
  __shared__ K sk[RADIX_TILE];       // the tile in digit order
  __shared__ int64_t gpos[256];      // global position minus tile position of each digit's keys
  __shared__ int wcnt[RADIX_THREADS / WAVE][256];       // per wave: keys of each digit so far, then their first tile position
  __shared__ u32 sh_w[4];
  const int64_t tile = radix_tile(ntiles);
  if (tile >= ntiles) return;
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  const int64_t goff = t < 256 ? offs[(int64_t)t * ntiles + tile] : 0;
  const int64_t tile0 = tile * RADIX_TILE;
  const int cnt = (int)min<int64_t>(m - tile0, RADIX_TILE);
  const u64 lt = (1ULL << lane) - 1ULL;
  // the whole tile is requested at once, so its load latency is paid once
  K kk[RADIX_ITEMS];
  const int i0 = w * (WAVE * RADIX_ITEMS) + lane;
#pragma unroll
  for (int j = 0; j < RADIX_ITEMS; ++j) {
    const int i = i0 + j * WAVE;
    kk[j] = i < cnt ? __builtin_nontemporal_load(&keys[tile0 + i]) : (K)0;
  }
#pragma unroll
  for (int q = 0; q < 256 / WAVE; ++q) wcnt[w][q * WAVE + lane] = 0;
  __builtin_amdgcn_wave_barrier();
  int rank[RADIX_ITEMS];
#pragma unroll
  for (int j = 0; j < RADIX_ITEMS; ++j) {
    const bool valid = i0 + j * WAVE < cnt;
    const u32 d = (u32)(kk[j] >> shift) & 255u;
    u64 peers = __ballot(valid);
#pragma unroll
    for (int b = 0; b < 8; ++b) {
      const u64 ones = __ballot((d >> b) & 1u);
      peers &= ((d >> b) & 1u) ? ones : ~ones;
    }
    const int below = __popcll(peers & lt);
    const int before = wcnt[w][d];
    __builtin_amdgcn_wave_barrier();
    if (valid && below == 0) wcnt[w][d] = before + __popcll(peers);
    __builtin_amdgcn_wave_barrier();
    rank[j] = before + below;
  }
  __syncthreads();
  // exclusive scan over digits (thread t: digit t), then over the waves of a digit
  {
    u32 c = 0;
    if (t < 256)
#pragma unroll
      for (int q = 0; q < RADIX_THREADS / WAVE; ++q) c += (u32)wcnt[q][t];
    u32 x = c;
#pragma unroll
    for (int o = 1; o < WAVE; o <<= 1) {
      const u32 y = __shfl_up(x, o, WAVE);
      if (lane >= o) x += y;
    }
    if (t < 256 && lane == WAVE - 1) sh_w[w] = x;
    __syncthreads();
    if (t < 256) {
      int at = (int)(x - c);
      for (int i = 0; i < w; ++i) at += (int)sh_w[i];
      gpos[t] = goff - at;
#pragma unroll
      for (int q = 0; q < RADIX_THREADS / WAVE; ++q) {
        const int n = wcnt[q][t];
        wcnt[q][t] = at;
        at += n;
      }
    }
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < RADIX_ITEMS; ++j)
    if (i0 + j * WAVE < cnt) sk[wcnt[w][(u32)(kk[j] >> shift) & 255u] + rank[j]] = kk[j];
  __syncthreads();
#pragma unroll
  for (int j = 0; j < RADIX_ITEMS; ++j) {
    const int i = j * RADIX_THREADS + t;
    if (i < cnt) {
      const K key = sk[i];
      out[gpos[(u32)(key >> shift) & 255u] + i] = key;
    }
  }
}

// ---------------------------------------------------------------- in-degrees by partition
// Entries per target without an atomic per entry (device-wide atomics reach
// about 25 G/s here): targets are first partitioned by their high bits (one
// or two radix passes), so that a bucket's counters fit one workgroup's LDS;
// then one workgroup counts each bucket and writes its counters whole.
// First i in [0, m) with keys[i] >> shift >= b (m if none), for keys in bucket
// order; the whole wave searches.
__device__ inline int64_t wave_bucket_start(const u32 *__restrict__ keys, int64_t m, u32 shift, u32 b) {
  const int lane = threadIdx.x & (WAVE - 1);
  int64_t lo = -1, hi = m;  // keys[lo] is below the bucket, keys[hi] is not
  while (hi - lo > 1) {
    const int64_t step = (hi - lo + WAVE - 1) / WAVE;
    const int64_t at = lo + lane * step;
    const int below = __popcll(__ballot(lane == 0 || (at < hi && (keys[at] >> shift) < b)));
    lo += (below - 1) * step;
    hi = min(hi, lo + step);
  }
  return hi;
}

constexpr int BUCKET_THREADS = 1024;
// Counters of bucket b (targets [b << shift, (b + 1) << shift), shift <= WB)
// from its first `cap` entries; a bucket with more sets *rest, and the starts
// are kept for k_indegree_rest.
template <int WB>
__global__ void __launch_bounds__(BUCKET_THREADS) k_bucket_count(int64_t m, int64_t n, const u32 *__restrict__ keys,
                                                                 u32 shift, int64_t cap, int *__restrict__ indeg,
                                                                 int64_t *__restrict__ starts, int *rest) {
  __shared__ int cnt[1 << WB];
  __shared__ int64_t range[2];
  const int w = threadIdx.x >> 6;
  const u32 b = blockIdx.x, width = 1u << shift;
  for (u32 i = threadIdx.x; i < width; i += BUCKET_THREADS) cnt[i] = 0;
  if (w < 2) {
    const int64_t at = wave_bucket_start(keys, m, shift, b + w);
    if ((threadIdx.x & (WAVE - 1)) == 0) range[w] = at;
  }
  __syncthreads();
  const int64_t i0 = range[0], i1 = min(range[1], i0 + cap);
  if (threadIdx.x == 0) {
    starts[b] = i0;
    if (range[1] > i1) *rest = 1;
  }
  constexpr int U = 8;  // entries in flight per thread
  int64_t i = i0 + threadIdx.x;
  for (; i + (U - 1) * BUCKET_THREADS < i1; i += U * BUCKET_THREADS) {
    u32 k[U];
#pragma unroll
    for (int u = 0; u < U; ++u) k[u] = __builtin_nontemporal_load(&keys[i + u * BUCKET_THREADS]);
#pragma unroll
    for (int u = 0; u < U; ++u) atomicAdd(&cnt[k[u] & (width - 1u)], 1);
  }
  for (; i < i1; i += BUCKET_THREADS) atomicAdd(&cnt[keys[i] & (width - 1u)], 1);
  __syncthreads();
  const int64_t v0 = (int64_t)b << shift;
  for (u32 j = threadIdx.x; j < width; j += BUCKET_THREADS)
    if (v0 + j < n) indeg[v0 + j] = cnt[j];
}

// The entries past the first `cap` of their bucket (graphs where a few targets
// take most entries): chunks counted in LDS, one device atomic per distinct
// target of a chunk, as k_indegree.  Exits at once when no bucket was that long.
__global__ void __launch_bounds__(256) k_indegree_rest(int64_t m, const u32 *__restrict__ keys, u32 shift, int64_t cap,
                                                       const int64_t *__restrict__ starts,
                                                       const int *__restrict__ rest, int *indeg) {
  if (*rest == 0) return;
  __shared__ int key[INDEG_SLOTS];
  __shared__ int val[INDEG_SLOTS];
  for (int64_t base = (int64_t)blockIdx.x * INDEG_CHUNK; base < m; base += (int64_t)gridDim.x * INDEG_CHUNK) {
    const int cnt = (int)min<int64_t>(m - base, INDEG_CHUNK);
    // a chunk whose last entry is among the first of its bucket can still hold
    // late entries of the bucket before; its first entry's bucket tells
    const bool any = base + cnt > starts[keys[base] >> shift] + cap;
    if (!any) continue;  // uniform in the workgroup
    for (int i = threadIdx.x; i < INDEG_SLOTS; i += 256) {
      key[i] = -1;
      val[i] = 0;
    }
    __syncthreads();
    for (int i = threadIdx.x; i < cnt; i += 256) {
      const u32 c = keys[base + i];
      if (base + i < starts[c >> shift] + cap) continue;
      u32 sl = (c * 0x9E3779B1u) >> 20;  // 12 bits: INDEG_SLOTS
      while (true) {
        const int old = atomicCAS(&key[sl], -1, (int)c);
        if (old == -1 || old == (int)c) {
          atomicAdd(&val[sl], 1);
          break;
        }
        sl = (sl + 1) & (INDEG_SLOTS - 1);
      }
    }
    __syncthreads();
    for (int i = threadIdx.x; i < INDEG_SLOTS; i += 256)
      if (key[i] >= 0) atomicAdd(&indeg[key[i]], val[i]);
    __syncthreads();
  }
}

// ---------------------------------------------------------------- transpose by sorting
// One key per CSR entry: target << (lb + sb) | label << sb | source, so that a
// stable sort by target gives the rows of the transposed graph.  A workgroup
// takes TKEY_CHUNK consecutive entries; their rows come from two searches in
// the row offsets and a max-scan over row-start marks (or, where the chunk
// spans more than TKEY_ROWS rows, most of them empty, a search per entry).
constexpr int TKEY_CHUNK = 2048, TKEY_ROWS = 8192;
__global__ void __launch_bounds__(256) k_transpose_keys(int64_t n, int64_t m, const int64_t *__restrict__ row_ptr,
                                                        const int32_t *__restrict__ col,
                                                        const int32_t *__restrict__ elabel, u32 sb, u32 lb,
                                                        u64 *__restrict__ keys) {
  constexpr int PER = TKEY_CHUNK / 256;
  __shared__ u32 own[TKEY_CHUNK];
  __shared__ int64_t ends[2];
  __shared__ u32 wmax[4];
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  const int64_t e0 = (int64_t)blockIdx.x * TKEY_CHUNK;
  const int cnt = (int)min<int64_t>(m - e0, TKEY_CHUNK);
  for (int i = t; i < TKEY_CHUNK; i += 256) own[i] = 0;
  if (w < 2) {
    const int64_t r = wave_last_le(0, n, w == 0 ? e0 : e0 + cnt - 1, [&](int64_t i) { return row_ptr[i]; });
    if (lane == 0) ends[w] = r;
  }
  __syncthreads();
  const int64_t r0 = ends[0], rows = ends[1] - r0 + 1;
  if (rows <= TKEY_ROWS) {
    // rows that start inside the chunk; of those at one position the last is not empty
    for (int i = 1 + t; i < (int)rows; i += 256) atomicMax(&own[row_ptr[r0 + i] - e0], (u32)i);
    __syncthreads();
    u32 run = 0;
#pragma unroll
    for (int k = 0; k < PER; ++k) run = max(run, own[t * PER + k]);
    u32 x = run;
#pragma unroll
    for (int o = 1; o < WAVE; o <<= 1) {
      const u32 y = __shfl_up(x, o, WAVE);
      if (lane >= o) x = max(x, y);
    }
    if (lane == WAVE - 1) wmax[w] = x;
    u32 carry = __shfl_up(x, 1, WAVE);
    if (lane == 0) carry = 0;
    __syncthreads();
    for (int i = 0; i < w; ++i) carry = max(carry, wmax[i]);
#pragma unroll
    for (int k = 0; k < PER; ++k) {
      carry = max(carry, own[t * PER + k]);
      own[t * PER + k] = carry;
    }
    __syncthreads();
  }
  for (int i = t; i < cnt; i += 256) {
    const int64_t e = e0 + i;
    int64_t r;
    if (rows <= TKEY_ROWS) {
      r = r0 + own[i];
    } else {
      int64_t lo = r0, hi = ends[1] + 1;
      while (hi - lo > 1) {
        const int64_t mid = (lo + hi) >> 1;
        if (row_ptr[mid] <= e) lo = mid;
        else hi = mid;
      }
      r = lo;
    }
    u64 k = (u64)(u32)__builtin_nontemporal_load(&col[e]) << (lb + sb) | (u64)r;
    if (elabel) k |= (u64)(u32)__builtin_nontemporal_load(&elabel[e]) << sb;
    keys[e] = k;
  }
}

// The sorted keys back into (source, label) per entry, and the entries per
// target into cnt (zero on entry, modulo 2^32): the first entry of a target
// subtracts its position and the last one adds its end, two atomics per
// named target instead of one per entry.
__global__ void __launch_bounds__(256) k_transpose_unpack(int64_t m, const u64 *__restrict__ keys, u32 sb, u32 lb,
                                                          int32_t *__restrict__ out_col,
                                                          int32_t *__restrict__ out_elabel, int *cnt) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= m) return;
  const u64 k = keys[i];
  const u64 d = k >> (lb + sb);
  out_col[i] = (int32_t)(k & ((1ull << sb) - 1ull));
  if (out_elabel) out_elabel[i] = (int32_t)((k >> sb) & ((1ull << lb) - 1ull));
  if (i == 0 || (keys[i - 1] >> (lb + sb)) != d) atomicSub(&cnt[d], (int)(u32)i);
  if (i == m - 1 || (keys[i + 1] >> (lb + sb)) != d) atomicAdd(&cnt[d], (int)(u32)(i + 1));
}

// ---------------------------------------------------------------- degree schedule
// Non-empty rows are packed greedily into ranges of consecutive ones: a range
// closes before a row that would overflow it (range_edges entries), after
// RANGE_VERTS rows, before a longer row and at the end of its chunk of
// SCHED_CHUNK_V vertices; longer rows go to the row tiers (up to RANGE_DMAX,
// ROW_MAX and row_max entries) or are hubs.  Empty rows are in no range: where
// most vertices have none (70% on the 1B-edge graph) they would fill ranges
// that carry few entries.  The schedule depends on n and the degrees only.
// One workgroup takes one chunk, twice: the first launch counts per chunk
// (cnt[list * nchunks + chunk], lists: ranges, up to RANGE_DMAX, up to
// ROW_MAX, up to row_max, hubs; sums[i * nchunks + chunk]: vertices and
// entries of rows up to range_edges, of row-tier rows, non-empty rows, rows
// past SMALL_MAX); k_sched_scan turns the counts into offsets; the second
// launch writes the range lists one after another in `ranges`, the hubs in
// `hubs`, and every non-empty row's vertex and the low word of its offset in
// nzv and nzrow (a multi-row Range counts rows there, a single-row one
// vertices).
//
// Where a range that starts at row s would close depends on s alone, so all
// the closing points of a chunk are found in parallel (a binary search over
// the row offsets in LDS) and one thread then only follows them from the
// chunk's start, one LDS read per range.  A thread that walked a chunk row by
// row took 4 ms a launch at any size, and a host copy of the offsets with the
// packing there 1 ns per vertex and a synchronisation.
constexpr int SCHED_CHUNK_V = 16384;
constexpr int SCHED_THREADS = 1024;
constexpr int SCHED_PER = SCHED_CHUNK_V / SCHED_THREADS;

// Totals of a schedule, written by k_sched_scan: rows per list, then the sums.
constexpr int SCHED_TOTALS = 11;

// A graph of one chunk needs no totals of other chunks: one launch does both
// parts and leaves the totals itself (10k vertices: 30 us; the three launches
// took 87).
enum { SCHED_COUNT, SCHED_WRITE, SCHED_SINGLE };
template <int FORM>
__global__ void __launch_bounds__(SCHED_THREADS) k_sched_chunks(const int64_t *__restrict__ ptr, int64_t n,
                                                                int nchunks, int range_edges, int64_t row_max,
                                                                int *__restrict__ cnt, int64_t *__restrict__ sums,
                                                                int64_t *__restrict__ totals,
                                                                Range *__restrict__ ranges, int *__restrict__ hubs,
                                                                int *__restrict__ nzv, u32 *__restrict__ nzrow) {
  static_assert(SCHED_CHUNK_V <= 65536 && SCHED_PER == 16, "16-bit rows, one start bit per row of a thread");
  __shared__ u32 off[SCHED_CHUNK_V];                  // low word of each non-empty row's offset
  __shared__ unsigned short row[SCHED_CHUNK_V];       // its vertex in the chunk
  __shared__ unsigned short close_at[SCHED_CHUNK_V];  // last row of the range that starts at a row
  __shared__ unsigned char kind[SCHED_CHUNK_V];       // its list (0: a range)
  __shared__ unsigned short starts[SCHED_THREADS];    // bit j of word t: row 16 t + j starts a range (or is long)
  __shared__ int wl[SCHED_THREADS / WAVE];
  __shared__ int64_t wsum[6][SCHED_THREADS / WAVE];
  __shared__ int wcnt[5][SCHED_THREADS / WAVE];
  const int t = threadIdx.x, lane = t & 63, w = t >> 6, ci = blockIdx.x;
  const int64_t v0 = (int64_t)ci * SCHED_CHUNK_V;
  const int V = (int)min<int64_t>(n - v0, SCHED_CHUNK_V);
  // this thread's vertices 16 t .. 16 t + 15: degrees, sums, and the non-empty
  // ones of the chunk packed into LDS
  const int r0 = t * SCHED_PER;
  int64_t sm[6] = {0, 0, 0, 0, 0, 0};
  {
    int64_t e[SCHED_PER + 1];
    e[0] = r0 <= V ? ptr[v0 + r0] : 0;
#pragma unroll
    for (int j = 0; j < SCHED_PER; ++j) e[j + 1] = r0 + j < V ? ptr[v0 + r0 + j + 1] : e[j];
#pragma unroll
    for (int j = 0; j < SCHED_PER; ++j) {
      const int64_t d = e[j + 1] - e[j];
      if (r0 + j < V && d <= range_edges) {
        sm[0] += 1;
        sm[1] += d;
      } else if (d > 0 && d <= row_max) {
        sm[2] += 1;
        sm[3] += d;
      }
      sm[4] += d > 0;
      sm[5] += d > SMALL_MAX;
    }
    int x = (int)sm[4];
#pragma unroll
    for (int o = 1; o < WAVE; o <<= 1) {
      const int y = __shfl_up(x, o, WAVE);
      if (lane >= o) x += y;
    }
    if (lane == WAVE - 1) wl[w] = x;
    starts[t] = 0;
    __syncthreads();
    int at = x - (int)sm[4];
    for (int i = 0; i < w; ++i) at += wl[i];
#pragma unroll
    for (int j = 0; j < SCHED_PER; ++j) {
      const int64_t d = e[j + 1] - e[j];
      if (d == 0) continue;
      off[at] = (u32)e[j];
      row[at] = (unsigned short)(r0 + j);
      kind[at] = d <= range_edges ? 0 : d > row_max ? 4 : d > ROW_MAX ? 3 : d > RANGE_DMAX ? 2 : 1;
      ++at;
    }
  }
  int R = 0;  // non-empty rows of the chunk
  for (int i = 0; i < SCHED_THREADS / WAVE; ++i) R += wl[i];
  __syncthreads();
  const u32 chunk_end = (u32)ptr[v0 + V];
  // first long row at or after each row, then where its range closes
  u32 lmask = 0;
#pragma unroll
  for (int j = 0; j < SCHED_PER; ++j) lmask |= (r0 + j < R && kind[r0 + j] != 0 ? 1u : 0u) << j;
  int nl = lmask ? r0 + __ffs(lmask) - 1 : R;
#pragma unroll
  for (int o = 1; o < WAVE; o <<= 1) {
    const int y = __shfl_down(nl, o, WAVE);
    if (lane + o < WAVE) nl = min(nl, y);
  }
  if (lane == 0) wl[w] = nl;
  __syncthreads();
  int next_long = __shfl_down(nl, 1, WAVE);
  if (lane == WAVE - 1) next_long = R;
  for (int i = w + 1; i < SCHED_THREADS / WAVE; ++i) next_long = min(next_long, wl[i]);
  int last = R;  // end (exclusive) of the range of the row after
  // end of row e - 1: the next non-empty row's start (rows between are empty)
  auto end_of = [&](int e) { return e < R ? off[e] : chunk_end; };
#pragma unroll
  for (int j = SCHED_PER - 1; j >= 0; --j) {
    const int s = r0 + j;
    if (s >= R) continue;
    if ((lmask >> j) & 1u) {
      next_long = s;
      close_at[s] = (unsigned short)s;
      last = s;
      continue;
    }
    // largest e <= lim whose rows [s, e) fit (one row that is not long does);
    // low words differ exactly, no long row being among them.  It is no larger
    // than the row after's and mostly a few rows less: looked for from there.
    int lo = s + 1, hi = min(min(s + RANGE_VERTS, next_long), last);
    for (int step = 1; lo < hi; step *= 2) {
      const int at = max(hi - step + 1, lo);
      if (end_of(at) - off[s] <= (u32)range_edges) {
        lo = at;
        break;
      }
      hi = at - 1;
    }
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if (end_of(mid) - off[s] <= (u32)range_edges) lo = mid;
      else hi = mid - 1;
    }
    close_at[s] = (unsigned short)(lo - 1);
    last = lo;
  }
  __syncthreads();
  if (t == 0)
    for (int s = 0; s < R;) {
      starts[s >> 4] |= (unsigned short)(1u << (s & 15));
      s = (int)close_at[s] + 1;
    }
  __syncthreads();
  // lists of this thread's starts
  const u32 st = starts[t];
  int c[5] = {0, 0, 0, 0, 0};
#pragma unroll
  for (int j = 0; j < SCHED_PER; ++j) {
    if (!((st >> j) & 1u)) continue;
    const int list = kind[r0 + j];
#pragma unroll
    for (int l = 0; l < 5; ++l) c[l] += list == l;
  }
  if constexpr (FORM != SCHED_WRITE) {
#pragma unroll
    for (int l = 0; l < 6; ++l) {
      const u32 x = wave_sum_u32(l < 5 ? (u32)c[l < 5 ? l : 0] : 0u);
      const u64 y = wave_sum_u64((u64)sm[l]);
      if (lane == 0) {
        if (l < 5) wcnt[l][w] = (int)x;
        wsum[l][w] = (int64_t)y;
      }
    }
    __syncthreads();
    if (t < 6) {
      int x = 0;
      int64_t y = 0;
      for (int i = 0; i < SCHED_THREADS / WAVE; ++i) {
        if (t < 5) x += wcnt[t][i];
        y += wsum[t][i];
      }
      if constexpr (FORM == SCHED_COUNT) {
        if (t < 5) cnt[(int64_t)t * nchunks + ci] = x;
        sums[(int64_t)t * nchunks + ci] = y;
      } else {
        if (t < 5) totals[t] = x;
        totals[5 + t] = y;
      }
    }
    __syncthreads();  // wcnt is written again below
  }
  if constexpr (FORM != SCHED_COUNT) {
    // exclusive positions inside the chunk, per list
    int at[5];
#pragma unroll
    for (int l = 0; l < 5; ++l) {
      int x = c[l];
#pragma unroll
      for (int o = 1; o < WAVE; o <<= 1) {
        const int y = __shfl_up(x, o, WAVE);
        if (lane >= o) x += y;
      }
      if (lane == WAVE - 1) wcnt[l][w] = x;
      at[l] = x - c[l];
    }
    __syncthreads();
    // the scanned offsets: counts of the lists, sums[4] of the non-empty rows
    int64_t base = 0;
#pragma unroll
    for (int l = 0; l < 5; ++l) {
      int64_t whole = 0;  // rows of the list in all chunks
      for (int i = 0; i < SCHED_THREADS / WAVE; ++i) {
        if (i < w) at[l] += wcnt[l][i];
        whole += wcnt[l][i];
      }
      if constexpr (FORM == SCHED_WRITE) {
        at[l] += cnt[(int64_t)l * nchunks + ci];
        whole = totals[l];
      }
      if (l < 4) {
        at[l] += (int)base;
        base += whole;
      }
    }
    const int z0 = FORM == SCHED_WRITE ? (int)sums[(int64_t)4 * nchunks + ci] : 0;
    for (int i = t; i < R; i += SCHED_THREADS) {
      nzv[z0 + i] = (int)(v0 + row[i]);
      nzrow[z0 + i] = off[i];
    }
#pragma unroll
    for (int j = 0; j < SCHED_PER; ++j) {
      if (!((st >> j) & 1u)) continue;
      const int s = r0 + j, list = kind[s];
      const int v = (int)(v0 + row[s]);
      if (list == 4) {
        hubs[at[4]++] = v;
      } else if (list == 0) {
        const int z = (int)close_at[s] + 1;
        ranges[at[0]++] = Range{z0 + s, z0 + z, (int)(end_of(z) - off[s]), 0, ptr[v]};
      } else {
        const Range one{v, v + 1, (int)(end_of(s + 1) - off[s]), z0 + s, ptr[v]};
        if (list == 3) ranges[at[3]++] = one;
        else if (list == 2) ranges[at[2]++] = one;
        else ranges[at[1]++] = one;
      }
    }
  }
}

// One workgroup, a wave per list: in-place exclusive scan of the list's chunk
// counts and of the non-empty rows (sums[4]), and the totals of all.  (One
// list after another by the whole workgroup: 9.6 us for a single chunk.)
__global__ void __launch_bounds__(SCHED_TOTALS *WAVE) k_sched_scan(int nchunks, int *__restrict__ cnt,
                                                                   int64_t *__restrict__ sums,
                                                                   int64_t *__restrict__ totals) {
  const int l = threadIdx.x >> 6, lane = threadIdx.x & (WAVE - 1);
  int64_t carry = 0;
  for (int b0 = 0; b0 < nchunks; b0 += WAVE) {
    const int i = b0 + lane;
    const int64_t at = (int64_t)(l < 5 ? l : l - 5) * nchunks + i;
    const int64_t mine = i < nchunks ? (l < 5 ? (int64_t)cnt[at] : sums[at]) : 0;
    int64_t x = mine;
#pragma unroll
    for (int o = 1; o < WAVE; o <<= 1) {
      const int64_t y = __shfl_up(x, o, WAVE);
      if (lane >= o) x += y;
    }
    if (i < nchunks) {
      if (l < 5) cnt[at] = (int)(carry + x - mine);
      else if (l == 9) sums[at] = carry + x - mine;
    }
    carry += __shfl(x, WAVE - 1, WAVE);
  }
  if (lane == 0) totals[l] = carry;
}

// x on a logarithmic scale: 0 .. 15 exactly, then 8 classes an octave.
__device__ inline u32 log_class(u32 x) {
  const u32 y = max(x, 8u);
  const int e = 28 - __clz(y);  // y in [8, 16) << e
  return x < 8u ? x : ((u32)(e + 1) << 3) + ((y >> e) & 7u);
}

// In-degree ranking: key[v] = (RANK_CLASSES - 1 - class of v's in-degree) << 32
// | v; a stable sort on the high field orders vertices by decreasing class,
// ties by vertex id.  What the gathers need is that the few hot targets share
// lines, for which 8 classes an octave do as well as the in-degrees
// themselves, and their 8 bits are one pass of the sort instead of three (20
// bits): a call on 10k vertices 646 -> 596 us, on a batch of 64 small graphs
// 1.48 -> 1.35 ms, with refinement steps as fast (100M entries 8.77 / 8.75 ms).
constexpr int RANK_KEYBITS = 8;
constexpr u32 RANK_CLASSES = 1u << RANK_KEYBITS;
static_assert((28 + 1 + 1) * 8 <= RANK_CLASSES, "classes of a 31-bit in-degree");

__global__ void k_rank_keys(int64_t n, const int *__restrict__ indeg, u64 *keys) {
  for (int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; v < n; v += (int64_t)gridDim.x * blockDim.x)
    keys[v] = ((u64)(RANK_CLASSES - 1 - log_class((u32)indeg[v])) << 32) | (u64)v;
}

// Keys (graph of the vertex << 32 | vertex) in the order of `sorted`, for a
// stable sort by graph that keeps the in-degree order inside each graph.
__global__ void k_rank_gid_keys(int64_t n, const u64 *__restrict__ sorted, const int *__restrict__ gid, u64 *keys) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
    const u32 v = (u32)sorted[i];
    keys[i] = ((u64)(u32)gid[v] << 32) | (u64)v;
  }
}

// rank[v] = position of v in the sorted order, or -1 when no entry names v:
// such vertices are never gathered, so the rank-order copies skip them.
__global__ void k_rank_from_sorted(int64_t n, const u64 *__restrict__ sorted, const int *__restrict__ indeg,
                                   int *rank) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
    const u32 v = (u32)sorted[i];
    rank[v] = indeg[v] > 0 ? (int)i : -1;
  }
}

// The distinct keys of a sorted array: one kernel counts the run starts of each
// tile, a scan of the tiles' counts gives each tile its place, and a second
// kernel finds the same starts again and unpacks them (source block, label,
// target block) there.  Bound by HBM: both read the keys once and nothing
// else.  A flag per entry, scanned to a place per entry, moved 28 bytes more an
// entry (125M entries, nearly all distinct: 1.54 ms; now 0.22 + 0.45).  A wave holds 1024 keys of consecutive positions, 64 at a
// time, so its starts are ballots and the stores of consecutive starts meet.
constexpr int RUN_ITEMS = 16;
constexpr int RUN_TILE = 256 * RUN_ITEMS;

// Bit `lane` of start[j]: key `lane` of the wave's row j starts a run.
__device__ inline u32 run_starts(int64_t m, const u64 *__restrict__ keys, int64_t base, u64 *k, u64 *start) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int j = 0; j < RUN_ITEMS; ++j) {
    const int64_t i = base + j * 64 + lane;
    k[j] = i < m ? keys[i] : 0ull;
  }
  u64 before = base > 0 && base < m ? keys[base - 1] : 0ull;  // the key left of the wave's row
  u32 count = 0;
#pragma unroll
  for (int j = 0; j < RUN_ITEMS; ++j) {
    const int64_t i = base + j * 64 + lane;
    u64 left = __shfl_up(k[j], 1, WAVE);
    if (lane == 0) left = before;
    start[j] = __ballot(i < m && (i == 0 || left != k[j]));
    before = __shfl(k[j], 63, WAVE);
    count += (u32)__popcll(start[j]);
  }
  return count;
}

__global__ void __launch_bounds__(256) k_run_count(int64_t m, const u64 *__restrict__ keys, int *__restrict__ count) {
  __shared__ u32 sh[4];
  const int w = threadIdx.x >> 6;
  u64 k[RUN_ITEMS], start[RUN_ITEMS];
  const u32 c = run_starts(m, keys, (int64_t)blockIdx.x * RUN_TILE + w * (RUN_TILE / 4), k, start);
  if ((threadIdx.x & 63) == 0) sh[w] = c;
  __syncthreads();
  if (threadIdx.x == 0) count[blockIdx.x] = (int)(sh[0] + sh[1] + sh[2] + sh[3]);
}

__global__ void __launch_bounds__(256) k_quotient_write(int64_t m, const u64 *__restrict__ keys,
                                                        const int64_t *__restrict__ pos, QKey q, int32_t *out_src,
                                                        int32_t *out_lab, int32_t *out_dst) {
  __shared__ u32 sh[4];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  u64 k[RUN_ITEMS], start[RUN_ITEMS];
  const u32 c = run_starts(m, keys, (int64_t)blockIdx.x * RUN_TILE + w * (RUN_TILE / 4), k, start);
  if (lane == 0) sh[w] = c;
  __syncthreads();
  int64_t at = pos[blockIdx.x];
  for (int i = 0; i < w; ++i) at += sh[i];
  const u64 below = (1ull << lane) - 1ull;
#pragma unroll
  for (int j = 0; j < RUN_ITEMS; ++j) {
    if ((start[j] >> lane) & 1ull) {
      const int64_t o = at + __popcll(start[j] & below);
      out_dst[o] = (int32_t)(k[j] & ((1ULL << q.db) - 1ULL));
      out_lab[o] = q.lb ? (int32_t)((k[j] >> q.db) & ((1ULL << q.lb) - 1ULL)) : 0;
      out_src[o] = (int32_t)(k[j] >> (q.db + q.lb));
    }
    at += __popcll(start[j]);
  }
}

// ---------------------------------------------------------------- incremental updates
// After edits to a graph, P'_1..P'_k are recomputed from the signatures of the
// vertices whose key inputs changed, with the cached key hashes of the others
// (the paper names incremental computation on evolving graphs as future
// work, Sec. "Discussion").  Blocks are named by their minimum vertex inside
// such chains (a name does not move when other blocks appear or vanish), so
// the key hash of a vertex whose own name and targets' names are unchanged is
// unchanged.  Dense first-vertex ids are still produced for every output.

// A graph read straight from its CSR, with the previous block name of every
// vertex in vertex order: the rows of edited vertices in the edited graph.
template <bool HK>
struct PlainSrcT {
  static constexpr bool GRAPH = true;
  static constexpr bool HASHED = HK;
  const int64_t *row_ptr;
  const int32_t *col;
  const int32_t *elabel;  // null: every edge has label 0
  const int32_t *names;   // previous block name of every vertex
  u32 pb;
  u32 kmask = 0xFFFFFFFFu;
  __device__ inline int64_t begin(int v) const { return row_ptr[v]; }
  __device__ inline int64_t end(int v) const { return row_ptr[v + 1]; }
  __device__ inline u32 pmask() const { return pb >= 31 ? 0x7FFFFFFFu : (1u << pb) - 1u; }
  __device__ inline u32 label(int64_t e) const { return elabel ? (u32)elabel[e] : 0u; }
  __device__ inline u64 pair(int64_t e) const {
    return ((u64)label(e) << 31) | (u64)((u32)names[col[e]] & pmask());
  }
  __device__ inline u32 own(int v) const { return (u32)names[v]; }
  // the same key forms as GraphSrcT
  __device__ inline u32 key32(int64_t e) const { return key32_of(label(e), (u32)col[e]); }
  // the row kernels' interface (as GraphSrcT, with targets in vertex order):
  // (label, target) of entries first + min(t + u*STRIDE, count - 1)
  template <int U, int STRIDE>
  __device__ inline void entries(int64_t first, int t, int count, u32 (&l)[U], u32 (&r)[U]) const {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int64_t e = first + min(t + u * STRIDE, count - 1);
      r[u] = (u32)__builtin_nontemporal_load(&col[e]);
      l[u] = elabel ? (u32)__builtin_nontemporal_load(&elabel[e]) : 0u;
    }
  }
  __device__ inline u64 pair_of(u32 l, u32 r) const { return ((u64)l << 31) | (u64)((u32)names[r] & pmask()); }
  __device__ inline u32 key32_of(u32 l, u32 r) const {
    return narrow_key<HK>(l, (u32)names[r] & pmask(), pb, kmask);
  }
};

constexpr int LIST_SMALL = 64;          // rows up to this many entries: one wave per vertex
constexpr int LIST_SET_BYTES = 32768;   // LDS set of the workgroup-per-vertex kernel

constexpr int LIST_BIG = 4096;  // longer rows go to the row and hub tiers, or a global set

// Split a vertex list by row length (rows of `row_ptr`): <= LIST_SMALL entries
// to small[], up to huge_min to large[], longer ones to huge[].  Counters
// start at zero.
__global__ void k_split_list(int count, const int *__restrict__ list, const int64_t *__restrict__ row_ptr,
                             int *nsmall, int *small, int *nlarge, int *large, int64_t huge_min, int *nhuge,
                             int *huge) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  const bool act = i < count;
  const int v = act ? list[i] : 0;
  const int64_t d = act ? row_ptr[v + 1] - row_ptr[v] : 0;
  wave_append(nsmall, small, act && d <= LIST_SMALL, v);
  wave_append(nlarge, large, act && d > LIST_SMALL && d <= huge_min, v);
  wave_append(nhuge, huge, act && d > huge_min, v);
}

// Key hash of the listed vertices with short rows: one wave per vertex, an
// LDS set of 2 * LIST_SMALL slots per wave.  Writes H and DC and inserts the
// key into the grouping table (or the empty-signature representatives).
template <class Src, class K>
__global__ void __launch_bounds__(256) k_sig_list_small(Src src, const int *__restrict__ count,
                                                        const int *__restrict__ list, u64 *__restrict__ H,
                                                        u32 *__restrict__ DC, u64 *table, u64 tmask,
                                                        const u32 *__restrict__ dep, u64 hmask, u64 *zrep) {
  typedef Keys<K> KO;
  constexpr int SL = 2 * LIST_SMALL;
  __shared__ K set[4][SL];
  const u32 epoch = dep[EP_TABLE], zep = dep[EP_ZERO];
  const int lane = threadIdx.x & (WAVE - 1), w = threadIdx.x >> 6;
  const int total = *count;
  const int waves = gridDim.x * 4;
  for (int item = blockIdx.x * 4 + w; item < total; item += waves) {
    const int v = list[item];
    const int64_t b = src.begin(v);
    const int d = (int)(src.end(v) - b);
    set[w][lane] = KO::EMPTY;
    set[w][lane + WAVE] = KO::EMPTY;
    __builtin_amdgcn_wave_barrier();
    u64 a = 0;
    u32 c = 0;
    if (lane < d) {
      const K p = KO::load(src, b + lane);
      u32 sl = KO::hash(p) & (SL - 1);
      while (true) {
        const K old = atomicCAS(&set[w][sl], KO::EMPTY, p);
        if (old == KO::EMPTY) { a = KO::mix(p); c = 1; break; }
        if (old == p) break;
        sl = (sl + 1) & (SL - 1);
      }
    }
    a = wave_sum_u64(a);
    c = wave_sum_u32(c);
    if (lane == 0) {
      const u32 own = src.own(v);
      const u64 h = finalize_key(a, c, own) & hmask;
      H[v] = h;
      DC[v] = c;
      key_insert(table, tmask, zrep, h, c, own, (u32)v, epoch, zep);
    }
    __builtin_amdgcn_wave_barrier();
  }
}

// The same for longer rows: one workgroup per vertex.  The row's distinct keys
// go through an LDS set in Q passes (keys of sub-partition q in pass q), Q a
// power of two doubled whenever a pass fills the set beyond 3/4 (the
// partition is then redone), so any row length works.
template <class Src, class K>
__global__ void __launch_bounds__(256) k_sig_list_large(Src src, const int *__restrict__ count,
                                                        const int *__restrict__ list, u64 *__restrict__ H,
                                                        u32 *__restrict__ DC, u64 *table, u64 tmask,
                                                        const u32 *__restrict__ dep, u64 hmask, u64 *zrep,
                                                        u32 *err) {
  typedef Keys<K> KO;
  constexpr int PS = LIST_SET_BYTES / (int)sizeof(K);
  __shared__ K set[PS];
  __shared__ u64 sh_acc[4];
  __shared__ u32 sh_cnt[4];
  __shared__ u32 sh_fill[2];
  const u32 epoch = dep[EP_TABLE], zep = dep[EP_ZERO];
  const int total = *count;
  for (int item = blockIdx.x; item < total; item += gridDim.x) {
    const int v = list[item];
    const int64_t b = src.begin(v), e = src.end(v);
    const int64_t d = e - b;
    u32 Q = 1;
    while ((int64_t)Q * (PS / 2) < d && Q < (1u << 20)) Q <<= 1;
    u64 acc = 0;
    u32 cnt = 0;
    for (int i = threadIdx.x; i < PS; i += 256) set[i] = KO::EMPTY;
    for (u32 q = 0; q < Q;) {
      if (threadIdx.x == 0) { sh_fill[0] = 0; sh_fill[1] = 0; }
      __syncthreads();
      u64 pacc = 0;
      u32 pcnt = 0;
      for (int64_t j = b + threadIdx.x; j < e; j += 256) {
        const K p = KO::load(src, j);
        if (Q > 1 && (sub_hash((u64)p) & (Q - 1)) != q) continue;
        u32 sl = KO::hash(p) & (PS - 1);
        const bool full = set_full(&sh_fill[1]);  // at most one insertion per thread lands after the mark
        while (true) {
          const K cur = set[sl];
          if (cur == p) break;
          if (cur == KO::EMPTY) {
            if (full) break;  // overflowed: the pass is redone with more sub-partitions
            const K old = atomicCAS(&set[sl], KO::EMPTY, p);
            if (old == KO::EMPTY) {
              pacc += KO::mix(p);
              ++pcnt;
              if (atomicAdd(&sh_fill[0], 1u) + 1u >= (u32)(PS / 4 * 3)) mark_full(&sh_fill[1]);
              break;
            }
            if (old == p) break;
          }
          sl = (sl + 1) & (PS - 1);
        }
      }
      __syncthreads();
      const bool over = sh_fill[1] != 0;
      __syncthreads();
      for (int i = threadIdx.x; i < PS; i += 256) set[i] = KO::EMPTY;
      if (over) {
        if (Q >= (1u << 24)) {
          if (threadIdx.x == 0) atomicOr(err, ERR_VERIFY_OVERFLOW);
          break;
        }
        Q <<= 1;
        q = 0;
        acc = 0;
        cnt = 0;
      } else {
        acc += pacc;
        cnt += pcnt;
        ++q;
      }
      __syncthreads();
    }
    block_reduce_2(acc, cnt, sh_acc, sh_cnt);
    if (threadIdx.x == 0) {
      const u32 own = src.own(v);
      const u64 h = finalize_key(acc, cnt, own) & hmask;
      H[v] = h;
      DC[v] = cnt;
      key_insert(table, tmask, zrep, h, cnt, own, (u32)v, epoch, zep);
    }
    __syncthreads();
  }
}

// Vertices whose key inputs did not change take their cached key hash and
// distinct count.  Only some of them are inserted: a clean vertex that headed
// its cached block (mvc[v] == v), and every clean member of a cached block
// whose head changed.  Clean members of one cached block stay together with
// equal keys, so every new block's minimum vertex is inserted (its head if
// clean, else all its clean members; changed vertices insert themselves),
// and the table ends with the same minimum per slot as if all were inserted.
// Empty signatures go by their own block name, the same way.
__global__ void __launch_bounds__(256) k_insert_cached(int n, const unsigned char *__restrict__ dirty,
                                                       const u64 *__restrict__ Hc, const u32 *__restrict__ DCc,
                                                       const int32_t *__restrict__ mvc,
                                                       const int32_t *__restrict__ names, u64 *__restrict__ H,
                                                       u32 *__restrict__ DC, u64 *table, u64 tmask,
                                                       const u32 *__restrict__ dep, u64 *zrep) {
  const u32 epoch = dep[EP_TABLE], zep = dep[EP_ZERO];
  const int v = blockIdx.x * 256 + threadIdx.x;
  const bool act = v < n && !dirty[v];
  bool zero = false, keyed = false;
  u32 own = 0;
  u64 h = 0;
  if (act) {
    const u32 c = DCc[v];
    DC[v] = c;
    const int head = mvc[v];
    const bool ins = head == v || dirty[head];
    if (c) {
      h = Hc[v];
      H[v] = h;
      keyed = ins;
    } else if (ins) {
      zero = true;
      own = (u32)names[v];
    }
  }
  __shared__ u32 slots[4][2 * FIRST_SLOTS];
  u32 *sw = slots[threadIdx.x >> 6];
  if (wave_first_of_key(sw, keyed, h)) table_insert(table, tmask, h, (u32)v, epoch);
  zero_insert_wave(sw, zrep, zero, own, (u32)v, zep);
}

// Every vertex: dense id from its representative (head words), its new
// block name in vertex order and, for the next gather, in rank order.  The name is the representative (the block's minimum
// vertex), or with bname (an update) the name bname[] gives the
// representative's block; vertices whose name differs from the cached
// chain's (old_names) are then listed in changed[].
// list != NULL: only the `count` listed vertices (out may then be NULL).
__global__ void k_assign_names(int n, const int *__restrict__ rep, HeadIds ids, int *__restrict__ out,
                               int32_t *__restrict__ names_out,
                               const int *__restrict__ rank, int *__restrict__ gpid_next,
                               const int32_t *__restrict__ bname, const int32_t *__restrict__ keep,
                               const int32_t *__restrict__ old_names, int *nchanged, int *changed,
                               int count = 0, const int *__restrict__ list = nullptr) {
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  const bool act = t < (list ? count : n);
  const int v = act ? (list ? list[t] : t) : 0;
  bool moved = false;
  if (act) {
    const int r = rep[v];
    if (out) out[v] = r >= 0 ? head_id(ids, r) : -1;
    int nm = r;
    if (bname) {
      nm = r >= 0 ? bname[r] : -1;
      if (nm >= n && keep[r] < n) nm = keep[r];
    }
    names_out[v] = nm;
    if (rank) {
      const int rk = rank[v];
      if (rk >= 0) gpid_next[rk] = nm;
    }
    moved = old_names && old_names[v] != nm;
  }
  if (old_names) wave_append(nchanged, changed, moved, v);
}

// Update steps with few dirty vertices group only the blocks that can have
// changed.  Clean members of a cached block keep equal keys, so a cached
// block B keeps exactly its members (and its minimum vertex and name) unless
// it holds a dirty vertex (bit "minimum vertex" of touch, set by
// k_update_flags; a bitmap of n bits, so that its reads stay in the caches) or a
// dirty vertex now has B's key.  The second is found by each clean vertex
// looking its own cached key up among the dirty keys already inserted (the
// table, or zrep for an empty signature, whose key is the own name alone):
// every member of B asks with the same key and gets the same answer; a hash
// match whose keys differ only costs work, the exact check sorts it out.
// Dirty vertices and the clean members of such "touched" blocks are listed
// (the clean ones take their cached key hash and distinct count); every other
// vertex keeps its cached block: representative and name = the cached
// minimum vertex.
// A bit filter of the dirty keys lets most clean vertices skip the table
// probe: one of FILTER_BITS bits per key, from bits 36.. of its hash (as the
// table's slot tags), or for an empty signature from a multiplicative hash of
// the own name.  The same filter holds a bit per touched block (another
// multiplicative hash of its minimum vertex), so that most clean vertices
// skip the touch bitmap too.  Copied to LDS by every workgroup of
// k_classify, so the grid strides over vertices.  A clean vertex's bit is fixed by the cached chain
// (its key hash, distinct count and previous name do not change), so it is
// kept per step in the chain (k_filter_keys) and k_classify reads 2 bytes
// per vertex for the test instead of the hash, count and name.
constexpr int FILTER_BITS = 1 << 16;
constexpr int FILTER_WORDS = FILTER_BITS / 32;
constexpr int CLASSIFY_GRID = 2048;
__device__ inline u32 filter_key_bit(u64 h) { return (u32)(h >> 36) & (FILTER_BITS - 1); }
__device__ inline u32 filter_name_bit(u32 name) { return (name * 0x9E3779B1u) >> 16; }
__device__ inline u32 filter_touch_bit(u32 head) { return (head * 0x85EBCA6Bu) >> 16; }
// With many dirty keys the LDS filter fills up; a second, global filter of
// GFILTER_BITS bits (16 MB, held in the L2 and MALL) then keeps most clean
// vertices from a table probe in HBM.  Its key bits come from other hash bits
// than the LDS filter's.
constexpr int64_t GFILTER_BITS = int64_t(1) << 27;
constexpr int64_t GFILTER_WORDS = GFILTER_BITS / 32;
constexpr int GFILTER_MIN_DIRTY = FILTER_BITS / 16;  // fewer dirty keys: the LDS filter suffices
__device__ inline u32 gfilter_key_bit(u64 h) { return (u32)h & (u32)(GFILTER_BITS - 1); }
__device__ inline u32 gfilter_name_bit(u32 name) {
  return (u32)(((u64)name * 0x9E3779B97F4A7C15ull) >> 37) & (u32)(GFILTER_BITS - 1);
}

// Filter bit of every vertex's key at one step of a cached chain.
__global__ void k_filter_keys(int n, const u64 *__restrict__ H, const u32 *__restrict__ DC,
                              const int32_t *__restrict__ names_prev, uint16_t *__restrict__ fk) {
  const int v = blockIdx.x * blockDim.x + threadIdx.x;
  if (v >= n) return;
  fk[v] = (uint16_t)(DC[v] ? filter_key_bit(H[v]) : filter_name_bit((u32)names_prev[v]));
}

// gfilter: the global filter (cleared), or null.
__global__ void k_build_filter(const int *__restrict__ count, const int *__restrict__ dlist,
                               const u64 *__restrict__ H, const u32 *__restrict__ DC,
                               const int32_t *__restrict__ names, const int32_t *__restrict__ mvc, u32 *filter,
                               u32 *gfilter) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= *count) return;
  const int d = dlist[i];
  const u32 dc = DC[d];
  const u64 h = dc ? H[d] : 0ull;
  const u32 nm = (u32)names[d];
  const u32 b = dc ? filter_key_bit(h) : filter_name_bit(nm);
  atomicOr(&filter[b >> 5], 1u << (b & 31));
  const u32 t = filter_touch_bit((u32)mvc[d]);
  atomicOr(&filter[t >> 5], 1u << (t & 31));
  if (gfilter) {
    const u32 g = dc ? gfilter_key_bit(h) : gfilter_name_bit(nm);
    atomicOr(&gfilter[g >> 5], 1u << (g & 31));
  }
}

constexpr int CLASSIFY_HELD = 4096;
__global__ void __launch_bounds__(256) k_classify(int n, const int32_t *__restrict__ mvc,
                                                  const unsigned char *__restrict__ dirty,
                                                  const u32 *__restrict__ touch,
                                                  const uint16_t *__restrict__ fkc, const u64 *__restrict__ Hc,
                                                  const u32 *__restrict__ DCc, const int32_t *__restrict__ names,
                                                  const u32 *__restrict__ filter,
                                                  const u32 *__restrict__ gfilter, const u64 *table, u64 tmask,
                                                  const u32 *__restrict__ dep, const u64 *__restrict__ zrep,
                                                  u64 *__restrict__ H, u32 *__restrict__ DC, int *__restrict__ rep,
                                                  int32_t *__restrict__ names_out, int *count, int *list) {
  __shared__ u32 fl[FILTER_WORDS];
  for (int i = threadIdx.x; i < FILTER_WORDS; i += 256) fl[i] = filter[i];
  __syncthreads();
  const u32 epoch = dep[EP_TABLE], zep = dep[EP_ZERO];
  // CV consecutive vertices per thread and round, read and written 4 at a
  // time when every array's start allows (a step's slice of the chain starts
  // at step * n, so with n not a multiple of 4 they are read one by one).
  // Every vertex first gets its cached block as representative and name; a
  // listed vertex's are overwritten by the lookup and naming kernels of the
  // step.  The cached key itself is read only by vertices that pass the touch
  // or filter test.
  constexpr int CV = 4;
  const bool vec = ((reinterpret_cast<uintptr_t>(mvc) | reinterpret_cast<uintptr_t>(rep) |
                     reinterpret_cast<uintptr_t>(names_out)) & 15) == 0 &&
                   (reinterpret_cast<uintptr_t>(fkc) & 7) == 0 && (reinterpret_cast<uintptr_t>(dirty) & 3) == 0;
  // Listed vertices are held in LDS and appended CLASSIFY_HELD or so at a time:
  // with many dirty keys most rounds list some, and the atomics on the one
  // counter serialise (12 ns each; 8.4M vertices, one per round of 1024: 141 us
  // a step, now 116).
  __shared__ u32 sh_w[4];
  __shared__ int sh_base;
  __shared__ int buf[CLASSIFY_HELD];
  u32 held = 0;  // uniform in the workgroup
  auto flush = [&]() {
    __syncthreads();
    if (threadIdx.x == 0) sh_base = atomicAdd(count, (int)held);
    __syncthreads();
    for (u32 i = threadIdx.x; i < held; i += 256) list[sh_base + (int)i] = buf[i];
    __syncthreads();  // buf and sh_base are written again
    held = 0;
  };
  const int64_t stride = (int64_t)gridDim.x * 256 * CV;
  for (int64_t b0 = (int64_t)blockIdx.x * 256 * CV; b0 < n; b0 += stride) {  // uniform in the workgroup
    const int64_t v0 = b0 + (int64_t)threadIdx.x * CV;
    int hd[CV];
    u32 fk[CV], dv[CV];
    const bool full = vec && v0 + CV <= n;
    if (full) {
      const u32 d4 = *reinterpret_cast<const u32 *>(dirty + v0);
      const int4 m4 = *reinterpret_cast<const int4 *>(mvc + v0);
      const uint2 f2 = *reinterpret_cast<const uint2 *>(fkc + v0);
      hd[0] = m4.x; hd[1] = m4.y; hd[2] = m4.z; hd[3] = m4.w;
      fk[0] = f2.x & 0xffffu; fk[1] = f2.x >> 16; fk[2] = f2.y & 0xffffu; fk[3] = f2.y >> 16;
#pragma unroll
      for (int j = 0; j < CV; ++j) dv[j] = (d4 >> (8 * j)) & 0xffu;
      *reinterpret_cast<int4 *>(rep + v0) = m4;
      *reinterpret_cast<int4 *>(names_out + v0) = m4;
    } else {
#pragma unroll
      for (int j = 0; j < CV; ++j) {
        const bool in = v0 + j < n;
        dv[j] = in ? dirty[v0 + j] : 1u;
        hd[j] = in ? mvc[v0 + j] : 0;
        fk[j] = in ? fkc[v0 + j] : 0u;
        if (in) {
          rep[v0 + j] = hd[j];
          names_out[v0 + j] = hd[j];
        }
      }
    }
    u32 tb[CV];
#pragma unroll
    for (int j = 0; j < CV; ++j) {
      // the touch bitmap is read only where the filter says "maybe touched"
      const u32 t = filter_touch_bit((u32)hd[j]);
      if (dv[j]) tb[j] = 1u;
      else if ((fl[t >> 5] >> (t & 31)) & 1u) tb[j] = (touch[hd[j] >> 5] >> (hd[j] & 31)) & 1u;
      else tb[j] = 0u;
    }
    // clean vertices that may share a key with a dirty one (filter hit) or
    // belong to a touched block read their cached key; all such loads are
    // requested before the first is used (with many dirty keys most vertices
    // take this path)
    bool probe[CV], need[CV];
#pragma unroll
    for (int j = 0; j < CV; ++j) {
      const bool clean = v0 + j < n && !dv[j];
      probe[j] = clean && !tb[j] && ((fl[fk[j] >> 5] >> (fk[j] & 31)) & 1u);
      need[j] = clean && (tb[j] || probe[j]);
    }
    u32 dc[CV];
    u64 hv[CV];
#pragma unroll
    for (int j = 0; j < CV; ++j) {
      dc[j] = need[j] ? DCc[v0 + j] : 0u;
      hv[j] = need[j] ? Hc[v0 + j] : 0ull;
    }
    bool listed[CV];
#pragma unroll
    for (int j = 0; j < CV; ++j) {
      const int v = (int)(v0 + j);
      listed[j] = v0 + j < n && dv[j];
      if (need[j]) {
        bool hit = !probe[j];  // touched
        if (probe[j]) {
          const u32 nm = dc[j] == 0 ? (u32)names[v] : 0u;
          bool maybe = true;
          if (gfilter) {
            const u32 g = dc[j] ? gfilter_key_bit(hv[j]) : gfilter_name_bit(nm);
            maybe = (gfilter[g >> 5] >> (g & 31)) & 1u;
          }
          if (maybe) {
            if (dc[j] == 0) hit = (u32)(zrep[nm] >> 32) == ~zep;
            else hit = table_lookup(table, tmask, hv[j], epoch) >= 0;
          }
        }
        if (hit) {
          H[v] = hv[j];
          DC[v] = dc[j];
          listed[j] = true;
        }
      }
    }
    u32 mine = 0;
#pragma unroll
    for (int j = 0; j < CV; ++j) mine += listed[j] ? 1u : 0u;
    if (!__syncthreads_or(mine != 0)) continue;  // most rounds with few dirty keys
    u32 total;
    u32 at = held + block_exclusive_scan(mine, sh_w, &total);
#pragma unroll
    for (int j = 0; j < CV; ++j)
      if (listed[j]) buf[at++] = (int)(v0 + j);
    held += total;
    if (held > CLASSIFY_HELD - 256 * CV) flush();
  }
  if (held) flush();
}

// Inserts the listed vertices' keys (table, or zrep for empty signatures).
__global__ void __launch_bounds__(256) k_insert_list(int count, const int *__restrict__ list,
                                                     const u64 *__restrict__ H, const u32 *__restrict__ DC,
                                                     const int32_t *__restrict__ names, u64 *table, u64 tmask,
                                                     const u32 *__restrict__ dep, u64 *zrep) {
  const u32 epoch = dep[EP_TABLE], zep = dep[EP_ZERO];
  const int i = blockIdx.x * 256 + threadIdx.x;
  const bool act = i < count;
  const int v = act ? list[i] : 0;
  const u32 dc = act ? DC[v] : 0;
  // one insert per key of the wave (listed vertices are not in order)
  __shared__ u32 slots[4][2 * FIRST_SLOTS];
  const u64 h = act && dc ? H[v] : 0;
  u32 mv = (u32)v;
  u32 *sw = slots[threadIdx.x >> 6];
  if (wave_min_of_key(sw, act && dc, h, mv)) table_insert(table, tmask, h, mv, epoch);
  zero_insert_wave(sw, zrep, act && dc == 0, act ? (u32)names[v] : 0u, (u32)v, zep);
}

// Row extents (begin, end) of listed vertices.
__global__ void k_row_extents(int count, const int *__restrict__ list, const int64_t *__restrict__ row_ptr,
                              int64_t *__restrict__ be) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= count) return;
  const int v = list[i];
  be[2 * i] = row_ptr[v];
  be[2 * i + 1] = row_ptr[v + 1];
}

// Row lengths of listed vertices.
__global__ void k_row_degrees(int count, const int *__restrict__ list, const int64_t *__restrict__ row_ptr,
                              int64_t *__restrict__ deg) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= count) return;
  const int v = list[i];
  deg[i] = row_ptr[v + 1] - row_ptr[v];
}

// Dense id of every vertex: its representative's (head words).
__global__ void __launch_bounds__(256) k_assign_out(int n, const int *__restrict__ rep, HeadIds ids,
                                                    int *__restrict__ out) {
  const int64_t v0 = ((int64_t)blockIdx.x * 256 + threadIdx.x) * ASSIGN_V;
  if (v0 >= n) return;
  if (v0 + ASSIGN_V <= n && ((reinterpret_cast<uintptr_t>(rep) | reinterpret_cast<uintptr_t>(out)) & 15) == 0) {
    const int4 r4 = *reinterpret_cast<const int4 *>(rep + v0);
    *reinterpret_cast<int4 *>(out + v0) =
        make_int4(r4.x >= 0 ? head_id(ids, r4.x) : -1, r4.y >= 0 ? head_id(ids, r4.y) : -1,
                  r4.z >= 0 ? head_id(ids, r4.z) : -1, r4.w >= 0 ? head_id(ids, r4.w) : -1);
  } else {
    for (int64_t v = v0; v < v0 + ASSIGN_V && v < n; ++v) {
      const int r = rep[v];
      out[v] = r >= 0 ? head_id(ids, r) : -1;
    }
  }
}

// Block names of an update step.  A new block that keeps an unchanged
// (clean) member takes that member's cached name: clean members of one new
// block shared their cached block (their keys did not change), and no other
// new block holds a member of it, so such names stay distinct.  A block of
// changed vertices only is named n + its minimum vertex, above every cached
// name.  Clean vertices therefore never change names, and renaming does not
// spread through blocks that only gained or lost a few members.
// A block of changed vertices only that holds the vertex which named a cached
// block (old_names[v] == v), and whose cached name no clean member claimed,
// keeps that name (the smallest such vertex, so the choice is
// deterministic): a block whose members all changed keys but stayed
// together, e.g. a singleton, is not renamed.  No other new block can hold
// that vertex, so the name stays distinct.
// Each runs over every vertex, or over the `count` listed ones (list != NULL:
// the vertices of the blocks that can have changed; every other block keeps
// its members and its cached name).
__device__ inline int name_item(int n, int count, const int *list, bool &act) {
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  act = t < (list ? count : n);
  return act ? (list ? list[t] : t) : 0;
}
__global__ void k_block_names_fresh(int n, const int *__restrict__ rep, int32_t *__restrict__ bname,
                                    int32_t *__restrict__ keep, int count = 0, const int *__restrict__ list = nullptr) {
  bool act;
  const int v = name_item(n, count, list, act);
  if (act && rep[v] == v) {
    bname[v] = n + v;
    keep[v] = 0x7FFFFFFF;
  }
}
__global__ void k_block_names_clean(int n, const int *__restrict__ rep, const unsigned char *__restrict__ dirty,
                                    const int32_t *__restrict__ old_names, int32_t *__restrict__ bname,
                                    unsigned char *__restrict__ claimed, int count = 0,
                                    const int *__restrict__ list = nullptr) {
  bool act;
  const int v = name_item(n, count, list, act);
  if (act && !dirty[v]) {
    const int32_t nm = old_names[v];
    bname[rep[v]] = nm;
    claimed[nm] = 1;
  }
}
__global__ void k_block_names_keep(int n, const int *__restrict__ rep, const unsigned char *__restrict__ dirty,
                                   const int32_t *__restrict__ old_names, const int32_t *__restrict__ bname,
                                   const unsigned char *__restrict__ claimed, int32_t *keep, int count = 0,
                                   const int *__restrict__ list = nullptr) {
  bool act;
  const int v = name_item(n, count, list, act);
  if (act && dirty[v] && old_names[v] == v && !claimed[v]) {
    const int r = rep[v];
    if (bname[r] >= n) atomicMin(&keep[r], v);
  }
}

// Flags for the next step of an update: a vertex whose name changed, and every
// vertex with an edge into it (in-rows of the cached graph; an edge that an
// edit added starts at an edited row, which is recomputed at every step
// anyway).  One wave per changed vertex.
constexpr int MARK_LIGHT = 4096;  // in-rows up to this long are marked by one wave

__global__ void __launch_bounds__(256) k_mark_in_neighbours(const int *__restrict__ count, const int *__restrict__ list,
                                                            const int64_t *__restrict__ tptr,
                                                            const int32_t *__restrict__ tcol,
                                                            unsigned char *flag, int *nheavy, int *heavy) {
  const int lane = threadIdx.x & (WAVE - 1);
  const int total = *count;
  const int waves = (int)((gridDim.x * blockDim.x) >> 6);
  for (int item = (int)((blockIdx.x * blockDim.x + threadIdx.x) >> 6); item < total; item += waves) {
    const int w = list[item];
    const int64_t b = tptr[w], e = tptr[w + 1];
    if (lane == 0) {
      flag[w] = 1;
      if (e - b > MARK_LIGHT) heavy[atomicAdd(nheavy, 1)] = w;
    }
    if (e - b <= MARK_LIGHT)
      for (int64_t j = b + lane; j < e; j += WAVE) flag[tcol[j]] = 1;
  }
}

// In-rows longer than MARK_LIGHT: every workgroup takes its share of each.
__global__ void __launch_bounds__(256) k_mark_heavy(const int *__restrict__ nheavy, const int *__restrict__ heavy,
                                                    const int64_t *__restrict__ tptr,
                                                    const int32_t *__restrict__ tcol, unsigned char *flag) {
  const int total = *nheavy;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int h = 0; h < total; ++h) {
    const int w = heavy[h];
    for (int64_t j = tptr[w] + (int64_t)blockIdx.x * blockDim.x + threadIdx.x; j < tptr[w + 1]; j += stride)
      flag[tcol[j]] = 1;
  }
}

// Per vertex of an update step: dirty = its key inputs may have changed
// (edited row, or flagged by the previous step); skip = not refined by the
// tier kernels (clean, or edited: edited rows are read from the edited graph
// by the list kernels).
// The flagged vertices whose rows were not edited are also listed, split by
// row length (as k_split_list), so that few of them can be signed by the list
// kernels instead of the tier kernels: counts at cnt[0] (short) and cnt[1]
// (up to LIST_BIG entries); longer rows are counted at cnt[2] and left to
// the row and hub tiers (skip[v] = 0 for exactly them).
// Bit mvc[v] of touch is set for every dirty v: its cached block may lose members;
// the dirty vertices are listed in dlist (count at cnt[4]).
constexpr int FLAGS_GROUP = 16;  // vertices per thread in k_update_flags
__global__ void __launch_bounds__(256) k_update_flags(int n, const unsigned char *__restrict__ edited,
                                                      const unsigned char *__restrict__ flag,
                                                      unsigned char *__restrict__ dirty,
                                                      unsigned char *__restrict__ skip,
                                                      const int64_t *__restrict__ row_ptr, int *cnt, int *small,
                                                      int *large, const int32_t *__restrict__ mvc,
                                                      u32 *__restrict__ touch, int *dlist) {
  // FLAGS_GROUP vertices per thread, their bytes moved 16 at a time where the
  // arrays allow.  Most groups are clean (no byte set in either input): one
  // load and one store of each array.  A group with a set byte decides per
  // vertex; its list members are appended once per wave (bit masks).
  const int64_t v0 = ((int64_t)blockIdx.x * 256 + threadIdx.x) * FLAGS_GROUP;
  const bool vec = v0 + FLAGS_GROUP <= n &&
                   ((reinterpret_cast<uintptr_t>(edited) | reinterpret_cast<uintptr_t>(flag) |
                     reinterpret_cast<uintptr_t>(dirty) | reinterpret_cast<uintptr_t>(skip)) & 15) == 0;
  u32 eb = 0, fb = 0;  // bit j: vertex v0 + j edited / flagged
  if (vec) {
    const u32x4 e = *reinterpret_cast<const u32x4 *>(edited + v0);
    const u32x4 f = *reinterpret_cast<const u32x4 *>(flag + v0);
#pragma unroll
    for (int j = 0; j < FLAGS_GROUP; ++j) {
      const u32 sh = 8 * (j & 3);
      const u32 ew = j < 4 ? e.x : j < 8 ? e.y : j < 12 ? e.z : e.w;
      const u32 fw = j < 4 ? f.x : j < 8 ? f.y : j < 12 ? f.z : f.w;
      eb |= (((ew >> sh) & 0xffu) != 0u ? 1u : 0u) << j;
      fb |= (((fw >> sh) & 0xffu) != 0u ? 1u : 0u) << j;
    }
  } else {
    for (int j = 0; j < FLAGS_GROUP && v0 + j < n; ++j) {
      eb |= (edited[v0 + j] != 0 ? 1u : 0u) << j;
      fb |= (flag[v0 + j] != 0 ? 1u : 0u) << j;
    }
  }
  const u32 mdirty = eb | fb, mprop = fb & ~eb;
  // row lengths of the flagged unedited vertices, all requested together
  int64_t d[FLAGS_GROUP];
#pragma unroll
  for (int j = 0; j < FLAGS_GROUP; ++j) d[j] = (mprop >> j) & 1u ? row_ptr[v0 + j + 1] - row_ptr[v0 + j] : 0;
  u32 msmall = 0, mlarge = 0, mbig = 0;
#pragma unroll
  for (int j = 0; j < FLAGS_GROUP; ++j) {
    if (!((mprop >> j) & 1u)) continue;
    if (d[j] <= LIST_SMALL) msmall |= 1u << j;
    else if (d[j] <= LIST_BIG) mlarge |= 1u << j;
    else mbig |= 1u << j;
  }
  // dirty = edited or flagged; skip = all but the flagged unedited rows past LIST_BIG
  if (vec) {
    u32 dw[4] = {0u, 0u, 0u, 0u}, sw[4] = {0x01010101u, 0x01010101u, 0x01010101u, 0x01010101u};
#pragma unroll
    for (int j = 0; j < FLAGS_GROUP; ++j) {
      dw[j >> 2] |= ((mdirty >> j) & 1u) << (8 * (j & 3));
      sw[j >> 2] &= ~(((mbig >> j) & 1u) << (8 * (j & 3)));
    }
    *reinterpret_cast<u32x4 *>(dirty + v0) = u32x4{dw[0], dw[1], dw[2], dw[3]};
    *reinterpret_cast<u32x4 *>(skip + v0) = u32x4{sw[0], sw[1], sw[2], sw[3]};
  } else {
    for (int j = 0; j < FLAGS_GROUP && v0 + j < n; ++j) {
      dirty[v0 + j] = (mdirty >> j) & 1u;
      skip[v0 + j] = ((mbig >> j) & 1u) ? 0 : 1;
    }
  }
  // touch: the cached block of every dirty vertex (many share one: set its bit once)
  for (u32 m = mdirty; m; m &= m - 1u) {
    const int h = mvc[v0 + __ffs(m) - 1];
    const u32 bit = 1u << (h & 31);
    if (!(__hip_atomic_load(&touch[h >> 5], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & bit))
      atomicOr(&touch[h >> 5], bit);
  }
  if (!__ballot(mdirty != 0)) return;
  wave_append_mask(&cnt[0], small, msmall, v0);
  wave_append_mask(&cnt[1], large, mlarge, v0);
  wave_append_mask(&cnt[4], dlist, mdirty, v0);
  const u32 nbig = wave_sum_u32((u32)__popc(mbig));
  if ((threadIdx.x & (WAVE - 1)) == 0 && nbig) atomicAdd(&cnt[2], (int)nbig);
}

// Skip flags when every flagged unedited vertex goes to the tier kernels.
__global__ void k_skip_all_flagged(int n, const unsigned char *__restrict__ edited, const unsigned char *__restrict__ flag_dirty,
                                   unsigned char *__restrict__ skip) {
  const int v = blockIdx.x * blockDim.x + threadIdx.x;
  if (v < n) skip[v] = (flag_dirty[v] && !edited[v]) ? 0 : 1;
}

__global__ void k_set_flags(const int *__restrict__ count, const int *__restrict__ list, unsigned char *flag) {
  const int total = *count;
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < total; i += gridDim.x * blockDim.x) flag[list[i]] = 1;
}

// ---------------------------------------------------------------- epochs
__global__ void k_advance(u32 *dep, u32 mask) {
  if (threadIdx.x != 0 || blockIdx.x != 0) return;
  if (mask & ADV_TABLE) {
    dep[EP_TABLE] = dep[EP_TABLE] % 15u + 1u;
    dep[EP_CLR_TABLE] = dep[EP_TABLE] == 1u;
  } else {
    dep[EP_CLR_TABLE] = 0;
  }
  if (mask & ADV_CTABLE) {
    dep[EP_CTABLE] = dep[EP_CTABLE] % 15u + 1u;
    dep[EP_CLR_CTABLE] = dep[EP_CTABLE] == 1u;
  } else {
    dep[EP_CLR_CTABLE] = 0;
  }
  if (mask & ADV_ZERO) dep[EP_ZERO] = dep[EP_ZERO] + 1u;
  if (mask & ADV_HUB) {
    dep[EP_HUB] = dep[EP_HUB] % 3u + 1u;
    dep[EP_CLR_HUB] = dep[EP_HUB] == 1u;
  } else {
    dep[EP_CLR_HUB] = 0;
  }
}

// Counters and epochs of steps [i0, i0 + cnt) of a call (cnt <= 14), ahead of
// all of them: row i of `rows` (STEP_ROW words) gets zeroed counters and, from
// STEP_EPOCHS on, the step's own epochs, so a step launches nothing for them.
// Epochs that would wrap inside the segment start again from 1, and the table
// is cleared before it (k_clear_if).  Without `table` (steps that group by
// partition) the table's epoch stays: slots that such steps do not overwrite must
// not meet their epoch again.  reset_err: also clear the error word.
constexpr int STEP_ROW = 16, STEP_EPOCHS = 8, STEP_SEGMENT = 14;
__global__ void k_prepare_steps(u32 *dep, int *rows, int i0, int cnt, int table, u32 *err, int reset_err) {
  const int t = threadIdx.x;
  u32 e = dep[EP_TABLE];
  const u32 z = dep[EP_ZERO], hub = dep[EP_HUB], ec = dep[EP_CTABLE];
  const bool wrap = table && e + (u32)cnt > 15u;
  if (wrap) e = 0;
  if (t < cnt) {
    int *row = rows + (int64_t)(i0 + t) * STEP_ROW;
    for (int j = 0; j < STEP_EPOCHS; ++j) row[j] = 0;
    u32 *d = reinterpret_cast<u32 *>(row) + STEP_EPOCHS;
    d[EP_TABLE] = table ? e + (u32)t + 1u : e;
    d[EP_CTABLE] = ec;  // (these steps do not use the peeling table)
    d[EP_ZERO] = z + (u32)t + 1u;
    d[EP_HUB] = hub;
  }
  __syncthreads();  // every thread has read dep
  if (t == 0) {
    dep[EP_TABLE] = table ? e + (u32)cnt : e;
    dep[EP_ZERO] = z + (u32)cnt;
    dep[EP_CLR_TABLE] = wrap;
    dep[EP_CLR_CTABLE] = 0;
    dep[EP_CLR_HUB] = 0;
    if (reset_err) *err = 0;
  }
}

// Clears the tables whose epoch just wrapped (one launch; exits at once when
// nothing wrapped).
__global__ void k_clear_if(const u32 *__restrict__ dep, u64 *table, int64_t tslots, u64 *ctable, int64_t cslots,
                           u64 *hub_sets, int64_t hub_slots) {
  const bool ct = dep[EP_CLR_TABLE] != 0, cc = dep[EP_CLR_CTABLE] != 0, ch = dep[EP_CLR_HUB] != 0;
  if (!ct && !cc && !ch) return;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  const int64_t i0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (ct)
    for (int64_t i = i0; i < tslots; i += stride) table[i] = 0;
  if (cc)
    for (int64_t i = i0; i < cslots; i += stride) ctable[i] = 0;
  if (ch)
    for (int64_t i = i0; i < hub_slots; i += stride) hub_sets[i] = 0;
}

// ---------------------------------------------------------------- utilities
__global__ void k_fill_u64(u64 *p, int64_t cnt, u64 val) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < cnt; i += (int64_t)gridDim.x * blockDim.x)
    p[i] = val;
}
__global__ void k_fill_i32(int *p, int64_t cnt, int val) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < cnt; i += (int64_t)gridDim.x * blockDim.x)
    p[i] = val;
}
__global__ void k_copy_i32(int *dst, const int *src, int64_t cnt) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < cnt; i += (int64_t)gridDim.x * blockDim.x)
    dst[i] = src[i];
}
// One source copied to up to MAX destinations (read once).
struct CopyDsts {
  static constexpr int MAX = 16;
  int32_t *d[MAX];
  int nd;
};
__global__ void k_copy_multi(CopyDsts dst, const int32_t *__restrict__ src, int64_t cnt) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  uintptr_t a = reinterpret_cast<uintptr_t>(src);
  for (int q = 0; q < dst.nd; ++q) a |= reinterpret_cast<uintptr_t>(dst.d[q]);
  int64_t done = 0;
  if ((a & 15) == 0) {
    // 16 bytes per thread and step where every start is 16-byte aligned
    const int64_t n4 = cnt >> 2;
    for (int64_t i = t; i < n4; i += stride) {
      const int4 v = reinterpret_cast<const int4 *>(src)[i];
      for (int q = 0; q < dst.nd; ++q) reinterpret_cast<int4 *>(dst.d[q])[i] = v;
    }
    done = n4 << 2;
  }
  for (int64_t i = done + t; i < cnt; i += stride) {
    const int32_t v = src[i];
    for (int q = 0; q < dst.nd; ++q) dst.d[q][i] = v;
  }
}

// Streaming copy, 16 bytes per thread per step (bandwidth probe).
__global__ void k_copy16(uint4 *__restrict__ dst, const uint4 *__restrict__ src, int64_t n16) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n16; i += (int64_t)gridDim.x * blockDim.x)
    dst[i] = src[i];
}

// Gather probe: every CSR entry reads its target's previous block through the
// same index and layout the signature kernels use (one streamed word, one
// random 4-byte gather), and nothing else.  Measures the random-gather rate
// the signature kernels are bounded by; one value per workgroup is written so
// the loads cannot be dropped.
template <class Src>
__global__ void __launch_bounds__(256) k_gather_probe(Src src, int64_t m, u32 *out, u32 omask) {
  u32 acc = 0;
  constexpr int U = 4;
  for (int64_t base = (int64_t)blockIdx.x * 256 * U; base < m; base += (int64_t)gridDim.x * 256 * U) {
    u32 v[U];
    const int cnt = (int)min<int64_t>(m - base, 256 * U);
    load_keys<u32, U, 256>(src, base, (int)threadIdx.x, cnt, v);
#pragma unroll
    for (int u = 0; u < U; ++u) acc ^= v[u];
  }
  acc = wave_sum_u32(acc);
  if ((threadIdx.x & (WAVE - 1)) == 0) atomicAdd(&out[blockIdx.x & omask], acc);
}

}  // namespace kb
