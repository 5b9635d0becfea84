// Host engine and C ABI of the k-bisimulation refinement library (gfx950).
//
// The engine owns no device memory: kbisim_create carves every buffer from
// the caller's workspace, validates the graph, computes P0 (vertex label-set
// equality), renumbers gather targets by in-degree and builds a static degree
// schedule; kbisim_refine enqueues k refinement steps on the caller's stream
// with no host synchronisation inside the loop (and, when enabled, replays
// the whole loop as a captured HIP graph).  A step that met a hash collision
// it could not settle in its one in-loop peeling round is detected after the
// final synchronisation and recomputed, from that step on, with peeling
// rounds driven by the host.  A batch is the disjoint union of many graphs
// refined by the same launches, with per-graph ids and counts.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <new>
#include <type_traits>
#include <utility>
#include <vector>

#include "../../include/kbisim.h"
#include "kernels.h"

using namespace kb;

namespace {

thread_local char g_hip_msg[256] = "";

constexpr size_t ALIGN = 256;
constexpr int CNT_STRIDE = STEP_ROW;  // device counters per step
constexpr int PERSIST_GRID = 2048;
constexpr int RES_GRID = 256;
constexpr int CLEAR_GRID = 2048;
constexpr int MIN_RANGE_EDGES = 1024;  // smallest tunable range capacity
constexpr int MIN_HUB_CHUNK = 2048;    // smallest tunable hub chunk
// Non-empty rows from which a full step groups by partition (9 launches more,
// no device-wide atomics) instead of through the table.  k = 10 calls, table /
// partition, in ms: nearly distinct keys, rows of 8 entries 0.5M 0.96 / 1.00, 1.0M
// 1.55 / 1.35, 1.8M 2.87 / 2.29, rows of 24 1.0M 2.38 / 2.14; RMAT rows of 25 1.0M
// 2.80 / 2.90, 1.85M 4.82 / 4.63, 3.5M (the 100M-edge graph) 9.31 / 8.48; RDF 11M
// 31.2 / 27.4.  Rows that share keys (unlabelled sparse graphs) stay ahead in the
// table: 1.4M 1.42 / 1.73, 2.8M 2.68 / 3.04, 42M 43.2 / 46.4; how many do is only
// known step by step, on the device.  The line lies between: distinct keys would
// gain from 0.8M on, RMAT rows from 1.4M, shared keys lose less the more rows.
constexpr int64_t GROUP_MIN = 1800000;
constexpr int MAX_GRAPH_CACHE = 8;
constexpr size_t READBACK_MAX = 1 << 16;  // bytes of counters and counts copied back at once

inline size_t align_up(size_t x) { return (x + ALIGN - 1) / ALIGN * ALIGN; }

uint64_t pow2_at_least(uint64_t x) {
  uint64_t p = 512;
  while (p < x) p <<= 1;
  return p;
}

struct Plan {
  size_t off_H, off_DC, off_rep, off_p0, off_vlist, off_clA, off_clB, off_ranges, off_lists, off_gcol, off_rank,
      off_gpid, off_zrep;
  size_t off_table, off_ctable, off_hacc, off_hcnt, off_chunks, off_parts, off_gchunks, off_poff;
  size_t off_status, off_hw, off_counters, off_dcounts, off_err, off_dep, off_hubsets, off_single, off_multi, off_nzv;
  size_t off_gid, off_ibuf, off_first, off_next, off_bcounts;  // batches only
  uint64_t tslots;
  int64_t max_ranges, max_lists, nhub_max, nchunk_max, npart_max, ngchunk_max, npoff_max, ntiles, hubset_slots;
  int ncounter_steps;
  size_t total;
};

Plan make_plan(int64_t n, int64_t m, int64_t nl, int kmax, int64_t num_graphs) {
  Plan p{};
  size_t at = 0;
  auto take = [&](size_t bytes) {
    size_t o = at;
    at = align_up(at + std::max<size_t>(bytes, 1));
    return o;
  };
  const size_t N = (size_t)std::max<int64_t>(n, 1);
  const int64_t big = std::max<int64_t>(std::max<int64_t>(m, nl), 1);
  p.tslots = pow2_at_least(2 * (uint64_t)N);
  // A range closes at a hub, when the next row would overflow it (the closed
  // range and that row hold more than its capacity together, and each row is
  // "next" once), when full of vertices, or at the end; rows above the
  // capacity form ranges of their own.  Bounds use the smallest capacity.
  p.max_ranges = big / (RANGE_DMAX + 1) + 2 * big / (MIN_RANGE_EDGES + 1) + 2 * big / MIN_RANGE_EDGES +
                 (int64_t)N / RANGE_VERTS + 24 + (int64_t)N / SCHED_CHUNK_V + 1;
  p.max_lists = big / (RANGE_DMAX + 1) + 8;
  p.nhub_max = big / (BLOCK_MAX + 1) + 1;
  p.nchunk_max = big / MIN_HUB_CHUNK + p.nhub_max + 1;
  p.npart_max = big / (HUB_PART_TARGET / 4) + 2 * p.nhub_max + 1;
  p.ngchunk_max = big / HUB_GCHUNK + p.nhub_max + 1;
  p.npoff_max = big / 16 + 4 * (HUB_PMAX + 1) + p.nchunk_max;
  p.ntiles = (int64_t)(N + 256 * SCAN_ITEMS_MIN - 1) / (256 * SCAN_ITEMS_MIN) + 1;
  p.hubset_slots = 2 * big + 64;
  p.ncounter_steps = kmax + 4;
  p.off_H = take(8 * N);
  p.off_DC = take(4 * N);
  p.off_rep = take(4 * N);
  p.off_p0 = take(4 * N);
  p.off_vlist = take(4 * N);
  p.off_clA = take(4 * N);
  p.off_clB = take(4 * N);
  p.off_ranges = take(sizeof(Range) * (size_t)p.max_ranges);
  p.off_lists = take(4 * (size_t)p.max_lists);
  p.off_gcol = take(4 * (size_t)std::max<int64_t>(m, 1));
  p.off_rank = take(4 * N);
  p.off_gpid = take(8 * N);
  p.off_zrep = take(8 * N);
  p.off_table = take(8 * p.tslots);
  p.off_ctable = take(8 * p.tslots);
  p.off_hacc = take(8 * (size_t)p.nhub_max);
  p.off_hcnt = take(4 * (size_t)p.nhub_max);
  p.off_chunks = take(sizeof(HubChunk) * (size_t)p.nchunk_max);
  p.off_parts = take(sizeof(HubPart) * (size_t)p.npart_max);
  p.off_gchunks = take(sizeof(HubGChunk) * (size_t)p.ngchunk_max);
  p.off_poff = take(4 * (size_t)p.npoff_max);
  p.off_status = take(4 * (size_t)p.ntiles);
  p.off_hw = take(sizeof(HeadWord) * (N / 64 + 1));
  p.off_counters = take(4 * (size_t)CNT_STRIDE * (size_t)p.ncounter_steps);
  p.off_dcounts = take(8 * (size_t)p.ncounter_steps);
  p.off_err = take(16);
  p.off_dep = take(64);
  p.off_hubsets = take(8 * (size_t)p.hubset_slots);
  p.off_single = take(2 * N);
  p.off_multi = take(4 * N);
  p.off_nzv = take(4 * N);
  if (num_graphs > 0) {
    p.off_gid = take(4 * N);
    p.off_ibuf = take(8 * N);
    p.off_first = take(8 * (size_t)(num_graphs + 1));
    p.off_next = take(8 * (size_t)num_graphs);
    p.off_bcounts = take(8 * (size_t)num_graphs * (size_t)std::max(kmax, 1));
  }
  p.total = at;
  return p;
}

// Static degree schedule of one row structure (graph rows or label-set rows),
// built at create time (k_sched_chunks); degrees never change across iterations.
struct Schedule {
  int range_edges = RANGE_EDGES;  // range capacity of this schedule (1024 or 2048)
  int nranges = 0;  // multi-vertex ranges (at most range_edges entries)
  int nbig = 0;     // single-row ranges of range_edges < deg <= RANGE_DMAX
  int nrow8 = 0;    // single-row ranges of RANGE_DMAX < deg <= ROW_MAX (after the nbig ones)
  int nrow20 = 0;   // single-row ranges of ROW_MAX < deg <= ROW_MAX_NARROW, 32-bit keys only (after those)
  int nhub = 0, hub_off = 0;
  int nchunks = 0, nparts = 0, ngchunks = 0;
  int64_t gset_begin = 0, gset_end = 0;  // global hash sets of very large hubs
  int64_t nonempty = 0;                   // rows with at least one entry
  int64_t nlong = 0;                      // rows of more than SMALL_MAX entries
  const int *nzv = nullptr;               // their vertices in order (graph rows), or null
  int64_t info[8] = {0, 0, 0, 0, 0, 0, 0, 0};  // vertices, entries per tier
};

struct Tuning {
  int range_edges = 0;  // 0: by key width (range_cap)
  int hub_chunk = 2048;
  int hub_part_target = HUB_PART_TARGET;
  int key_bits = 0;  // LDS set keys: 0 = 32-bit (exact where pairs fit, else hashed), 32 = hashed, 64 = 64-bit
  int hub_parts_cap = HUB_PMAX;  // most partitions per staged hub (a smaller cap is a test knob)
  int scan_items = SCAN_ITEMS;   // vertices per thread in the numbering scan: 8 or 16
  int64_t group_min = GROUP_MIN;  // non-empty rows from which full steps group by partition
  u32 group_mask = GROUP_MASK;    // bits of the hash that choose a bucket there (fewer: a test knob)
  int group_mean_bits = GROUP_BITS;  // bucket bits that the sub-passes begun with are planned for
  int gfilter_min = GFILTER_MIN_DIRTY;  // dirty vertices from which update steps use the global filter
};

struct GraphKey {
  const void *start;
  int k;
  std::vector<const void *> outs;
  bool operator<(const GraphKey &o) const {
    if (start != o.start) return start < o.start;
    if (k != o.k) return k < o.k;
    return outs < o.outs;
  }
};

}  // namespace

struct kbisim_ctx {
  kbisim_graph g;
  int kmax;
  hipStream_t stream;
  Plan plan;
  Tuning tune;
  char *ws;
  u64 *H, *table, *ctable, *hacc, *hubsets, *zrep;
  int64_t cslots = 0;    // slots of the peeling table: half of its space, nzrow has the rest
  u32 *nzrow = nullptr;  // low word of the offset of every non-empty row (in the order of nzv)
  u32 *DC, *hcnt, *err, *tiles, *dep;
  const u32 *cur = nullptr;  // the epochs of the step being enqueued: dep, or its row (k_prepare_steps)
  HeadWord *hw;
  int *rep, *p0, *vlist, *clA, *clB, *lists, *counters, *poff, *gcol, *rank, *gpid[2], *nzv;
  int64_t *dcounts;
  Range *ranges;
  HubChunk *chunks;
  HubPart *parts;
  HubGChunk *gchunks;
  Schedule sched;  // graph rows
  u64 hmask = ~0ULL;
  u32 kmask = 0xFFFFFFFFu;  // bits kept of hashed set keys (test knob)
  u64 tmask_steps = 0;   // grouping-table mask of refinement steps (sized by vertices with edges)
  size_t table_dirty = 0;  // bytes at the start of the grouping table's space used by partitioned steps
  bool work_eff = false;  // skip singleton blocks, stop at the fixpoint
  int we_steps = 0;       // steps computed by the last work-efficient call
  unsigned char *single[2] = {nullptr, nullptr};  // singleton flags of the last two partitions
  u32 *multi = nullptr;  // stamps of heads that have a non-head member
  u32 prof_mask = ~0u;   // kernel kinds timed by the profiler
  bool narrow = false;  // 32-bit LDS keys
  bool hashed = false;  // ... that hash the pair (it does not fit 31 bits, or 32-bit keys were asked for)
  u32 pb = 31;
  u32 max_label = 0;    // largest edge label (0 without labels)
  bool packed = false;  // edge labels packed above the target ranks in gcol
  u32 rbits = 31;       // bits of the target rank in gcol
  int32_t *glab = nullptr;  // separate labels in the order of the sorted rows (else the caller's)
  int64_t p0_count = 0;
  // batches
  int64_t num_graphs = 0;
  int *gid = nullptr, *ibuf[2] = {nullptr, nullptr};
  int64_t *first = nullptr, *next = nullptr, *bcounts = nullptr;
  // per-kernel profiling
  bool prof = false;
  std::vector<hipEvent_t> ev_pool;
  size_t ev_used = 0;
  struct Pending {
    int kind;
    size_t a, b;
  };
  std::vector<Pending> ev_pending;
  double prof_ms[KBISIM_NKERNELS] = {0};
  int64_t prof_n[KBISIM_NKERNELS] = {0};
  // captured refinement loops
  bool use_graphs = false;
  std::map<GraphKey, hipGraphExec_t> graphs;
  // incremental updates: refine calls from P0 cache their chain (key hashes,
  // distinct counts and minimum-vertex block names per step) in the caller's
  // state buffer; updates recompute only what edits can have changed
  bool incr = false;
  int incr_k = 0;  // steps of the cached chain
  struct {
    u64 *Hc;
    u32 *DCc;
    int32_t *MVc;
    uint16_t *FKc;  // filter bit of each vertex's cached key, per step
    int64_t *tptr;
    int32_t *tcol;
    int32_t *names[2];
    unsigned char *edited, *flag, *dirty, *skip;
    int *small, *large, *psmall, *plarge, *changed, *cnt;
    int32_t *bname;   // block names of an update step, by representative
    int32_t *keep;    // cached names kept by blocks of changed vertices, by representative
    unsigned char *claimed;  // cached names taken by blocks with an unchanged member
    int *heavy;       // changed vertices with long in-rows
    u32 *touch;  // bitmap of the cached blocks (by minimum vertex) that can change in this step
    int *lk;               // the dirty vertices, then these and the clean members of touched blocks
    u32 *filter;           // bit filter of the dirty keys
    u32 *gfilter;          // the larger global filter (GFILTER_BITS) used with many dirty keys
    // edited rows longer than LIST_BIG: one global set each (chunks of HUB_GCHUNK)
    int *huge;
    HubGChunk *huge_chunks;
    u64 *huge_acc;
    u32 *huge_cnt;
    int nhuge = 0, nhuge_chunks = 0;
    // edited rows of LIST_BIG < length <= ROW_MAX (and, with 32-bit keys,
    // <= ROW_MAX_NARROW after them): one row-kernel workgroup each
    Range *erows;
    int nerows8 = 0, nerows20 = 0;
    int64_t huge_set_begin = 0, huge_set_slots = 0;
    int64_t huge_cap = 0, huge_chunk_cap = 0;
    int64_t nrows = 0;  // edited rows listed by the caller
    u64 *zrep;        // empty-signature representatives by block name (names reach 2n)
  } is{};
};

struct kbisim_batch {
  kbisim_ctx *c;
};

namespace {

int hip_fail(hipError_t e) {
  snprintf(g_hip_msg, sizeof g_hip_msg, "HIP error %d: %s", (int)e, hipGetErrorString(e));
  return KBISIM_EHIP;
}

#define HIP_TRY(expr)                          \
  do {                                         \
    hipError_t _e = (expr);                    \
    if (_e != hipSuccess) return hip_fail(_e); \
  } while (0)

#define LAUNCH_CHECK() HIP_TRY(hipGetLastError())

inline unsigned blocks_for(int64_t items, int per) { return (unsigned)((items + per - 1) / per); }

// Workgroups of the radix kernels (see radix_tile).
unsigned radix_grid(int64_t ntiles) { return (unsigned)((ntiles + XCDS - 1) / XCDS * XCDS); }

// Range check of cnt int32 values on stream s, and their maximum into
// *max_out unless null (see k_validate_vals).
void validate_vals(hipStream_t s, int64_t cnt, const int32_t *vals, int64_t upper, u32 *err, u32 bit,
                   u32 *max_out = nullptr) {
  if (cnt <= 0) return;
  const unsigned g = (unsigned)std::min<int64_t>(VALIDATE_GRID, blocks_for(cnt / 4 + 1, 256));
  if (max_out) k_validate_vals<true><<<g, 256, 0, s>>>(cnt, vals, upper, err, bit, max_out);
  else k_validate_vals<false><<<g, 256, 0, s>>>(cnt, vals, upper, err, bit, nullptr);
}

// ---- per-kernel profiling: events around each launch, resolved after syncs.
hipEvent_t prof_event(kbisim_ctx *c) {
  if (c->ev_used == c->ev_pool.size()) {
    hipEvent_t e;
    if (hipEventCreate(&e) != hipSuccess) return nullptr;
    c->ev_pool.push_back(e);
  }
  return c->ev_pool[c->ev_used++];
}

struct ProfScope {
  kbisim_ctx *c;
  int kind;
  size_t start = (size_t)-1;
  ProfScope(kbisim_ctx *c_, int kind_) : c(c_), kind(kind_) {
    if (!c->prof || !((c->prof_mask >> kind) & 1u)) return;
    hipEvent_t e = prof_event(c);
    if (!e) return;
    start = c->ev_used - 1;
    (void)hipEventRecord(e, c->stream);
  }
  ~ProfScope() {
    if (start == (size_t)-1) return;
    hipEvent_t e = prof_event(c);
    if (!e) return;
    (void)hipEventRecord(e, c->stream);
    c->ev_pending.push_back({kind, start, c->ev_used - 1});
  }
};

// Fold pending event pairs into the sums (the stream must be synchronised).
void prof_collect(kbisim_ctx *c) {
  for (auto &p : c->ev_pending) {
    float ms = 0.f;
    if (hipEventElapsedTime(&ms, c->ev_pool[p.a], c->ev_pool[p.b]) == hipSuccess) {
      c->prof_ms[p.kind] += ms;
      c->prof_n[p.kind] += 1;
    }
  }
  c->ev_pending.clear();
  c->ev_used = 0;
}

int fill_u64(kbisim_ctx *c, u64 *p, int64_t cnt, u64 val) {
  if (cnt <= 0) return 0;
  ProfScope ps(c, KBISIM_K_FILL);
  unsigned g = (unsigned)std::min<int64_t>(blocks_for(cnt, 256), 65536);
  k_fill_u64<<<g, 256, 0, c->stream>>>(p, cnt, val);
  LAUNCH_CHECK();
  return 0;
}

int fill_i32(kbisim_ctx *c, int *p, int64_t cnt, int val) {
  if (cnt <= 0) return 0;
  ProfScope ps(c, KBISIM_K_FILL);
  unsigned g = (unsigned)std::min<int64_t>(blocks_for(cnt, 256), 65536);
  k_fill_i32<<<g, 256, 0, c->stream>>>(p, cnt, val);
  LAUNCH_CHECK();
  return 0;
}

// Advance the device-side epochs named in `mask` and clear the tables whose
// epoch wrapped.
int advance(kbisim_ctx *c, u32 mask, const Schedule &s) {
  ProfScope ps(c, KBISIM_K_FILL);
  k_advance<<<1, 64, 0, c->stream>>>(c->dep, mask);
  LAUNCH_CHECK();
  k_clear_if<<<CLEAR_GRID, 256, 0, c->stream>>>(c->dep, c->table, (int64_t)c->plan.tslots, c->ctable, c->cslots,
                                                c->hubsets + s.gset_begin, s.gset_end - s.gset_begin);
  LAUNCH_CHECK();
  return 0;
}

int read_err(kbisim_ctx *c, u32 *out) {
  HIP_TRY(hipMemcpyAsync(out, c->err, sizeof(u32), hipMemcpyDeviceToHost, c->stream));
  HIP_TRY(hipStreamSynchronize(c->stream));
  return 0;
}

// Range capacity: the tuned one, else 2048 entries with 32-bit set keys and
// 1024 with 64-bit keys (the larger LDS set would cost occupancy).
int range_cap(const kbisim_ctx *c, bool wide_keys) {
  if (c->tune.range_edges) return c->tune.range_edges;
  return wide_keys ? 1024 : 2048;
}

int hub_parts_for(const Tuning &t, int64_t d) {
  int P = 1;
  while ((int64_t)P * t.hub_part_target < d && P < t.hub_parts_cap) P <<= 1;
  return P;
}

// Edge labels read from their own array (not packed into gcol, and present).
bool separate_labels(const kbisim_ctx *c) { return !c->packed && c->g.elabel != nullptr; }
// The separate labels the kernels read: the rank-sorted copy, if made.
const int32_t *sep_labels(const kbisim_ctx *c) { return c->glab ? c->glab : c->g.elabel; }

// A step's numbering: head words and the tile prefixes of the heads in
// vertex order (k_head_words, k_tile_scan); the block count to count_dev.
// The assign kernels then read every vertex's dense id through the result.
// With scan_tiles, up to 256 tiles are left unscanned and their number put
// there, for k_assign.
int numbering_words(kbisim_ctx *c, int n, int64_t *count_dev, HeadIds *ids, int *scan_tiles = nullptr) {
  const int items = c->tune.scan_items;
  const int ntiles = (int)blocks_for(n, 256 * items);
  if (items == 8) k_head_words<8><<<(unsigned)ntiles, 256, 0, c->stream>>>(n, c->rep, c->hw, c->tiles);
  else k_head_words<16><<<(unsigned)ntiles, 256, 0, c->stream>>>(n, c->rep, c->hw, c->tiles);
  LAUNCH_CHECK();
  *ids = HeadIds{c->hw, c->tiles, items == 8 ? 11 : 12};
  if (scan_tiles && ntiles <= 256) {
    *scan_tiles = ntiles;
    return 0;
  }
  k_tile_scan<<<1, 1024, 0, c->stream>>>(ntiles, c->tiles, count_dev);
  LAUNCH_CHECK();
  return 0;
}

// Order the entries of every row of the range and row tiers, and of every
// staged hub chunk, by target rank (results do not depend on the order
// inside a row).  Separate edge labels move with their entries, in a copy
// kept in the unused tail of the hub staging region; when the tail is too
// small, such graphs stay unsorted.  PAY: that copy is in use.
template <bool PAY>
int sort_rows_impl(kbisim_ctx *c, const Schedule &s, u32 *lab) {
  u32 *g = reinterpret_cast<u32 *>(c->gcol);
  if (s.nranges) {
    if (s.range_edges == 1024)
      k_sort_ranges<1024, PAY><<<(unsigned)s.nranges, 256, 0, c->stream>>>(g, lab, c->ranges, c->nzrow, c->rbits);
    else
      k_sort_ranges<2048, PAY><<<(unsigned)s.nranges, 256, 0, c->stream>>>(g, lab, c->ranges, c->nzrow, c->rbits);
    LAUNCH_CHECK();
  }
  const Range *rows = c->ranges + s.nranges;
  if (s.nbig) {
    k_sort_rows<RANGE_DMAX, PAY><<<(unsigned)s.nbig, 1024, 0, c->stream>>>(g, lab, rows, c->rbits);
    LAUNCH_CHECK();
  }
  if (s.nrow8) {
    k_sort_rows<ROW_MAX, PAY><<<(unsigned)s.nrow8, 1024, 0, c->stream>>>(g, lab, rows + s.nbig, c->rbits);
    LAUNCH_CHECK();
  }
  if (s.nrow20) {
    k_sort_rows<19 * 1024, PAY><<<(unsigned)s.nrow20, 1024, 0, c->stream>>>(g, lab, rows + s.nbig + s.nrow8, c->rbits);
    LAUNCH_CHECK();
  }
  if (s.nchunks) {
    k_sort_hub_chunks<HUB_CHUNK_MAX, PAY><<<(unsigned)s.nchunks, 1024, 0, c->stream>>>(
        g, lab, c->g.row_ptr, c->lists + s.hub_off, c->chunks, c->rbits);
    LAUNCH_CHECK();
  }
  return 0;
}

int sort_long_rows(kbisim_ctx *c, const Schedule &s) {
  if (!separate_labels(c)) return sort_rows_impl<false>(c, s, nullptr);
  const int64_t m = c->g.m;
  const int64_t need = (m + 1) / 2 + 1;  // u64 slots for m int32 labels
  if (m == 0 || s.gset_end + need > c->plan.hubset_slots) return 0;
  int32_t *lab = reinterpret_cast<int32_t *>(c->hubsets + (c->plan.hubset_slots - need));
  HIP_TRY(hipMemcpyAsync(lab, c->g.elabel, 4 * (size_t)m, hipMemcpyDeviceToDevice, c->stream));
  c->glab = lab;
  return sort_rows_impl<true>(c, s, reinterpret_cast<u32 *>(lab));
}

// Hub plan (staged chunks and partitions, global-set chunks) of a schedule
// whose range lists are on the device and counted in s.
// staged_max: longest hub staged in partitions (longer hubs use a global set).
// Synchronises when there are hubs.
int plan_hubs(kbisim_ctx *c, Schedule &s, const std::vector<int> &hubs, const std::vector<int64_t> &hub_deg,
              int64_t staged_max) {
  const Tuning &t = c->tune;
  const int64_t nranges_total = (int64_t)s.nranges + s.nbig + s.nrow8 + s.nrow20;
  // hubs: staged (partitioned) unless very large or out of offset space
  std::vector<HubChunk> chunks;
  std::vector<HubPart> parts;
  std::vector<HubGChunk> gchunks;
  std::vector<char> is_staged(hubs.size(), 0);
  int64_t stage_at = 0, poff_at = 0;
  for (size_t i = 0; i < hubs.size(); ++i) {
    const int64_t d = hub_deg[i];
    const int64_t C = (d + t.hub_chunk - 1) / t.hub_chunk;
    const int P = hub_parts_for(t, d);
    const bool staged = d <= staged_max && C <= HUB_PMAX && poff_at + C * (P + 1) <= c->plan.npoff_max;
    if (!staged) continue;
    HubPart hp;
    hp.hub = (int)i;
    hp.chunk0 = (int)chunks.size();
    hp.nchunks = (int)C;
    for (int64_t k = 0; k < C; ++k) {
      HubChunk hc;
      hc.hub = (int)i;
      hc.parts = P;
      hc.b = k * t.hub_chunk;
      hc.e = std::min<int64_t>(d, (k + 1) * t.hub_chunk);
      hc.stage = stage_at;
      hc.poff = poff_at;
      stage_at += t.hub_chunk;
      poff_at += P + 1;
      chunks.push_back(hc);
    }
    for (int q = 0; q < P; ++q) {
      hp.part = q;
      parts.push_back(hp);
    }
    is_staged[i] = 1;
    s.info[4] += 1;
    s.info[5] += d;
  }
  // global sets of the remaining hubs follow the staging areas
  s.gset_begin = stage_at;
  int64_t gset_at = stage_at;
  for (size_t i = 0; i < hubs.size(); ++i) {
    if (is_staged[i]) continue;
    const int64_t d = hub_deg[i];
    const int64_t size = 2 * d;
    for (int64_t b = 0; b < d; b += HUB_GCHUNK) {
      HubGChunk g;
      g.hub = (int)i;
      g.pad = 0;
      g.b = b;
      g.e = std::min<int64_t>(d, b + HUB_GCHUNK);
      g.set_off = gset_at;
      g.set_size = size;
      gchunks.push_back(g);
    }
    gset_at += size;
    s.info[6] += 1;
    s.info[7] += d;
  }
  s.gset_end = gset_at;
  if (nranges_total > c->plan.max_ranges || gset_at > c->plan.hubset_slots ||
      (int64_t)chunks.size() > c->plan.nchunk_max || (int64_t)parts.size() > c->plan.npart_max ||
      (int64_t)gchunks.size() > c->plan.ngchunk_max || (int64_t)hubs.size() > c->plan.nhub_max ||
      (int64_t)hubs.size() > c->plan.max_lists)
    return KBISIM_EINTERNAL;
  s.hub_off = 0;
  s.nhub = (int)hubs.size();
  s.nchunks = (int)chunks.size();
  s.nparts = (int)parts.size();
  s.ngchunks = (int)gchunks.size();
  if (!chunks.empty())
    HIP_TRY(hipMemcpyAsync(c->chunks, chunks.data(), sizeof(HubChunk) * chunks.size(), hipMemcpyHostToDevice,
                           c->stream));
  if (!parts.empty())
    HIP_TRY(hipMemcpyAsync(c->parts, parts.data(), sizeof(HubPart) * parts.size(), hipMemcpyHostToDevice, c->stream));
  if (!gchunks.empty())
    HIP_TRY(hipMemcpyAsync(c->gchunks, gchunks.data(), sizeof(HubGChunk) * gchunks.size(), hipMemcpyHostToDevice,
                           c->stream));
  int rc = 0;
  if (!s.nhub) return 0;
  if ((rc = fill_u64(c, c->hacc, s.nhub, 0))) return rc;
  if ((rc = fill_i32(c, (int *)c->hcnt, s.nhub, 0))) return rc;
  if ((rc = fill_u64(c, c->hubsets + s.gset_begin, s.gset_end - s.gset_begin, 0))) return rc;
  HIP_TRY(hipStreamSynchronize(c->stream));
  return 0;
}

// Static schedule of the rows of `ptr`, built on the device in two parts.
// sched_enqueue launches the kernels (range lists, hub list, non-empty rows) and leaves the totals on the device;
// sched_finish takes the totals, once copied to the host, and plans the hubs.
// row_max: longest row with a workgroup of its own (longer rows are hubs).
// Scratch: c->vlist (68 bytes per chunk); the totals go to
// `totals` (SCHED_TOTALS words).
int sched_enqueue(kbisim_ctx *c, const int64_t *ptr, int range_edges, int64_t row_max, int64_t *totals) {
  const int64_t n = c->g.n;
  const int nch = (int)((n + SCHED_CHUNK_V - 1) / SCHED_CHUNK_V);
  int64_t *sums = reinterpret_cast<int64_t *>(c->vlist);
  int *cnt = reinterpret_cast<int *>(sums + 6 * (size_t)nch);
  if (nch == 1) {
    k_sched_chunks<SCHED_SINGLE><<<1, SCHED_THREADS, 0, c->stream>>>(ptr, n, 1, range_edges, row_max, nullptr, nullptr,
                                                                     totals, c->ranges, c->lists, c->nzv, c->nzrow);
    LAUNCH_CHECK();
    return 0;
  }
  k_sched_chunks<SCHED_COUNT><<<(unsigned)nch, SCHED_THREADS, 0, c->stream>>>(
      ptr, n, nch, range_edges, row_max, cnt, sums, nullptr, nullptr, nullptr, nullptr, nullptr);
  k_sched_scan<<<1, SCHED_TOTALS * WAVE, 0, c->stream>>>(nch, cnt, sums, totals);
  k_sched_chunks<SCHED_WRITE><<<(unsigned)nch, SCHED_THREADS, 0, c->stream>>>(
      ptr, n, nch, range_edges, row_max, cnt, sums, totals, c->ranges, c->lists, c->nzv, c->nzrow);
  LAUNCH_CHECK();
  return 0;
}

int sched_finish(kbisim_ctx *c, const int64_t *ptr, Schedule &s, int range_edges, int64_t staged_max,
                 const int64_t *tot, const int *nzv) {
  s = Schedule{};
  s.range_edges = range_edges;
  s.nranges = (int)tot[0];
  s.nbig = (int)tot[1];
  s.nrow8 = (int)tot[2];
  s.nrow20 = (int)tot[3];
  for (int i = 0; i < 4; ++i) s.info[i] = tot[5 + i];
  s.nonempty = tot[9];
  s.nlong = tot[10];
  s.nzv = nzv;
  const int nh = (int)tot[4];
  std::vector<int> hubs((size_t)nh);
  std::vector<int64_t> hub_deg((size_t)nh);
  if (nh > 0) {
    // the hubs' degrees, in the key-hash array (8n bytes, unused at create time; nh <= n)
    int64_t *deg = reinterpret_cast<int64_t *>(c->H);
    k_row_degrees<<<blocks_for(nh, 256), 256, 0, c->stream>>>(nh, c->lists, ptr, deg);
    LAUNCH_CHECK();
    HIP_TRY(hipMemcpyAsync(hubs.data(), c->lists, 4 * (size_t)nh, hipMemcpyDeviceToHost, c->stream));
    HIP_TRY(hipMemcpyAsync(hub_deg.data(), deg, 8 * (size_t)nh, hipMemcpyDeviceToHost, c->stream));
    HIP_TRY(hipStreamSynchronize(c->stream));
  }
  return plan_hubs(c, s, hubs, hub_deg, staged_max);
}

// Bits needed for x (0 for 0).
int bit_width(uint64_t x) {
  int b = 0;
  while (b < 64 && (x >> b) != 0) ++b;
  return b;
}

// Exclusive scan of cnt[0..len) into out[0..len] (64-bit), on `s`.
int scan64(hipStream_t s, int64_t len, const int *cnt, int64_t *tiles, int64_t *out) {
  const int64_t nt = (len + SCAN_TILE - 1) / SCAN_TILE;
  k_sum_tiles64<<<(unsigned)nt, 256, 0, s>>>(len, cnt, tiles);
  if (nt <= 256) {
    k_write_ptr64<true><<<(unsigned)nt, 256, 0, s>>>(len, cnt, tiles, out, nullptr);
  } else {
    k_scan_tiles64<<<1, 256, 0, s>>>(nt, tiles);
    k_write_ptr64<false><<<(unsigned)nt, 256, 0, s>>>(len, cnt, tiles, out, nullptr);
  }
  HIP_TRY(hipGetLastError());
  return 0;
}

// Stable sort of m keys by their bits [lo, hi), 8 bits per pass, between ka and
// kb; on return ka points to the sorted keys.
template <class K>
int radix_sort(hipStream_t s, int64_t m, K *&ka, K *&kb, int lo, int hi, int64_t rtiles, int *hist, int64_t *tiles,
               int64_t *offs) {
  int rc = 0;
  for (int shift = lo; shift < hi; shift += 8) {
    k_radix_hist<<<radix_grid(rtiles), RADIX_THREADS, 0, s>>>(m, ka, shift, rtiles, hist);
    HIP_TRY(hipGetLastError());
    if ((rc = scan64(s, 256 * rtiles, hist, tiles, offs))) return rc;
    k_radix_scatter<<<radix_grid(rtiles), RADIX_THREADS, 0, s>>>(m, ka, shift, rtiles, offs, kb);
    HIP_TRY(hipGetLastError());
    std::swap(ka, kb);
  }
  return 0;
}
// Entries per target of the context's graph into indeg.  Graphs of at least
// INDEG_SORT_MIN entries partition the targets first (k_bucket_count): 24M
// entries 0.95 -> 0.17 ms, 40M 1.65 -> 0.27.  Not those of at most INDEG_FEW
// vertices, where a chunk adds to so few counters that its atomics are cheap
// (200M entries, create without / with the partition: 2 vertices 3.8 / 7.9 ms,
// 4: 6.0 / 7.6, 8: 10.3 / 7.3).  Scratch: the hub-set space, not yet in use.
constexpr int64_t INDEG_SORT_MIN = (int64_t)1 << 21, INDEG_FEW = 4;
int in_degrees(kbisim_ctx *c, int *indeg) {
  const int64_t n = c->g.n, m = c->g.m;
  hipStream_t s = c->stream;
  int rc = 0;
  if (m < INDEG_SORT_MIN || n <= INDEG_FEW) {
    if ((rc = fill_i32(c, indeg, n, 0))) return rc;
    if (m > 0) {
      k_indegree<<<(unsigned)std::min<int64_t>(blocks_for(m, INDEG_CHUNK), 1 << 16), 256, 0, s>>>(m, c->g.col, indeg);
      LAUNCH_CHECK();
    }
    return 0;
  }
  // buckets of 2^shift targets: 8 high bits (one pass) while 2^15 counters
  // hold a bucket, else 16 (two passes)
  const int bits = std::max(9, bit_width((uint64_t)(n - 1)));
  const int passes = bits <= 23 ? 1 : 2;
  const int shift = bits - 8 * passes;
  const int64_t nb = ((n - 1) >> shift) + 1;
  const int64_t rtiles = (m + RADIX_TILE - 1) / RADIX_TILE, hist_n = 256 * rtiles;
  char *w = (char *)c->hubsets;
  size_t at = 0;
  auto take = [&](size_t bytes) {
    char *p = w + at;
    at = align_up(at + bytes);
    return p;
  };
  u32 *ka = (u32 *)take(4 * (size_t)m), *kb = (u32 *)take(4 * (size_t)m);
  int *hist = (int *)take(4 * (size_t)hist_n);
  int64_t *offs = (int64_t *)take(8 * (size_t)(hist_n + 1));
  int64_t *tiles = (int64_t *)take(8 * (size_t)(hist_n / SCAN_TILE + 1));
  int64_t *starts = (int64_t *)take(8 * (size_t)nb);
  int *rest = (int *)take(4);
  if (at > 8 * (size_t)c->plan.hubset_slots) return KBISIM_EINTERNAL;
  u32 *from = reinterpret_cast<u32 *>(const_cast<int32_t *>(c->g.col)), *to = ka;  // the caller's array is only read
  for (int p = 0; p < passes; ++p) {
    u32 *next = to == ka ? kb : ka;
    if ((rc = radix_sort(s, m, from, to, shift + 8 * p, shift + 8 * p + 8, rtiles, hist, tiles, offs))) return rc;
    to = next;  // radix_sort left the result in `from`
  }
  if ((rc = fill_i32(c, rest, 1, 0))) return rc;
  // A bucket of several times the mean is finished by the whole grid (the mean
  // over 256 buckets at least: a graph of few vertices has fewer, and the cap
  // then let one workgroup count up to all entries; 200M entries of 40 vertices:
  // create 7.0 -> 5.7 ms, of two: 98.6 -> 7.9).
  const int64_t cap = std::max<int64_t>(1 << 16, 8 * (m / std::max<int64_t>(nb, 256)));
  if (shift <= 13)
    k_bucket_count<13><<<(unsigned)nb, BUCKET_THREADS, 0, s>>>(m, n, from, (u32)shift, cap, indeg, starts, rest);
  else
    k_bucket_count<15><<<(unsigned)nb, BUCKET_THREADS, 0, s>>>(m, n, from, (u32)shift, cap, indeg, starts, rest);
  LAUNCH_CHECK();
  k_indegree_rest<<<(unsigned)std::min<int64_t>(blocks_for(m, INDEG_CHUNK), 8192), 256, 0, s>>>(m, from, (u32)shift,
                                                                                            cap, starts, rest, indeg);
  LAUNCH_CHECK();
  return 0;
}

// Rank vertices by decreasing class of in-degree (ties by vertex id) and renumber the
// targets of every CSR entry: gcol[e] = rank[col[e]].  Vertices no entry
// names get rank -1: they are never gathered.  A stable LSD radix sort of
// (class key, vertex) on the device; the grouping tables serve as
// scratch, so this runs before they are cleared.
int build_rank(kbisim_ctx *c) {
  const int64_t n = c->g.n, m = c->g.m;
  if (n == 0) return 0;
  int *indeg = c->vlist;  // scratch
  int rc = in_degrees(c, indeg);
  if (rc) return rc;
  u64 *ka = c->table, *kb = c->table + n;  // 8 * tslots >= 16 n bytes
  const int64_t rtiles = (n + RADIX_TILE - 1) / RADIX_TILE, hist_n = 256 * rtiles;
  int *hist = (int *)c->ctable;
  int64_t *offs = (int64_t *)(c->ctable) + (hist_n + 1) / 2 + 1;
  int64_t *tiles = offs + hist_n + 2;
  if ((size_t)((char *)(tiles + (hist_n + SCAN_TILE - 1) / SCAN_TILE + 1) - (char *)c->ctable) > 8 * c->plan.tslots)
    return KBISIM_EINTERNAL;
  k_rank_keys<<<(unsigned)std::min<int64_t>(blocks_for(n, 256), 1 << 16), 256, 0, c->stream>>>(n, indeg, ka);
  LAUNCH_CHECK();
  // stable passes over key bits [32, 32 + bits)
  auto radix_passes = [&](int bits) { return radix_sort(c->stream, n, ka, kb, 32, 32 + bits, rtiles, hist, tiles, offs); };
  if ((rc = radix_passes(RANK_KEYBITS))) return rc;
  if (c->num_graphs > 1) {
    // In a batch, ranks stay inside each graph's vertex range (ordered by
    // in-degree within the graph): a graph's gathers then touch its own
    // part of the partition only, instead of the whole union's.
    k_rank_gid_keys<<<(unsigned)std::min<int64_t>(blocks_for(n, 256), 1 << 16), 256, 0, c->stream>>>(n, ka, c->gid,
                                                                                                    kb);
    LAUNCH_CHECK();
    std::swap(ka, kb);
    if ((rc = radix_passes(bit_width((uint64_t)(c->num_graphs - 1))))) return rc;
  }
  k_rank_from_sorted<<<(unsigned)std::min<int64_t>(blocks_for(n, 256), 1 << 16), 256, 0, c->stream>>>(n, ka, indeg,
                                                                                                 c->rank);
  LAUNCH_CHECK();
  if (m > 0) {
    k_remap<<<(unsigned)std::min<int64_t>(blocks_for(m, 256), 1 << 16), 256, 0, c->stream>>>(
        m, c->g.col, c->rank, c->gcol, c->packed ? c->g.elabel : nullptr, c->rbits);
    LAUNCH_CHECK();
  }
  return 0;
}

// One peeling round over `in_list` (count at in_cnt) into out_list/out_cnt.
template <class Src>
int peel_round(kbisim_ctx *c, const Src &src, int *in_cnt, int *in_list, int *out_cnt, int *out_list) {
  ProfScope ps(c, KBISIM_K_PEEL);
  k_res_insert<<<RES_GRID, 256, 0, c->stream>>>(in_cnt, in_list, c->H, c->ctable, (u64)c->cslots - 1, c->cur);
  LAUNCH_CHECK();
  k_res_verify<Src><<<RES_GRID, 256, 0, c->stream>>>(src, in_cnt, in_list, c->H, c->DC, c->ctable,
                                                     (u64)c->cslots - 1, c->cur, c->rep, out_cnt, out_list, c->err);
  LAUNCH_CHECK();
  return 0;
}

// Refinement steps group only vertices with edges (the rest go by previous
// block alone), so their table span is sized by that count; P0 uses it all.
template <class Src>
u64 table_mask(const kbisim_ctx *c) {
  if constexpr (Src::GRAPH) return c->tmask_steps;
  return c->plan.tslots - 1;
}

// Up to two ranges per CU are taken by workgroups of 1024 threads: each is one
// latency chain, which more threads shorten.  Random graphs of 8 edges a
// vertex, 10 steps, 256 / 1024 threads: 39 ranges 403 / 338 us, 250 ranges
// 523 / 469, 500 ranges 599 / 550; but 1000 ranges 721 / 750 and 2000 ranges
// 1075 / 1120, where 1024 threads leave too few ranges in flight.
constexpr int FEW_RANGES = 512, FEW_THREADS = 1024;

template <class Src, class K, bool SKIP>
int launch_range_kernel(kbisim_ctx *c, const Src &src, const Schedule &s, KeySink sink, const unsigned char *skip) {
  ProfScope ps(c, KBISIM_K_SIG_RANGE);
  if constexpr (!SKIP) {
    if (s.range_edges == 2048 && s.nranges <= FEW_RANGES) {
      k_sig_range<Src, 2048, K, false, FEW_THREADS><<<(unsigned)s.nranges, FEW_THREADS, 0, c->stream>>>(
          src, c->ranges, c->H, c->DC, sink, c->cur, c->hmask, c->nzv, c->nzrow, skip);
      LAUNCH_CHECK();
      return 0;
    }
  }
  if (s.range_edges == 1024)
    k_sig_range<Src, 1024, K, SKIP><<<(unsigned)s.nranges, 256, 0, c->stream>>>(
        src, c->ranges, c->H, c->DC, sink, c->cur, c->hmask, c->nzv, c->nzrow, skip);
  else
    k_sig_range<Src, 2048, K, SKIP><<<(unsigned)s.nranges, 256, 0, c->stream>>>(
        src, c->ranges, c->H, c->DC, sink, c->cur, c->hmask, c->nzv, c->nzrow, skip);
  LAUNCH_CHECK();
  return 0;
}

// skip: singleton flags of the previous partition (work-efficient mode), or NULL.
template <class Src, class K>
int launch_ranges_k(kbisim_ctx *c, const Src &src, const Schedule &s, KeySink sink, const unsigned char *skip,
                    bool range_tier) {
  if (s.nranges && range_tier) {
    int rc = 0;
    if constexpr (Src::GRAPH) {
      rc = skip ? launch_range_kernel<Src, K, true>(c, src, s, sink, skip)
                : launch_range_kernel<Src, K, false>(c, src, s, sink, nullptr);
    } else {
      rc = launch_range_kernel<Src, K, false>(c, src, s, sink, nullptr);
    }
    if (rc) return rc;
  }
  if (s.nbig || s.nrow8 || s.nrow20) {
    ProfScope ps(c, KBISIM_K_SIG_BLOCK);
    if (s.nbig) {
      k_sig_row<Src, RANGE_DMAX, 512, K><<<(unsigned)s.nbig, 512, 0, c->stream>>>(
          src, c->ranges + s.nranges, c->H, c->DC, sink, c->cur, c->hmask, c->zrep, skip);
      LAUNCH_CHECK();
    }
    if (s.nrow8) {
      k_sig_row<Src, ROW_MAX, 1024, K><<<(unsigned)s.nrow8, 1024, 0, c->stream>>>(
          src, c->ranges + s.nranges + s.nbig, c->H, c->DC, sink, c->cur, c->hmask, c->zrep, skip);
      LAUNCH_CHECK();
    }
    if constexpr (std::is_same<K, u32>::value) {
      if (s.nrow20) {
        k_sig_row<Src, ROW_MAX_NARROW, 1024, u32><<<(unsigned)s.nrow20, 1024, 0, c->stream>>>(
            src, c->ranges + s.nranges + s.nbig + s.nrow8, c->H, c->DC, sink, c->cur, c->hmask, c->zrep,
            skip);
        LAUNCH_CHECK();
      }
    }
  }
  return 0;
}

template <class Src>
int launch_ranges(kbisim_ctx *c, const Src &src, const Schedule &s, KeySink sink, const unsigned char *skip,
                  bool range_tier) {
  if constexpr (Src::HASHED) {
    return launch_ranges_k<Src, u32>(c, src, s, sink, skip, range_tier);
  } else {
    if constexpr (Src::GRAPH) {
      if (c->narrow) return launch_ranges_k<Src, u32>(c, src, s, sink, skip, range_tier);
    }
    return launch_ranges_k<Src, u64>(c, src, s, sink, skip, range_tier);
  }
}

// Staged hub rows: chunk dedupe and partitioned staging, then per-partition
// dedupe and sums.  K: width of the staged keys.
template <class Src, class K>
int launch_hub_staged(kbisim_ctx *c, const Src &src, const Schedule &s, const int *hubs,
                      const unsigned char *skip) {
  K *stage = reinterpret_cast<K *>(c->hubsets);
  {
    ProfScope ps(c, KBISIM_K_HUB_STAGE);
    if (c->tune.hub_chunk == 2048)
      k_hub_stage<Src, 2048, K><<<(unsigned)s.nchunks, 256, 0, c->stream>>>(src, c->chunks, hubs, stage, c->poff,
                                                                            c->err, skip);
    else
      k_hub_stage<Src, 4096, K><<<(unsigned)s.nchunks, 256, 0, c->stream>>>(src, c->chunks, hubs, stage, c->poff,
                                                                            c->err, skip);
    LAUNCH_CHECK();
  }
  ProfScope ps(c, KBISIM_K_HUB_REDUCE);
  k_hub_reduce<Src, K><<<(unsigned)s.nparts, 256, 0, c->stream>>>(src, c->parts, c->chunks, stage, c->poff, c->hacc,
                                                                  c->hcnt, c->err, hubs, skip);
  LAUNCH_CHECK();
  return 0;
}

// One refinement step: src (previous partition inside) -> out, block count
// into *count_dev.  cnt: CNT_STRIDE zeroed device counters for this step.
// careful: settle every collision with host-driven peeling rounds.
// gpid_next: where to write the new partition in rank order (NULL: not needed).
// zfresh: group vertices with an empty signature afresh (the first step of a
// call); otherwise their representatives from that step are kept, since two
// such vertices share a block after a step exactly when they did before it.
// skip_in / single_out (work-efficient mode, else NULL): singleton flags of
// the previous partition (those vertices are not refined: a singleton block
// cannot split) and of the new one.
// Signatures of every vertex not flagged in skip_in (all tiers): key hash,
// distinct count and the insertion into the grouping table.
template <class Src>
int launch_signatures(kbisim_ctx *c, const Src &src, const Schedule &s, bool zfresh, const unsigned char *skip_in,
                      bool range_tier = true, bool partition = false) {
  const u64 tmask = table_mask<Src>(c);
  // (the partition's keys lie where the table is otherwise)
  const KeySink sink{partition ? nullptr : c->table, tmask, c->rep, partition ? c->table : nullptr};
  int rc = 0;
  if constexpr (!Src::GRAPH) {
    if (!src.ptr) {  // one label per vertex
      ProfScope ps(c, KBISIM_K_SIG_RANGE);
      k_sig_one<Src><<<blocks_for(c->g.n, ONE_VERTS), ONE_THREADS, 0, c->stream>>>(src, (int)c->g.n, c->H, c->DC, c->table, tmask,
                                                                    c->cur, c->hmask);
      LAUNCH_CHECK();
      return 0;
    }
  }
  if (zfresh && range_tier && s.nonempty < c->g.n) {
    ProfScope ps(c, KBISIM_K_LOOKUP);  // it forms representatives; a launch of the range kernel holds entries
    k_sig_empty<Src><<<blocks_for(c->g.n, EMPTY_VERTS), EMPTY_THREADS, 0, c->stream>>>(src, (int)c->g.n, c->DC,
                                                                                       c->zrep, c->cur, skip_in);
    LAUNCH_CHECK();
  }
  if ((rc = launch_ranges(c, src, s, sink, skip_in, range_tier))) return rc;
  if (s.nhub) {
    const int *hubs = c->lists + s.hub_off;
    if (s.nchunks) {
      if constexpr (Src::HASHED) {
        rc = launch_hub_staged<Src, u32>(c, src, s, hubs, skip_in);
      } else if constexpr (Src::GRAPH) {
        rc = c->narrow ? launch_hub_staged<Src, u32>(c, src, s, hubs, skip_in)
                       : launch_hub_staged<Src, u64>(c, src, s, hubs, skip_in);
      } else {
        rc = launch_hub_staged<Src, u64>(c, src, s, hubs, skip_in);
      }
      if (rc) return rc;
    }
    if (s.ngchunks) {
      ProfScope ps(c, KBISIM_K_HUB_STAGE);
      auto global_sets = [&](auto key) {
        k_sig_hub_global<Src, decltype(key)><<<(unsigned)s.ngchunks, 256, 0, c->stream>>>(
            src, c->gchunks, hubs, c->hubsets, c->hacc, c->hcnt, c->cur, skip_in);
      };
      if constexpr (Src::HASHED) {
        global_sets(u32{});
      } else if constexpr (Src::GRAPH) {
        if (c->narrow) global_sets(u32{});
        else global_sets(u64{});
      } else {
        global_sets(u64{});
      }
      LAUNCH_CHECK();
    }
    ProfScope ps(c, KBISIM_K_HUB_FINAL);
    k_hub_final<Src><<<blocks_for(s.nhub, 256), 256, 0, c->stream>>>(src, hubs, s.nhub, c->hacc, c->hcnt, c->H, c->DC,
                                                                     sink, c->cur, c->hmask, c->zrep, skip_in, s.nzv, (int)s.nonempty);
    LAUNCH_CHECK();
  }
  return 0;
}

// Candidate representatives of the non-empty vertices by partition (see
// k_group_hist).  The signature kernels left the keys at the start of the
// grouping table's space; pairs go to the list space (vlist, clA, clB: 12 n
// bytes, free until the lookup), then back to the table's space, which also
// holds the histograms.  What it used there is cleared before the table is next
// used (table_dirty).
struct GroupPlan {
  int64_t nt, hist_n;  // tiles, histogram counters
  size_t off_ka, off_va, off_hist, off_offs[2], off_tiles, total;
};
GroupPlan group_plan(int64_t N) {
  GroupPlan p{};
  size_t at = 0;
  auto take = [&](size_t bytes) {
    size_t o = at;
    at = align_up(at + bytes);
    return o;
  };
  p.nt = (N + GROUP_TILE - 1) / GROUP_TILE;
  p.hist_n = 256 * p.nt;
  p.off_ka = take(8 * (size_t)N);
  p.off_va = take(4 * (size_t)N);
  p.off_hist = take(4 * (size_t)p.hist_n);
  p.off_offs[0] = take(8 * (size_t)(p.hist_n + 1));
  p.off_offs[1] = take(8 * (size_t)(p.hist_n + 1));
  p.off_tiles = take(8 * (size_t)(p.hist_n / SCAN_TILE + 1));
  p.total = at;
  return p;
}
int group_by_partition(kbisim_ctx *c, const Schedule &s) {
  ProfScope ps(c, KBISIM_K_LOOKUP);
  hipStream_t st = c->stream;
  const int64_t N = s.nonempty;
  const GroupPlan p = group_plan(N);
  if (p.total > 8 * c->plan.tslots) return KBISIM_EINTERNAL;
  const int64_t nt = p.nt, hist_n = p.hist_n;
  char *w = (char *)c->table;
  u64 *ka = (u64 *)(w + p.off_ka);
  int *va = (int *)(w + p.off_va), *hist = (int *)(w + p.off_hist);
  int64_t *offs[2] = {(int64_t *)(w + p.off_offs[0]), (int64_t *)(w + p.off_offs[1])};
  int64_t *tiles = (int64_t *)(w + p.off_tiles);
  u64 *kb = (u64 *)c->vlist;
  int *vb = (int *)(kb + N);
  const int64_t *total = offs[0] + hist_n, *left = offs[1] + hist_n;  // pairs after each pass
  const unsigned grid = radix_grid(nt);
  int rc = 0;
  c->table_dirty = p.total;
  const u32 mask = c->tune.group_mask;
  k_group_hist<false><<<grid, GROUP_THREADS, 0, st>>>(N, nullptr, nullptr, nullptr, ka, mask, 0, nt, hist);
  LAUNCH_CHECK();
  if ((rc = scan64(st, hist_n, hist, tiles, offs[0]))) return rc;
  k_group_scatter<<<grid, GROUP_THREADS, 0, st>>>(N, nullptr, ka, s.nzv, mask, 0, offs[0], kb, vb);
  k_group_hist<true><<<grid, GROUP_THREADS, 0, st>>>(N, total, vb, c->rep, kb, mask, 8, nt, hist);
  LAUNCH_CHECK();
  if ((rc = scan64(st, hist_n, hist, tiles, offs[1]))) return rc;
  k_group_scatter<<<grid, GROUP_THREADS, 0, st>>>(N, total, kb, vb, mask, 8, offs[1], ka, va);
  auto buckets = [&](auto kernel, int u) {
    kernel<<<blocks_for(N, u * BUCKET_GROUP), BUCKET_GROUP, 0, st>>>(left, ka, va, mask, c->tune.group_mean_bits, c->rep,
                                                                     c->err);
  };
  if ((N >> c->tune.group_mean_bits) < BUCKET_WIDE) buckets(k_group_buckets<2>, 2);
  else buckets(k_group_buckets<4>, 4);
  LAUNCH_CHECK();
  return 0;
}

// The grouping table empty again after partitioned steps used its space: only
// as far as they did (3.5M rows of an 8.4M-vertex graph: 47 MB of 134).
int clean_table(kbisim_ctx *c) {
  const size_t dirty = c->table_dirty;
  c->table_dirty = 0;
  return dirty ? fill_u64(c, c->table, (int64_t)(dirty / sizeof(u64)), 0) : 0;
}

// Whether full steps of this schedule group by partition.
bool by_partition(const kbisim_ctx *c, const Schedule &s) {
  return s.nzv && s.nonempty >= c->tune.group_min && 14 * (u64)s.nonempty + 16384 <= 8 * c->plan.tslots;
}

// After the lookup: exact checks of longer rows (any_long: the schedule has
// some), one peeling round and, when careful, host-driven peeling rounds until
// no collision is left.
template <class Src>
int settle_collisions(kbisim_ctx *c, const Src &src, const Schedule &s, int *cnt, bool careful, bool any_long = true) {
  const int n = (int)c->g.n;
  int rc = 0;
  if (any_long) {
    ProfScope ps(c, KBISIM_K_VERIFY);
    k_verify<Src><<<PERSIST_GRID, 256, 0, c->stream>>>(src, &cnt[0], c->vlist, c->DC, c->rep, &cnt[1], c->clA,
                                                       c->err);
    LAUNCH_CHECK();
  }
  if (!careful) {
    ProfScope ps(c, KBISIM_K_PEEL);
    k_peel_few<Src><<<1, 256, 0, c->stream>>>(src, &cnt[1], c->clA, c->H, c->DC, c->rep, &cnt[2], c->err);
    LAUNCH_CHECK();
  } else {
    if ((rc = peel_round(c, src, &cnt[1], c->clA, &cnt[2], c->clB))) return rc;
    int *in_cnt = &cnt[2], *out_cnt = &cnt[3];
    int *in_list = c->clB, *out_list = c->clA;
    for (int round = 0;; ++round) {
      int left = 0;
      HIP_TRY(hipMemcpyAsync(&left, in_cnt, sizeof(int), hipMemcpyDeviceToHost, c->stream));
      HIP_TRY(hipStreamSynchronize(c->stream));
      prof_collect(c);
      if (left == 0) break;
      if (round > n + 1) return KBISIM_EINTERNAL;
      if ((rc = fill_i32(c, out_cnt, 1, 0))) return rc;
      if ((rc = advance(c, ADV_CTABLE, s))) return rc;
      if ((rc = peel_round(c, src, in_cnt, in_list, out_cnt, out_list))) return rc;
      std::swap(in_cnt, out_cnt);
      std::swap(in_list, out_list);
    }
  }
  return 0;
}

template <class Src>
int run_step(kbisim_ctx *c, const Src &src, const Schedule &s, int *out, int64_t *count_dev, int *cnt,
             bool careful, int *gpid_next, bool zfresh, const unsigned char *skip_in = nullptr,
             unsigned char *single_out = nullptr, int32_t *names_out = nullptr, int *local_out = nullptr) {
  const int n = (int)c->g.n;
  if (n == 0) return 0;
  const u64 tmask = table_mask<Src>(c);
  int rc = 0;
  if (c->cur == c->dep && (rc = advance(c, ADV_TABLE | ADV_CTABLE | ADV_ZERO | (s.ngchunks ? ADV_HUB : 0u), s)))
    return rc;
  bool partition = false;
  if constexpr (Src::GRAPH) partition = !c->work_eff && by_partition(c, s);
  if (!partition && (rc = clean_table(c))) return rc;
  if ((rc = launch_signatures(c, src, s, zfresh, skip_in, true, partition))) return rc;
  if (partition && (rc = group_by_partition(c, s))) return rc;
  {
    ProfScope ps(c, KBISIM_K_LOOKUP);
    // Vertices without edges keep the representative of a call's first step;
    // the others are looked up through the list (label rows have none: every
    // vertex, empty ones included).
    if (s.nzv && zfresh && s.nonempty < n) {
      k_rep_empty<Src><<<blocks_for(n, 256), 256, 0, c->stream>>>(src, n, c->DC, c->zrep, c->cur, c->rep, c->err,
                                                                  skip_in);
      LAUNCH_CHECK();
    }
    const int count = s.nzv ? (int)s.nonempty : n;
    if (partition) {
      k_resolve<Src><<<blocks_for(count, 4 * RESOLVE_V), 256, 0, c->stream>>>(
          src, count, s.nzv, c->DC, c->rep, &cnt[0], c->vlist, &cnt[1], c->clA);
    } else if (count) {
      k_lookup<Src><<<blocks_for(count, 256), 256, 0, c->stream>>>(
          src, count, s.nzv, c->H, c->DC, c->table, tmask, c->cur, c->rep, &cnt[0], c->vlist, &cnt[1], c->clA, c->err,
          c->zrep, zfresh ? 1 : 0, skip_in, nullptr, nullptr);
    }
    LAUNCH_CHECK();
  }
  if ((rc = settle_collisions(c, src, s, cnt, careful, careful || s.nlong > 0))) return rc;
  HeadIds ids{};
  int scan_tiles = 0;  // tile counts that k_assign scans itself
  {
    ProfScope ps(c, KBISIM_K_SCAN);
    if ((rc = numbering_words(c, n, count_dev, &ids, names_out ? nullptr : &scan_tiles))) return rc;
  }
  {
    ProfScope ps(c, KBISIM_K_ASSIGN);
    if (names_out) {
      k_assign_names<<<blocks_for(n, 256), 256, 0, c->stream>>>(n, c->rep, ids, out, names_out,
                                                                gpid_next ? c->rank : nullptr, gpid_next, nullptr,
                                                                nullptr, nullptr, nullptr, nullptr);
    } else {
      const unsigned ag = blocks_for((n + ASSIGN_V - 1) / ASSIGN_V, 256);
      const int *rank = gpid_next ? c->rank : nullptr;
      u32 *multi = single_out ? c->multi : nullptr;
      const LocalIds loc{c->gid, c->first, local_out};
      auto *assign = scan_tiles ? (local_out ? k_assign<true, true> : k_assign<true, false>)
                                : (local_out ? k_assign<false, true> : k_assign<false, false>);
      assign<<<ag, 256, 0, c->stream>>>(n, c->rep, ids, out, rank, gpid_next, multi, c->cur, scan_tiles, count_dev,
                                        loc);
    }
    LAUNCH_CHECK();
    if (single_out) {
      k_singletons<<<blocks_for(n, 256), 256, 0, c->stream>>>(n, c->rep, c->multi, c->cur, single_out);
      LAUNCH_CHECK();
    }
  }
  return 0;
}

// Enqueue steps [i0, k) starting from partition `prev` (no host
// synchronisation unless careful).  In a batch, step i refines into an
// internal buffer of global ids and writes the caller's per-graph ids and
// counts (graph g's count of step i at bcounts[g * cstride + i]).  scatter:
// copy prev into the rank-ordered buffer first (false only when the previous
// step of this context already left it there).
int enqueue_steps(kbisim_ctx *c, const int32_t *prev, int i0, int k, int32_t *const *out, bool careful,
                  int cstride, bool scatter = true, bool reset_err = false) {
  const int n = (int)c->g.n;
  const bool batch = c->num_graphs > 0;
  // Counters and epochs are laid out ahead, for up to STEP_SEGMENT steps in one
  // launch; not where the host drives peeling rounds (they advance the epochs
  // too) or global hub sets need clearing every third step.
  const bool ahead = !careful && !c->sched.ngchunks;
  struct Restore {  // whatever way this returns, later calls use the context's epochs
    kbisim_ctx *c;
    ~Restore() { c->cur = c->dep; }
  } restore{c};
  int rc = 0;
  if (!ahead) {
    if (reset_err && (rc = fill_i32(c, (int *)c->err, 1, 0))) return rc;
    if ((rc = fill_i32(c, c->counters + CNT_STRIDE * (size_t)i0, CNT_STRIDE * (int64_t)(k - i0), 0))) return rc;
  }
  if (scatter) {
    k_scatter_rank<<<blocks_for(n, 256), 256, 0, c->stream>>>(n, prev, c->rank, c->gpid[i0 & 1]);
    LAUNCH_CHECK();
  }
  for (int i = i0; i < k; ++i) {
    if (ahead) {
      if ((i - i0) % STEP_SEGMENT == 0) {
        ProfScope ps(c, KBISIM_K_FILL);
        const bool table = c->work_eff || !by_partition(c, c->sched);
        k_prepare_steps<<<1, 64, 0, c->stream>>>(c->dep, c->counters, i, std::min(STEP_SEGMENT, k - i), table, c->err,
                                                 reset_err && i == i0 ? 1 : 0);
        LAUNCH_CHECK();
        if (table) {
          k_clear_if<<<CLEAR_GRID, 256, 0, c->stream>>>(c->dep, c->table, (int64_t)c->plan.tslots, nullptr, 0, nullptr,
                                                        0);
          LAUNCH_CHECK();
        }
      }
      c->cur = reinterpret_cast<const u32 *>(c->counters + CNT_STRIDE * (size_t)i) + STEP_EPOCHS;
    }
    int *dst = batch ? c->ibuf[i & 1] : out[i];
    // work-efficient mode: singletons of P_i (flags of step i-1) are not refined
    const unsigned char *skip_in = (c->work_eff && i > 0) ? c->single[(i - 1) & 1] : nullptr;
    unsigned char *single_out = c->work_eff ? c->single[i & 1] : nullptr;
    // with a cached chain (incremental updates) the next step names blocks by
    // their minimum vertex, written into the cache
    const bool cache = c->incr && !batch;
    int32_t *names_out = cache ? c->is.MVc + (size_t)i * (size_t)n : nullptr;
    auto step = [&](auto src) {
      return run_step(c, src, c->sched, dst, &c->dcounts[i], c->counters + CNT_STRIDE * i, careful,
                      c->gpid[(i + 1) & 1], i == 0, skip_in, single_out, names_out, batch ? out[i] : nullptr);
    };
    const int32_t *lab = separate_labels(c) ? sep_labels(c) : nullptr;
    if (c->hashed) {
      if (lab)
        rc = step(GraphSrcT<true, true>{c->g.row_ptr, c->gcol, lab, c->gpid[i & 1], prev, c->pb, c->rbits, c->kmask});
      else
        rc = step(
            GraphSrcT<false, true>{c->g.row_ptr, c->gcol, nullptr, c->gpid[i & 1], prev, c->pb, c->rbits, c->kmask});
    } else {
      if (lab) rc = step(GraphSrcT<true>{c->g.row_ptr, c->gcol, lab, c->gpid[i & 1], prev, c->pb, c->rbits});
      else rc = step(GraphSrcT<false>{c->g.row_ptr, c->gcol, nullptr, c->gpid[i & 1], prev, c->pb, c->rbits});
    }
    if (rc) return rc;
    if (batch) {
      k_batch_counts<<<blocks_for(c->num_graphs, 256), 256, 0, c->stream>>>((int)c->num_graphs, c->first, c->next,
                                                                            dst, &c->dcounts[i], cstride, i, c->bcounts);
      LAUNCH_CHECK();
    }
    if (names_out) {
      const unsigned g = std::min<unsigned>(blocks_for(2 * (int64_t)n, 256), 65536);
      k_copy_i32<<<g, 256, 0, c->stream>>>(reinterpret_cast<int *>(c->is.Hc + (size_t)i * (size_t)n),
                                           reinterpret_cast<const int *>(c->H), 2 * (int64_t)n);
      k_copy_i32<<<g, 256, 0, c->stream>>>(reinterpret_cast<int *>(c->is.DCc + (size_t)i * (size_t)n),
                                           reinterpret_cast<const int *>(c->DC), (int64_t)n);
      k_filter_keys<<<blocks_for(n, 256), 256, 0, c->stream>>>(n, c->H, c->DC, prev,
                                                                c->is.FKc + (size_t)i * (size_t)n);
      LAUNCH_CHECK();
      prev = names_out;
    } else {
      prev = dst;
    }
  }
  return 0;
}

// out[done - 1] copied to out[done .. k), read once for up to CopyDsts::MAX of
// them (6 copies of 33.5M ids: 350 -> 166 us).
int copy_outputs(kbisim_ctx *c, int32_t *const *out, int done, int k) {
  const int64_t n = c->g.n;
  for (int j0 = done; j0 < k; j0 += CopyDsts::MAX) {
    CopyDsts d{};
    d.nd = std::min(k - j0, (int)CopyDsts::MAX);
    for (int q = 0; q < d.nd; ++q) d.d[q] = out[j0 + q];
    k_copy_multi<<<std::min<unsigned>(blocks_for(n, 256), 65536), 256, 0, c->stream>>>(d, out[done - 1], n);
    LAUNCH_CHECK();
  }
  return 0;
}

// Work-efficient refinement: singleton blocks are not refined (skip flags
// from the previous step), and once a step leaves the block count unchanged
// the partition is a fixpoint (a refinement with as many blocks is the same
// partition), so the remaining outputs are copies.  Synchronises after every
// step to read its count.
int refine_we(kbisim_ctx *c, const int32_t *start, int k, int32_t *const *out, int64_t *counts) {
  const int n = (int)c->g.n;
  const bool batch = c->num_graphs > 0;
  const int32_t *p0 = start ? start : c->p0;
  int64_t prev_count = start ? -1 : c->p0_count;
  int rc = 0;
  int done = k;
  for (int i = 0; i < k; ++i) {
    const int32_t *prev = i == 0 ? p0 : (batch ? c->ibuf[(i - 1) & 1] : out[i - 1]);
    if ((rc = enqueue_steps(c, prev, i, i + 1, out, false, k, i == 0, i == 0))) return rc;
    int left = 0;
    u32 err = 0;
    int64_t cnt = 0;
    HIP_TRY(hipMemcpyAsync(&left, c->counters + CNT_STRIDE * i + 2, sizeof(int), hipMemcpyDeviceToHost, c->stream));
    HIP_TRY(hipMemcpyAsync(&err, c->err, sizeof err, hipMemcpyDeviceToHost, c->stream));
    HIP_TRY(hipMemcpyAsync(&cnt, &c->dcounts[i], 8, hipMemcpyDeviceToHost, c->stream));
    HIP_TRY(hipStreamSynchronize(c->stream));
    prof_collect(c);
    if (err) return KBISIM_EINTERNAL;
    if (left) {
      if ((rc = enqueue_steps(c, prev, i, i + 1, out, true, k, true))) return rc;
      HIP_TRY(hipMemcpyAsync(&err, c->err, sizeof err, hipMemcpyDeviceToHost, c->stream));
      HIP_TRY(hipMemcpyAsync(&cnt, &c->dcounts[i], 8, hipMemcpyDeviceToHost, c->stream));
      HIP_TRY(hipStreamSynchronize(c->stream));
      prof_collect(c);
      if (err) return KBISIM_EINTERNAL;
    }
    if (cnt == prev_count) {
      done = i + 1;
      break;
    }
    prev_count = cnt;
  }
  if (n > 0 && (rc = copy_outputs(c, out, done, k))) return rc;
  if (batch) {
    const int64_t G = c->num_graphs;
    HIP_TRY(hipMemcpyAsync(counts, c->bcounts, 8 * (size_t)(G * k), hipMemcpyDeviceToHost, c->stream));
    HIP_TRY(hipStreamSynchronize(c->stream));
    for (int64_t g = 0; g < G; ++g)
      for (int j = done; j < k; ++j) counts[g * k + j] = counts[g * k + done - 1];
  } else {
    HIP_TRY(hipMemcpyAsync(counts, c->dcounts, 8 * (size_t)done, hipMemcpyDeviceToHost, c->stream));
    HIP_TRY(hipStreamSynchronize(c->stream));
    for (int j = done; j < k; ++j) counts[j] = counts[done - 1];
  }
  c->we_steps = done;
  return KBISIM_OK;
}

int refine_impl(kbisim_ctx *c, const int32_t *start, int k, int32_t *const *out, int64_t *counts) {
  if (!c) return KBISIM_EINVAL;
  if (k < 0 || k > c->kmax) return KBISIM_EINVAL;
  if (k == 0) return KBISIM_OK;
  if (!out || !counts) return KBISIM_EINVAL;
  for (int i = 0; i < k; ++i)
    if (!out[i] && c->g.n > 0) return KBISIM_EINVAL;
  const int n = (int)c->g.n;
  const bool batch = c->num_graphs > 0;
  const int64_t ncounts = batch ? c->num_graphs * (int64_t)k : (int64_t)k;
  if (n == 0) {
    for (int64_t i = 0; i < ncounts; ++i) counts[i] = 0;
    return KBISIM_OK;
  }
  if (c->work_eff) return refine_we(c, start, k, out, counts);
  if (c->incr) c->incr_k = 0;  // until this call completes
  const int32_t *p0 = start ? start : c->p0;
  int rc = 0;
  const bool graphed = c->use_graphs && !c->prof;
  if (graphed) {
    GraphKey key{start, k, std::vector<const void *>(out, out + k)};
    auto it = c->graphs.find(key);
    if (it == c->graphs.end()) {
      if ((int)c->graphs.size() >= MAX_GRAPH_CACHE) {
        (void)hipGraphExecDestroy(c->graphs.begin()->second);
        c->graphs.erase(c->graphs.begin());
      }
      HIP_TRY(hipStreamBeginCapture(c->stream, hipStreamCaptureModeThreadLocal));
      const int rc1 = enqueue_steps(c, p0, 0, k, out, false, k, true, true);
      hipGraph_t graph = nullptr;
      hipError_t e = hipStreamEndCapture(c->stream, &graph);
      if (rc1) {
        if (graph) (void)hipGraphDestroy(graph);
        return rc1;
      }
      if (e != hipSuccess) return hip_fail(e);
      hipGraphExec_t exec = nullptr;
      e = hipGraphInstantiate(&exec, graph, nullptr, nullptr, 0);
      (void)hipGraphDestroy(graph);
      if (e != hipSuccess) return hip_fail(e);
      it = c->graphs.emplace(key, exec).first;
    }
    if (by_partition(c, c->sched)) c->table_dirty = group_plan(c->sched.nonempty).total;  // by the captured steps
    HIP_TRY(hipGraphLaunch(it->second, c->stream));
  } else {
    if ((rc = enqueue_steps(c, p0, 0, k, out, false, k, true, true))) return rc;
  }
  // Counters, block counts and the error word are one stretch of the
  // workspace: one copy brings them back, as long as it is short.
  const size_t span = c->plan.off_err + sizeof(u32) - c->plan.off_counters;
  const bool whole = span <= READBACK_MAX;
  std::vector<int> hc(whole ? (span + 3) / 4 : (size_t)CNT_STRIDE * k);
  u32 err = 0;
  HIP_TRY(hipMemcpyAsync(hc.data(), c->counters, whole ? span : 4 * hc.size(), hipMemcpyDeviceToHost, c->stream));
  if (!whole) HIP_TRY(hipMemcpyAsync(&err, c->err, sizeof err, hipMemcpyDeviceToHost, c->stream));
  if (batch) HIP_TRY(hipMemcpyAsync(counts, c->bcounts, 8 * (size_t)ncounts, hipMemcpyDeviceToHost, c->stream));
  HIP_TRY(hipStreamSynchronize(c->stream));
  prof_collect(c);
  if (whole) memcpy(&err, (const char *)hc.data() + (c->plan.off_err - c->plan.off_counters), sizeof err);
  if (err) return KBISIM_EINTERNAL;
  int first_bad = -1;
  for (int i = 0; i < k; ++i)
    if (hc[(size_t)CNT_STRIDE * i + 2] != 0) {
      first_bad = i;
      break;
    }
  if (first_bad >= 0) {
    const int32_t *prev = first_bad == 0 ? p0 : (batch ? c->ibuf[(first_bad - 1) & 1] : out[first_bad - 1]);
    if (c->incr && !batch && first_bad > 0) prev = c->is.MVc + (size_t)(first_bad - 1) * (size_t)n;
    if ((rc = enqueue_steps(c, prev, first_bad, k, out, true, k))) return rc;
    HIP_TRY(hipMemcpyAsync(&err, c->err, sizeof err, hipMemcpyDeviceToHost, c->stream));
    HIP_TRY(hipStreamSynchronize(c->stream));
    prof_collect(c);
    if (err) return KBISIM_EINTERNAL;
  }
  if (!batch && whole && first_bad < 0) {
    memcpy(counts, (const char *)hc.data() + (c->plan.off_dcounts - c->plan.off_counters), 8 * (size_t)k);
  } else if (!batch || first_bad >= 0) {
    HIP_TRY(hipMemcpyAsync(counts, batch ? c->bcounts : c->dcounts, 8 * (size_t)ncounts, hipMemcpyDeviceToHost,
                           c->stream));
    HIP_TRY(hipStreamSynchronize(c->stream));
  }
  if (c->incr && !batch) c->incr_k = start ? 0 : k;  // the cache holds a chain from P0
  return KBISIM_OK;
}

// ---------------------------------------------------------------- incremental updates
// The cached chain lives in a caller buffer: per step the key hash, distinct
// count and minimum-vertex block name of every vertex, plus the in-rows of
// the cached graph (to find the vertices whose targets' names changed) and
// per-update scratch.
struct IncrPlan {
  size_t off_hc, off_dcc, off_mvc, off_fk, off_tptr, off_tcol, off_names, off_edited, off_flag, off_dirty, off_skip,
      off_small, off_large, off_psmall, off_plarge, off_changed, off_bname, off_keep, off_claimed, off_heavy, off_touch,
      off_lk, off_filter, off_gfilter, off_zrep, off_huge, off_hchunks, off_hacc, off_hcnt, off_erows, off_cnt, total;
  int64_t huge_cap, huge_chunk_cap;
};
IncrPlan incr_plan(int64_t n, int64_t m, int kmax) {
  IncrPlan p{};
  size_t at = 0;
  auto take = [&](size_t bytes) {
    size_t o = at;
    at = align_up(at + std::max<size_t>(bytes, 1));
    return o;
  };
  const size_t N = (size_t)std::max<int64_t>(n, 1), K = (size_t)std::max(kmax, 1);
  p.off_hc = take(8 * N * K);
  p.off_dcc = take(4 * N * K);
  p.off_mvc = take(4 * N * K);
  p.off_fk = take(2 * N * K);
  p.off_tptr = take(8 * (N + 1));
  p.off_tcol = take(4 * (size_t)std::max<int64_t>(m, 1));
  p.off_names = take(8 * N);
  p.off_edited = take(N);
  p.off_flag = take(N);
  p.off_dirty = take(N);
  p.off_skip = take(N);
  p.off_small = take(4 * N);
  p.off_large = take(4 * N);
  p.off_psmall = take(4 * N);
  p.off_plarge = take(4 * N);
  p.off_changed = take(4 * N);
  p.off_bname = take(4 * N);
  p.off_keep = take(4 * N);
  p.off_claimed = take(N);
  p.off_heavy = take(4 * N);
  p.off_touch = take(4 * (N / 32 + 1));
  p.off_lk = take(4 * N);
  p.off_filter = take(4 * FILTER_WORDS);
  p.off_gfilter = take(4 * (size_t)GFILTER_WORDS);
  p.off_zrep = take(16 * N);
  p.huge_cap = std::max<int64_t>(m, 0) / LIST_BIG + 1;
  p.huge_chunk_cap = std::max<int64_t>(m, 0) / HUB_GCHUNK + p.huge_cap + 1;
  p.off_huge = take(4 * (size_t)p.huge_cap);
  p.off_hchunks = take(sizeof(HubGChunk) * (size_t)p.huge_chunk_cap);
  p.off_hacc = take(8 * (size_t)p.huge_cap);
  p.off_hcnt = take(4 * (size_t)p.huge_cap);
  p.off_erows = take(sizeof(Range) * (size_t)p.huge_cap);
  p.off_cnt = take(64);
  p.total = at;
  return p;
}

constexpr int LIST_GRID_SMALL = 2048, LIST_GRID_LARGE = 1024, MARK_GRID = 2048;

// Grouping-table mask for about `keys` keys at a load of at most 1/4 (a
// small table stays in the caches), within the allocated table.
u64 mask_for_keys(const kbisim_ctx *c, int64_t keys) {
  return std::min<u64>(pow2_at_least((uint64_t)std::max<int64_t>(4 * keys, 4096)), c->plan.tslots) - 1;
}

// One update step: P'_{i+1} from names_prev (P0 for i = 0, else the block
// names of P'_i).  Vertices flagged dirty had their key inputs changed: the
// edited rows are read from the edited graph (list kernels); the others whose
// targets' names changed are signed by the list kernels too when they are few
// (prop_lists), else by the cached graph's tiers with every other vertex
// skipped.  With few dirty vertices (prop_lists; at most ndirty of them) only
// the touched cached blocks are regrouped (k_classify), in a
// table sized for them, and every other vertex keeps its cached block and
// name; otherwise all vertices take their cached key hashes and go through
// the table.  Exact checks read the edited graph; numbering covers every
// vertex; block names follow k_block_names_*.  Returns in *gpid_written
// whether the names were also written in rank order for the next step.
template <class K, class TierSrc, class ListSrc>
int update_step(kbisim_ctx *c, const TierSrc &tsrc, const ListSrc &lsrc, int i, const int32_t *names_prev,
                int32_t *out, int64_t *count_dev, int *cnt, bool prop_lists, int nbig, int64_t ndirty,
                bool *gpid_written) {
  const int n = (int)c->g.n;
  const size_t at = (size_t)i * (size_t)n;
  auto &S = c->is;
  c->tmask_steps = prop_lists ? mask_for_keys(c, ndirty) : c->plan.tslots - 1;
  u64 tmask = c->tmask_steps;
  const Schedule &s = c->sched;
  // the hub epoch starts at 0 and must be in 1..3 before any global set is used
  int rc = advance(c, ADV_TABLE | ADV_CTABLE | ADV_ZERO | (s.ngchunks || S.nhuge ? ADV_HUB : 0u), s);
  if (rc) return rc;
  auto lists = [&](int *count, int *small, int *large) -> int {
    k_sig_list_small<ListSrc, K><<<LIST_GRID_SMALL, 256, 0, c->stream>>>(lsrc, count, small, c->H, c->DC, c->table,
                                                                         tmask, c->cur, c->hmask, c->zrep);
    LAUNCH_CHECK();
    k_sig_list_large<ListSrc, K><<<LIST_GRID_LARGE, 256, 0, c->stream>>>(lsrc, count + 1, large, c->H, c->DC,
                                                                         c->table, tmask, c->cur, c->hmask, c->zrep,
                                                                         c->err);
    LAUNCH_CHECK();
    return 0;
  };
  if (prop_lists) {
    // short and medium rows from lists, long ones by the row and hub tiers
    if ((rc = lists(&cnt[8], S.psmall, S.plarge))) return rc;
    if (nbig && (rc = launch_signatures(c, tsrc, s, true, S.skip, false))) return rc;
  } else {
    k_skip_all_flagged<<<blocks_for(n, 256), 256, 0, c->stream>>>(n, S.edited, S.dirty, S.skip);
    LAUNCH_CHECK();
    if ((rc = launch_signatures(c, tsrc, s, true, S.skip))) return rc;
  }
  if ((rc = lists(&S.cnt[0], S.small, S.large))) return rc;
  const KeySink sink{c->table, tmask, nullptr, nullptr};
  if (S.nerows8) {
    k_sig_row<ListSrc, ROW_MAX, 1024, K><<<(unsigned)S.nerows8, 1024, 0, c->stream>>>(
        lsrc, S.erows, c->H, c->DC, sink, c->cur, c->hmask, c->zrep, nullptr);
    LAUNCH_CHECK();
  }
  if constexpr (std::is_same<K, u32>::value) {
    if (S.nerows20) {
      k_sig_row<ListSrc, ROW_MAX_NARROW, 1024, u32><<<(unsigned)S.nerows20, 1024, 0, c->stream>>>(
          lsrc, S.erows + S.nerows8, c->H, c->DC, sink, c->cur, c->hmask, c->zrep, nullptr);
      LAUNCH_CHECK();
    }
  }
  if (S.nhuge) {
    // edited rows too long for one workgroup: global hash sets in the spare hub-set space
    if ((rc = fill_u64(c, c->hubsets + S.huge_set_begin, S.huge_set_slots, 0))) return rc;
    k_sig_hub_global<ListSrc, K><<<(unsigned)S.nhuge_chunks, 256, 0, c->stream>>>(
        lsrc, S.huge_chunks, S.huge, c->hubsets + S.huge_set_begin, S.huge_acc, S.huge_cnt, c->cur, nullptr);
    LAUNCH_CHECK();
    k_hub_final<ListSrc><<<blocks_for(S.nhuge, 256), 256, 0, c->stream>>>(lsrc, S.huge, S.nhuge, S.huge_acc,
                                                                          S.huge_cnt, c->H, c->DC, sink, c->cur,
                                                                          c->hmask, c->zrep, nullptr, nullptr, 0);
    LAUNCH_CHECK();
  }
  int nlk = 0;
  if (prop_lists) {
    // touched blocks: the cached blocks of dirty vertices (k_update_flags) and
    // those whose key a dirty vertex now has (k_classify)
    if ((rc = fill_i32(c, (int *)S.filter, FILTER_WORDS, 0))) return rc;
    u32 *gfilter = ndirty >= c->tune.gfilter_min ? S.gfilter : nullptr;
    if (gfilter && (rc = fill_i32(c, (int *)gfilter, GFILTER_WORDS, 0))) return rc;
    if (ndirty > 0) {
      // the dirty vertices were listed by k_update_flags (count at cnt[12])
      k_build_filter<<<blocks_for(ndirty, 256), 256, 0, c->stream>>>(&cnt[12], S.lk, c->H, c->DC, names_prev,
                                                                      S.MVc + at, S.filter, gfilter);
      LAUNCH_CHECK();
    }
    k_classify<<<(unsigned)std::min<int64_t>(CLASSIFY_GRID, blocks_for(n, 256)), 256, 0, c->stream>>>(
        n, S.MVc + at, S.dirty, S.touch, S.FKc + at, S.Hc + at, S.DCc + at, names_prev, S.filter, gfilter, c->table,
        tmask, c->cur, c->zrep, c->H, c->DC, c->rep, S.names[i & 1], &cnt[11], S.lk);
    LAUNCH_CHECK();
    HIP_TRY(hipMemcpyAsync(&nlk, &cnt[11], sizeof nlk, hipMemcpyDeviceToHost, c->stream));
    HIP_TRY(hipStreamSynchronize(c->stream));
    if (2 * (int64_t)nlk > (int64_t)tmask + 1) {
      // more keys than the dirty-sized table holds: a larger one, all listed keys again
      if ((rc = advance(c, ADV_TABLE, s))) return rc;
      c->tmask_steps = tmask = mask_for_keys(c, nlk);
    }
    if (nlk) {
      k_insert_list<<<blocks_for(nlk, 256), 256, 0, c->stream>>>(nlk, S.lk, c->H, c->DC, names_prev, c->table, tmask,
                                                                  c->cur, c->zrep);
      k_lookup<ListSrc><<<blocks_for(nlk, 256), 256, 0, c->stream>>>(
          lsrc, nlk, S.lk, c->H, c->DC, c->table, tmask, c->cur, c->rep, &cnt[0], c->vlist, &cnt[1], c->clA, c->err,
          c->zrep, 1, nullptr, S.dirty, S.MVc + at);
      LAUNCH_CHECK();
    }
  } else {
    k_insert_cached<<<blocks_for(n, 256), 256, 0, c->stream>>>(n, S.dirty, S.Hc + at, S.DCc + at, S.MVc + at,
                                                                names_prev, c->H, c->DC, c->table, tmask, c->cur,
                                                                c->zrep);
    LAUNCH_CHECK();
    k_lookup<ListSrc><<<blocks_for(n, 256), 256, 0, c->stream>>>(lsrc, n, nullptr, c->H, c->DC, c->table, tmask,
                                                                 c->cur, c->rep, &cnt[0], c->vlist, &cnt[1], c->clA,
                                                                 c->err, c->zrep, 1, nullptr, S.dirty, S.MVc + at);
    LAUNCH_CHECK();
  }
  if ((rc = settle_collisions(c, lsrc, s, cnt, true))) return rc;
  HeadIds ids{};
  if ((rc = numbering_words(c, n, count_dev, &ids))) return rc;
  if ((rc = fill_i32(c, reinterpret_cast<int *>(S.claimed), (n + 3) / 4, 0))) return rc;
  if (prop_lists) {
    k_assign_out<<<blocks_for((n + ASSIGN_V - 1) / ASSIGN_V, 256), 256, 0, c->stream>>>(n, c->rep, ids, out);
    LAUNCH_CHECK();
    if (nlk) {
      const unsigned g = blocks_for(nlk, 256);
      k_block_names_fresh<<<g, 256, 0, c->stream>>>(n, c->rep, S.bname, S.keep, nlk, S.lk);
      k_block_names_clean<<<g, 256, 0, c->stream>>>(n, c->rep, S.dirty, S.MVc + at, S.bname, S.claimed, nlk, S.lk);
      k_block_names_keep<<<g, 256, 0, c->stream>>>(n, c->rep, S.dirty, S.MVc + at, S.bname, S.claimed, S.keep, nlk,
                                                   S.lk);
      k_assign_names<<<g, 256, 0, c->stream>>>(n, c->rep, ids, nullptr, S.names[i & 1], nullptr, nullptr, S.bname,
                                               S.keep, S.MVc + at, &cnt[6], S.changed, nlk, S.lk);
      LAUNCH_CHECK();
    }
    *gpid_written = false;
  } else {
    k_block_names_fresh<<<blocks_for(n, 256), 256, 0, c->stream>>>(n, c->rep, S.bname, S.keep);
    k_block_names_clean<<<blocks_for(n, 256), 256, 0, c->stream>>>(n, c->rep, S.dirty, S.MVc + at, S.bname,
                                                                    S.claimed);
    k_block_names_keep<<<blocks_for(n, 256), 256, 0, c->stream>>>(n, c->rep, S.dirty, S.MVc + at, S.bname,
                                                                   S.claimed, S.keep);
    k_assign_names<<<blocks_for(n, 256), 256, 0, c->stream>>>(n, c->rep, ids, out, S.names[i & 1], c->rank,
                                                              c->gpid[(i + 1) & 1], S.bname, S.keep, S.MVc + at,
                                                              &cnt[6], S.changed);
    LAUNCH_CHECK();
    *gpid_written = true;
  }
  k_mark_in_neighbours<<<MARK_GRID, 256, 0, c->stream>>>(&cnt[6], S.changed, S.tptr, S.tcol, S.flag, &cnt[7],
                                                         S.heavy);
  k_mark_heavy<<<MARK_GRID, 256, 0, c->stream>>>(&cnt[7], S.heavy, S.tptr, S.tcol, S.flag);
  LAUNCH_CHECK();
  return 0;
}

template <bool HK, class K>
int update_steps_t(kbisim_ctx *c, const kbisim_graph *gn, int k, int32_t *const *out) {
  const int n = (int)c->g.n;
  auto &S = c->is;
  const int32_t *lab = separate_labels(c) ? sep_labels(c) : nullptr;
  int rc = 0;
  bool gpid_ok = false;  // gpid[i & 1] holds names_prev in rank order (written when a step needs it)
  for (int i = 0; i < k; ++i) {
    if (i >= 2) {
      // P'_{i-1} refines P'_{i-2}: with as many blocks it is the same
      // partition, and so is every later one (a step depends on the previous
      // partition alone): copies, no more steps
      int64_t pc[2] = {0, 0};
      HIP_TRY(hipMemcpyAsync(pc, &c->dcounts[i - 2], sizeof pc, hipMemcpyDeviceToHost, c->stream));
      HIP_TRY(hipStreamSynchronize(c->stream));
      if (pc[0] == pc[1]) {
        if ((rc = copy_outputs(c, out, i, k))) return rc;
        for (int j = i; j < k; ++j)
          HIP_TRY(hipMemcpyAsync(&c->dcounts[j], &c->dcounts[i - 1], sizeof(int64_t), hipMemcpyDeviceToDevice,
                                 c->stream));
        return 0;
      }
    }
    const int32_t *names_prev = i == 0 ? c->p0 : S.names[(i - 1) & 1];
    int *cnt = c->counters + CNT_STRIDE * i;
    if ((rc = fill_i32(c, cnt, CNT_STRIDE, 0))) return rc;
    if ((rc = fill_i32(c, reinterpret_cast<int *>(S.touch), (n + 31) / 32, 0))) return rc;
    k_update_flags<<<blocks_for((n + FLAGS_GROUP - 1) / FLAGS_GROUP, 256), 256, 0, c->stream>>>(
        n, S.edited, S.flag, S.dirty, S.skip, gn->row_ptr, cnt + 8, S.psmall, S.plarge, S.MVc + (size_t)i * n, S.touch,
        S.lk);
    LAUNCH_CHECK();
    if ((rc = fill_i32(c, reinterpret_cast<int *>(S.flag), (n + 3) / 4, 0))) return rc;
    // few vertices flagged by the previous step: sign them from lists
    int np[3] = {0, 0, 0};
    HIP_TRY(hipMemcpyAsync(np, cnt + 8, sizeof np, hipMemcpyDeviceToHost, c->stream));
    HIP_TRY(hipStreamSynchronize(c->stream));
    const int64_t nprop = (int64_t)np[0] + np[1] + np[2];
    const bool prop_lists = nprop <= std::max<int64_t>(n / 8, 1);
    if ((!prop_lists || np[2] > 0) && !gpid_ok) {
      // the tier kernels read the previous names in rank order
      k_scatter_rank<<<blocks_for(n, 256), 256, 0, c->stream>>>(n, names_prev, c->rank, c->gpid[i & 1]);
      LAUNCH_CHECK();
    }
    const PlainSrcT<HK> lsrc{gn->row_ptr, gn->col, gn->elabel, names_prev, c->pb, c->kmask};
    const int64_t ndirty = nprop + S.nrows;
    if (lab)
      rc = update_step<K>(c, GraphSrcT<true, HK>{c->g.row_ptr, c->gcol, lab, c->gpid[i & 1], names_prev, c->pb,
                                                 c->rbits, c->kmask},
                          lsrc, i, names_prev, out[i], &c->dcounts[i], cnt, prop_lists, np[2], ndirty, &gpid_ok);
    else
      rc = update_step<K>(c, GraphSrcT<false, HK>{c->g.row_ptr, c->gcol, nullptr, c->gpid[i & 1], names_prev, c->pb,
                                                  c->rbits, c->kmask},
                          lsrc, i, names_prev, out[i], &c->dcounts[i], cnt, prop_lists, np[2], ndirty, &gpid_ok);
    if (rc) return rc;
  }
  return 0;
}

int update_impl(kbisim_ctx *c, const kbisim_graph *gn, const int32_t *rows, int64_t nrows, int k,
                int32_t *const *out, int64_t *counts) {
  if (!c || !gn || !c->incr || c->num_graphs > 0) return KBISIM_EINVAL;
  if (k < 0 || k > c->incr_k) return KBISIM_EINVAL;
  if (k == 0) return KBISIM_OK;
  if (!out || !counts) return KBISIM_EINVAL;
  const int64_t n = c->g.n;
  if (gn->n != n || gn->m < 0 || (gn->elabel == nullptr) != (c->g.elabel == nullptr)) return KBISIM_EINVAL;
  if (gn->m >= (int64_t(1) << 62)) return KBISIM_ERANGE;
  if (nrows < 0 || nrows > n || (nrows > 0 && !rows)) return KBISIM_EINVAL;
  if (n == 0) {
    for (int i = 0; i < k; ++i) counts[i] = 0;
    return KBISIM_OK;
  }
  for (int i = 0; i < k; ++i)
    if (!out[i]) return KBISIM_EINVAL;
  if (!gn->row_ptr || (gn->m > 0 && !gn->col)) return KBISIM_EINVAL;
  auto &S = c->is;
  int rc = 0;
  // the edited graph: row offsets, every target and label (any row is read by
  // the exact checks), the listed vertices
  if ((rc = fill_i32(c, (int *)c->err, 1, 0))) return rc;
  k_validate_rows<<<blocks_for(n + 1, 256), 256, 0, c->stream>>>(n, gn->m, gn->row_ptr, c->err, ERR_GRAPH_ROWPTR);
  if (gn->m > 0) {
    validate_vals(c->stream, gn->m, gn->col, n, c->err, ERR_GRAPH_COL);
    if (gn->elabel)
      validate_vals(c->stream, gn->m, gn->elabel, (int64_t)c->max_label + 1, c->err, ERR_GRAPH_ELABEL);
  }
  if (nrows) validate_vals(c->stream, nrows, rows, n, c->err, ERR_BAD_PID);
  LAUNCH_CHECK();
  u32 err = 0;
  if ((rc = read_err(c, &err))) return rc;
  if (err & ERR_BAD_PID) return KBISIM_EINVAL;
  if (err) return KBISIM_EGRAPH;
  // flags and the edited rows, split by length
  if ((rc = fill_i32(c, reinterpret_cast<int *>(S.edited), (n + 3) / 4, 0))) return rc;
  if ((rc = fill_i32(c, reinterpret_cast<int *>(S.flag), (n + 3) / 4, 0))) return rc;
  if ((rc = fill_i32(c, S.cnt, 16, 0))) return rc;
  if ((rc = fill_i32(c, S.cnt + 2, 1, (int)nrows))) return rc;
  S.nhuge = 0;
  S.nhuge_chunks = 0;
  S.nerows8 = S.nerows20 = 0;
  S.nrows = nrows;
  if (nrows) {
    k_set_flags<<<std::min<unsigned>(blocks_for(nrows, 256), 65536), 256, 0, c->stream>>>(S.cnt + 2, rows, S.edited);
    // edited rows longer than LIST_BIG: a row-kernel workgroup each up to
    // what one workgroup's LDS holds, longer ones global sets when the spare
    // hub-set space holds them (else they stay with the multi-pass list kernel)
    const int64_t free_begin = c->sched.gset_end;
    const int64_t free_end = c->glab ? (int64_t)(reinterpret_cast<const u64 *>(c->glab) - c->hubsets)
                                     : c->plan.hubset_slots;
    const int64_t row_cap = c->narrow ? ROW_MAX_NARROW : ROW_MAX;
    k_split_list<<<blocks_for(nrows, 256), 256, 0, c->stream>>>((int)nrows, rows, gn->row_ptr, &S.cnt[0], S.small,
                                                                  &S.cnt[1], S.large, (int64_t)LIST_BIG, &S.cnt[3],
                                                                  S.huge);
    LAUNCH_CHECK();
    {
      int nh = 0;
      HIP_TRY(hipMemcpyAsync(&nh, &S.cnt[3], sizeof nh, hipMemcpyDeviceToHost, c->stream));
      HIP_TRY(hipStreamSynchronize(c->stream));
      if (nh > 0) {
        std::vector<int> hv((size_t)nh);
        std::vector<int64_t> be(2 * (size_t)nh);
        // extents staged in the chunk buffer (rewritten below)
        int64_t *be_dev = reinterpret_cast<int64_t *>(S.huge_chunks);
        k_row_extents<<<blocks_for(nh, 256), 256, 0, c->stream>>>(nh, S.huge, gn->row_ptr, be_dev);
        LAUNCH_CHECK();
        HIP_TRY(hipMemcpyAsync(hv.data(), S.huge, 4 * (size_t)nh, hipMemcpyDeviceToHost, c->stream));
        HIP_TRY(hipMemcpyAsync(be.data(), be_dev, 16 * (size_t)nh, hipMemcpyDeviceToHost, c->stream));
        HIP_TRY(hipStreamSynchronize(c->stream));
        std::vector<HubGChunk> ch;
        std::vector<int> keep_list;
        std::vector<Range> r8, r20;
        int64_t at = free_begin;
        int nglob = 0;
        for (int i = 0; i < nh; ++i) {
          const int v = hv[(size_t)i];
          const int64_t b = be[2 * (size_t)i], d = be[2 * (size_t)i + 1] - b;
          if (d <= row_cap) {
            (d <= ROW_MAX ? r8 : r20).push_back(Range{v, v + 1, (int)d, 0, b});
            continue;
          }
          if (at + 2 * d > free_end || (int64_t)ch.size() + d / HUB_GCHUNK + 1 > S.huge_chunk_cap) {
            keep_list.push_back(v);  // no room: back to the list kernel
            continue;
          }
          for (int64_t x = 0; x < d; x += HUB_GCHUNK)
            ch.push_back(HubGChunk{nglob, 0, x, std::min<int64_t>(d, x + HUB_GCHUNK), at - free_begin, 2 * d});
          hv[(size_t)nglob++] = v;
          at += 2 * d;
        }
        S.nerows8 = (int)r8.size();
        S.nerows20 = (int)r20.size();
        r8.insert(r8.end(), r20.begin(), r20.end());
        if (!r8.empty())
          HIP_TRY(hipMemcpyAsync(S.erows, r8.data(), sizeof(Range) * r8.size(), hipMemcpyHostToDevice, c->stream));
        S.nhuge = nglob;
        S.nhuge_chunks = (int)ch.size();
        S.huge_set_begin = free_begin;
        S.huge_set_slots = at - free_begin;
        if (S.nhuge) {
          HIP_TRY(hipMemcpyAsync(S.huge, hv.data(), 4 * (size_t)S.nhuge, hipMemcpyHostToDevice, c->stream));
          HIP_TRY(hipMemcpyAsync(S.huge_chunks, ch.data(), sizeof(HubGChunk) * ch.size(), hipMemcpyHostToDevice,
                                 c->stream));
        }
        if (!keep_list.empty()) {  // append to the large list (its count is on the device)
          int nl = 0;
          HIP_TRY(hipMemcpyAsync(&nl, &S.cnt[1], sizeof nl, hipMemcpyDeviceToHost, c->stream));
          HIP_TRY(hipStreamSynchronize(c->stream));
          HIP_TRY(hipMemcpyAsync(S.large + nl, keep_list.data(), 4 * keep_list.size(), hipMemcpyHostToDevice,
                                 c->stream));
          if ((rc = fill_i32(c, &S.cnt[1], 1, nl + (int)keep_list.size()))) return rc;
        }
        HIP_TRY(hipStreamSynchronize(c->stream));
      }
    }
  }
  if ((rc = clean_table(c))) return rc;
  // every vertex may carry a key in an update (edited rows can gain entries),
  // and empty signatures are grouped by block names below 2n
  const u64 tmask_saved = c->tmask_steps;
  u64 *zrep_saved = c->zrep;
  c->tmask_steps = c->plan.tslots - 1;
  c->zrep = S.zrep;
  if (c->hashed) rc = update_steps_t<true, u32>(c, gn, k, out);
  else if (c->narrow) rc = update_steps_t<false, u32>(c, gn, k, out);
  else rc = update_steps_t<false, u64>(c, gn, k, out);
  c->tmask_steps = tmask_saved;
  c->zrep = zrep_saved;
  if (rc) return rc;
  HIP_TRY(hipMemcpyAsync(&err, c->err, sizeof err, hipMemcpyDeviceToHost, c->stream));
  HIP_TRY(hipMemcpyAsync(counts, c->dcounts, 8 * (size_t)k, hipMemcpyDeviceToHost, c->stream));
  HIP_TRY(hipStreamSynchronize(c->stream));
  prof_collect(c);
  if (err) return KBISIM_EINTERNAL;
  return KBISIM_OK;
}

int incr_enable_impl(kbisim_ctx *c, void *state, size_t bytes) {
  if (!c || c->num_graphs > 0 || c->work_eff || c->kmax < 1 || !state) return KBISIM_EINVAL;
  const int64_t n = c->g.n, m = c->g.m;
  if (n >= (int64_t(1) << 30)) return KBISIM_ERANGE;  // update block names reach 2n
  const IncrPlan p = incr_plan(n, m, c->kmax);
  if (bytes < p.total) return KBISIM_ENOSPACE;
  char *w = (char *)state;
  auto &S = c->is;
  S.Hc = (u64 *)(w + p.off_hc);
  S.DCc = (u32 *)(w + p.off_dcc);
  S.MVc = (int32_t *)(w + p.off_mvc);
  S.FKc = (uint16_t *)(w + p.off_fk);
  S.tptr = (int64_t *)(w + p.off_tptr);
  S.tcol = (int32_t *)(w + p.off_tcol);
  S.names[0] = (int32_t *)(w + p.off_names);
  S.names[1] = S.names[0] + std::max<int64_t>(n, 1);
  S.edited = (unsigned char *)(w + p.off_edited);
  S.flag = (unsigned char *)(w + p.off_flag);
  S.dirty = (unsigned char *)(w + p.off_dirty);
  S.skip = (unsigned char *)(w + p.off_skip);
  S.small = (int *)(w + p.off_small);
  S.large = (int *)(w + p.off_large);
  S.psmall = (int *)(w + p.off_psmall);
  S.plarge = (int *)(w + p.off_plarge);
  S.changed = (int *)(w + p.off_changed);
  S.bname = (int32_t *)(w + p.off_bname);
  S.keep = (int32_t *)(w + p.off_keep);
  S.claimed = (unsigned char *)(w + p.off_claimed);
  S.heavy = (int *)(w + p.off_heavy);
  S.touch = (u32 *)(w + p.off_touch);
  S.lk = (int *)(w + p.off_lk);
  S.filter = (u32 *)(w + p.off_filter);
  S.gfilter = (u32 *)(w + p.off_gfilter);
  S.huge = (int *)(w + p.off_huge);
  S.huge_chunks = (HubGChunk *)(w + p.off_hchunks);
  S.huge_acc = (u64 *)(w + p.off_hacc);
  S.huge_cnt = (u32 *)(w + p.off_hcnt);
  S.erows = (Range *)(w + p.off_erows);
  S.huge_cap = p.huge_cap;
  S.huge_chunk_cap = p.huge_chunk_cap;
  S.zrep = (u64 *)(w + p.off_zrep);
  S.cnt = (int *)(w + p.off_cnt);
  int rc0 = 0;
  if (n > 0) {
    // in-rows of the cached graph: count per target, offsets, scatter
    int *cnt = S.names[0];
    auto *cursor = reinterpret_cast<unsigned long long *>(S.Hc);
    auto *tiles = reinterpret_cast<int64_t *>(S.small);
    const int64_t nt = (n + SCAN_TILE - 1) / SCAN_TILE;
    int rc = fill_i32(c, cnt, n, 0);
    if (rc) return rc;
    if (m > 0)
      k_indegree<<<(unsigned)std::min<int64_t>(blocks_for(m, INDEG_CHUNK), 65536), 256, 0, c->stream>>>(m, c->g.col,
                                                                                                       cnt);
    k_sum_tiles64<<<(unsigned)nt, 256, 0, c->stream>>>(n, cnt, tiles);
    k_scan_tiles64<<<1, 256, 0, c->stream>>>(nt, tiles);
    k_write_ptr64<false><<<(unsigned)nt, 256, 0, c->stream>>>(n, cnt, tiles, S.tptr, cursor);
    if (m > 0)
      k_transpose_scatter<<<(unsigned)std::min<int64_t>(blocks_for(n * WAVE, 256), 65536), 256, 0, c->stream>>>(
          n, c->g.row_ptr, c->g.col, nullptr, cursor, S.tcol, nullptr);
    LAUNCH_CHECK();
    HIP_TRY(hipStreamSynchronize(c->stream));
  }
  if ((rc0 = fill_u64(c, S.zrep, 2 * std::max<int64_t>(n, 1), ~0ULL))) return rc0;
  if ((rc0 = fill_u64(c, S.huge_acc, S.huge_cap, 0))) return rc0;
  if ((rc0 = fill_i32(c, (int *)S.huge_cnt, S.huge_cap, 0))) return rc0;
  // Update steps name blocks below 2n, so pairs keep one more bit of block
  // name; a pair's value (label << 31 | name) does not depend on that width,
  // only whether exact 32-bit keys still fit does.
  {
    u32 pb = 1, lb = 0;
    while (pb < 31 && (int64_t(1) << pb) < 2 * n) ++pb;
    while (lb < 32 && (c->max_label >> lb) != 0) ++lb;
    c->pb = pb;
    c->hashed = c->narrow && (c->tune.key_bits == 32 || pb + lb > 31);
  }
  // loops captured before did not cache their steps
  for (auto &kv : c->graphs) (void)hipGraphExecDestroy(kv.second);
  c->graphs.clear();
  c->incr = true;
  c->incr_k = 0;
  return KBISIM_OK;
}

int check_sizes(const kbisim_graph *g) {
  if (!g) return KBISIM_EINVAL;
  if (g->n < 0 || g->m < 0 || g->nlabels < 0) return KBISIM_EINVAL;
  if (g->n >= (int64_t(1) << 31) || g->m >= (int64_t(1) << 62) || g->nlabels >= (int64_t(1) << 62))
    return KBISIM_ERANGE;
  return 0;
}

int read_tuning(const kbisim_tuning *t, Tuning &out) {
  out = Tuning{};
  if (!t) return 0;
  if (t->range_edges) {
    if (t->range_edges != 1024 && t->range_edges != 2048) return KBISIM_EINVAL;
    out.range_edges = t->range_edges;
  }
  if (t->hub_chunk) {
    if (t->hub_chunk != 2048 && t->hub_chunk != 4096) return KBISIM_EINVAL;
    out.hub_chunk = t->hub_chunk;
  }
  if (t->hub_part_target) {
    if (t->hub_part_target != 1024 && t->hub_part_target != 2048) return KBISIM_EINVAL;
    out.hub_part_target = t->hub_part_target;
  }
  if (t->key_bits) {
    if (t->key_bits != 32 && t->key_bits != 64) return KBISIM_EINVAL;
    out.key_bits = t->key_bits;
  }
  if (t->scan_items) {
    if (t->scan_items != 8 && t->scan_items != 16) return KBISIM_EINVAL;
    out.scan_items = t->scan_items;
  }
  return 0;
}

// Shared by kbisim_create and kbisim_batch_create.  With vert_off (host,
// num_graphs + 1) the graph is a batch of disjoint graphs.
int create_impl(const kbisim_graph *g, int kmax, const kbisim_tuning *tuning, void *workspace, size_t ws_bytes,
                void *stream, int64_t num_graphs, const int64_t *vert_off, kbisim_ctx **out) {
  int rc = check_sizes(g);
  if (rc) return rc;
  if (!out || kmax < 0 || kmax > (1 << 20)) return KBISIM_EINVAL;
  *out = nullptr;
  Tuning tune;
  if ((rc = read_tuning(tuning, tune))) return rc;
  const int64_t n = g->n, m = g->m;
  if (n > 0 && !g->row_ptr) return KBISIM_EINVAL;
  if (m > 0 && !g->col) return KBISIM_EINVAL;
  if (g->vlabel_ptr && !g->vlabel && g->nlabels > 0) return KBISIM_EINVAL;
  if (!g->vlabel_ptr && !g->vlabel && g->nlabels > 0) return KBISIM_EINVAL;
  if (num_graphs > 0) {
    if (!vert_off || vert_off[0] != 0 || vert_off[num_graphs] != n) return KBISIM_EINVAL;
    for (int64_t i = 0; i < num_graphs; ++i)
      if (vert_off[i + 1] < vert_off[i]) return KBISIM_EINVAL;
  }
  const int64_t nl = g->vlabel_ptr ? g->nlabels : 0;
  Plan plan = make_plan(n, m, nl, kmax, num_graphs);
  if (!workspace || (reinterpret_cast<uintptr_t>(workspace) & (ALIGN - 1))) return KBISIM_EINVAL;
  if (ws_bytes < plan.total) return KBISIM_ENOSPACE;

  kbisim_ctx *c = new (std::nothrow) kbisim_ctx();
  if (!c) return KBISIM_EINTERNAL;
  c->g = *g;
  c->kmax = kmax;
  c->stream = (hipStream_t)stream;
  c->plan = plan;
  c->tune = tune;
  c->ws = (char *)workspace;
  char *w = c->ws;
  c->H = (u64 *)(w + plan.off_H);
  c->DC = (u32 *)(w + plan.off_DC);
  c->rep = (int *)(w + plan.off_rep);
  c->p0 = (int *)(w + plan.off_p0);
  c->vlist = (int *)(w + plan.off_vlist);
  c->clA = (int *)(w + plan.off_clA);
  c->clB = (int *)(w + plan.off_clB);
  c->ranges = (Range *)(w + plan.off_ranges);
  c->lists = (int *)(w + plan.off_lists);
  c->table = (u64 *)(w + plan.off_table);
  c->ctable = (u64 *)(w + plan.off_ctable);
  c->cslots = (int64_t)(plan.tslots / 2);  // still at least n
  c->nzrow = reinterpret_cast<u32 *>(c->ctable + c->cslots);
  c->hacc = (u64 *)(w + plan.off_hacc);
  c->hcnt = (u32 *)(w + plan.off_hcnt);
  c->chunks = (HubChunk *)(w + plan.off_chunks);
  c->parts = (HubPart *)(w + plan.off_parts);
  c->gchunks = (HubGChunk *)(w + plan.off_gchunks);
  c->poff = (int *)(w + plan.off_poff);
  c->tiles = (u32 *)(w + plan.off_status);
  c->hw = (HeadWord *)(w + plan.off_hw);
  c->gcol = (int *)(w + plan.off_gcol);
  c->rank = (int *)(w + plan.off_rank);
  c->gpid[0] = (int *)(w + plan.off_gpid);
  c->gpid[1] = c->gpid[0] + std::max<int64_t>(n, 1);
  c->zrep = (u64 *)(w + plan.off_zrep);
  c->counters = (int *)(w + plan.off_counters);
  c->dcounts = (int64_t *)(w + plan.off_dcounts);
  c->err = (u32 *)(w + plan.off_err);
  c->dep = (u32 *)(w + plan.off_dep);
  c->cur = c->dep;
  c->hubsets = (u64 *)(w + plan.off_hubsets);
  c->single[0] = (unsigned char *)(w + plan.off_single);
  c->single[1] = c->single[0] + std::max<int64_t>(n, 1);
  c->multi = (u32 *)(w + plan.off_multi);
  c->nzv = (int *)(w + plan.off_nzv);
  if (num_graphs > 0) {
    c->num_graphs = num_graphs;
    c->gid = (int *)(w + plan.off_gid);
    c->ibuf[0] = (int *)(w + plan.off_ibuf);
    c->ibuf[1] = c->ibuf[0] + std::max<int64_t>(n, 1);
    c->first = (int64_t *)(w + plan.off_first);
    c->next = (int64_t *)(w + plan.off_next);
    c->bcounts = (int64_t *)(w + plan.off_bcounts);
  }
  const char *dbg = getenv("KBISIM_DEBUG_HASH_BITS");
  if (dbg && *dbg) {
    int b = atoi(dbg);
    if (b >= 0 && b < 64) c->hmask = b == 0 ? 0ULL : ((1ULL << b) - 1ULL);
  }
  // Test knob: at most this many partitions per staged hub, so that hub
  // partitions overflow their sets and take the sub-pass path.
  const char *pdbg = getenv("KBISIM_DEBUG_HUB_PARTS");
  if (pdbg && *pdbg) {
    int q = atoi(pdbg);
    if (q >= 1 && q <= HUB_PMAX && (q & (q - 1)) == 0) c->tune.hub_parts_cap = q;
  }
  // Test knob: keep only this many bits of hashed set keys, so that keys
  // collide inside rows (the exact check must still separate the pair sets).
  const char *kdbg = getenv("KBISIM_DEBUG_KEY_BITS");
  if (kdbg && *kdbg) {
    int b = atoi(kdbg);
    if (b >= 1 && b < 32) c->kmask = (1u << b) - 1u;
  }
  // Test knob: group by partition from this many non-empty rows on (at least 1).
  const char *qdbg = getenv("KBISIM_DEBUG_GROUP_MIN");
  if (qdbg && *qdbg) {
    const long q = atol(qdbg);
    if (q >= 1) c->tune.group_min = q;
  }
  // Test knob: only this many bucket bits, so that small graphs have buckets
  // of more keys than a workgroup's set holds and take its sub-passes; after
  // a comma, the bits that their number is planned for (16: planned for one).
  const char *bdbg = getenv("KBISIM_DEBUG_GROUP_BITS");
  if (bdbg && *bdbg) {
    const int b = atoi(bdbg);
    if (b >= 0 && b < GROUP_BITS) c->tune.group_mask = (1u << b) - 1u;
    const char *comma = strchr(bdbg, ',');
    const int e = comma ? atoi(comma + 1) : GROUP_BITS;
    if (e >= 0 && e <= GROUP_BITS) c->tune.group_mean_bits = e;
  }
  // Test knob: update steps use the global dirty-key filter from this many
  // dirty vertices on (at least 1), so that small graphs take that path.
  const char *gdbg = getenv("KBISIM_DEBUG_GFILTER_MIN");
  if (gdbg && *gdbg) {
    int q = atoi(gdbg);
    if (q >= 1) c->tune.gfilter_min = q;
  }

  auto fail = [&](int code) {
    delete c;
    return code;
  };
  // Validation (Def. multi-relational-labeled-property-graph as a CSR contract).
  if ((rc = fill_i32(c, (int *)c->err, 4, 0))) return fail(rc);
  if ((rc = fill_i32(c, (int *)c->dep, 16, 0))) return fail(rc);
  if (n == 0 && m > 0) return fail(KBISIM_EGRAPH);
  if (n > 0) {
    k_validate_rows<<<blocks_for(n + 1, 256), 256, 0, c->stream>>>(n, m, g->row_ptr, c->err, ERR_GRAPH_ROWPTR);
    if (hipGetLastError() != hipSuccess) return fail(KBISIM_EHIP);
  }
  if (m > 0) {
    validate_vals(c->stream, m, g->col, n, c->err, ERR_GRAPH_COL);
    if (g->elabel) validate_vals(c->stream, m, g->elabel, -1, c->err, ERR_GRAPH_ELABEL, c->err + 2);
  }
  if (g->vlabel_ptr) {
    k_validate_rows<<<blocks_for(n + 1, 256), 256, 0, c->stream>>>(n, nl, g->vlabel_ptr, c->err, ERR_GRAPH_VPTR);
    if (nl > 0) validate_vals(c->stream, nl, g->vlabel, -1, c->err, ERR_GRAPH_VLABEL);
  } else if (g->vlabel && n > 0) {
    validate_vals(c->stream, n, g->vlabel, -1, c->err, ERR_GRAPH_VLABEL);
  }
  if (hipGetLastError() != hipSuccess) return fail(KBISIM_EHIP);
  std::vector<int64_t> nxt;
  if (num_graphs > 0) {
    // graph of every vertex; first vertex of the next non-empty graph
    nxt.assign((size_t)num_graphs, -1);
    int64_t after = -1;
    for (int64_t i = num_graphs - 1; i >= 0; --i) {
      nxt[(size_t)i] = after;
      if (vert_off[i + 1] > vert_off[i]) after = vert_off[i];
    }
    if (hipMemcpyAsync(c->first, vert_off, 8 * (size_t)(num_graphs + 1), hipMemcpyHostToDevice, c->stream) !=
            hipSuccess ||
        hipMemcpyAsync(c->next, nxt.data(), 8 * (size_t)num_graphs, hipMemcpyHostToDevice, c->stream) != hipSuccess)
      return fail(KBISIM_EHIP);
    if (n > 0) {
      const unsigned vchunks = blocks_for(n, GRAPH_CHUNK);
      k_graph_ids<<<vchunks + blocks_for(m, GRAPH_CHUNK), 256, 0, c->stream>>>(num_graphs, n, m, vchunks, c->first,
                                                                             g->row_ptr, g->col, c->gid, c->err);
      if (hipGetLastError() != hipSuccess) return fail(KBISIM_EHIP);
    }
  }
  u32 ew[4] = {0, 0, 0, 0};  // error bits, -, largest edge label
  if (hipMemcpyAsync(ew, c->err, sizeof ew, hipMemcpyDeviceToHost, c->stream) != hipSuccess ||
      hipStreamSynchronize(c->stream) != hipSuccess)
    return fail(KBISIM_EHIP);
  if (ew[0]) return fail(KBISIM_EGRAPH);
  u32 err = 0;

  // Pairs keep block ids modulo 2^pb, pb = bit width of the largest graph's
  // vertex count (the block ids of one graph form an interval no longer than
  // that).  Keys inside LDS sets are (edge label << pb) | reduced block, in
  // 31 bits, when the labels allow.
  {
    int64_t gmax = n;
    if (num_graphs > 0) {
      gmax = 0;
      for (int64_t i = 0; i < num_graphs; ++i) gmax = std::max<int64_t>(gmax, vert_off[i + 1] - vert_off[i]);
    }
    const u32 max_label = ew[2];
    u32 pb = 1, lb = 0;
    while (pb < 31 && (int64_t(1) << pb) < gmax) ++pb;
    while (lb < 32 && (max_label >> lb) != 0) ++lb;
    c->pb = pb;
    c->max_label = max_label;
    // pack (label, rank) into one 32-bit gather index when both fit
    u32 rb = 1;
    while (rb < 31 && (int64_t(1) << rb) < n) ++rb;
    if (g->elabel && rb + lb <= 32) {
      c->packed = true;
      c->rbits = rb;
    }
    // 32-bit set keys unless 64-bit ones are asked for: exact when the label
    // and reduced block fit 31 bits together, else a hash of the pair
    // (key_bits = 32 asks for hashed keys in any case)
    c->narrow = c->tune.key_bits != 64;
    c->hashed = c->narrow && (c->tune.key_bits == 32 || pb + lb > 31);
  }

  // Gather renumbering: rank vertices by decreasing in-degree class (ties by id).
  // Uses the grouping tables as scratch, before they are cleared below.
  if ((rc = build_rank(c))) return fail(rc);
  // Fresh state: tables start empty; empty-signature slots start above any entry.
  if ((rc = fill_u64(c, c->table, (int64_t)plan.tslots, 0))) return fail(rc);
  if ((rc = fill_u64(c, c->ctable, c->cslots, 0))) return fail(rc);
  if ((rc = fill_u64(c, c->zrep, std::max<int64_t>(n, 1), ~0ULL))) return fail(rc);
  if ((rc = fill_i32(c, (int *)c->multi, std::max<int64_t>(n, 1), 0))) return fail(rc);

  // P0: blocks of equal vertex label sets, numbered by first vertex; in a
  // batch the graph id joins the key, so no block spans two graphs.  Then the
  // static schedule of the graph rows.  What the host has to know of both
  // comes back in one copy: the schedule's totals in the counter rows kmax
  // and kmax + 1, P0's counters after them, its count and the error bits.
  static_assert((SCHED_TOTALS + 2) * sizeof(int64_t) <= 2 * CNT_STRIDE * sizeof(int), "two counter rows");
  const int gcap = range_cap(c, !c->narrow);
  const int64_t grow_max = c->narrow ? ROW_MAX_NARROW : ROW_MAX;
  int *back = c->counters + (size_t)CNT_STRIDE * kmax, *cnt = back + 2 * CNT_STRIDE;
  int64_t *totals = reinterpret_cast<int64_t *>(back);
  int64_t host[3 * CNT_STRIDE * sizeof(int) / sizeof(int64_t)] = {};
  if (!g->vlabel && num_graphs == 0) {
    if ((rc = fill_i32(c, c->p0, n, 0))) return fail(rc);
    c->p0_count = n > 0 ? 1 : 0;
  }
  if (n > 0) {
    Schedule ls;
    LabelSrc src{g->vlabel_ptr, g->vlabel, c->gid};
    if (!g->vlabel) src = LabelSrc{nullptr, c->gid, nullptr};  // batch without labels: one block per graph
    const bool labelled = g->vlabel || num_graphs > 0;
    auto copy_back = [&]() -> int {
      HIP_TRY(hipMemcpyAsync(host, back, sizeof host, hipMemcpyDeviceToHost, c->stream));
      HIP_TRY(hipStreamSynchronize(c->stream));
      return 0;
    };
    // A hash collision that P0's one peeling round did not settle: all again,
    // with host-driven rounds (the label rows' schedule shares the range lists).
    for (bool careful = false;; careful = true) {
      if (labelled && src.ptr) {
        const int lcap = range_cap(c, true);
        if ((rc = sched_enqueue(c, src.ptr, lcap, ROW_MAX, totals))) return fail(rc);
        if ((rc = copy_back())) return fail(rc);
        if ((rc = sched_finish(c, src.ptr, ls, lcap, HUB_STAGED_MAX_WIDE, host, nullptr))) return fail(rc);
      }
      if ((rc = fill_i32(c, back, 3 * CNT_STRIDE, 0))) return fail(rc);
      if (labelled &&
          (rc = run_step(c, src, ls, c->p0, &totals[SCHED_TOTALS], cnt, careful, nullptr, true)))
        return fail(rc);
      if ((rc = sched_enqueue(c, g->row_ptr, gcap, grow_max, totals))) return fail(rc);
      k_copy_i32<<<1, 1, 0, c->stream>>>((int *)&totals[SCHED_TOTALS + 1], (const int *)c->err, 1);
      if (hipGetLastError() != hipSuccess) return fail(KBISIM_EHIP);
      if ((rc = copy_back())) return fail(rc);
      err = (u32)host[SCHED_TOTALS + 1];
      if (labelled) c->p0_count = host[SCHED_TOTALS];
      if (careful || err || !labelled || reinterpret_cast<const int *>(host)[2 * CNT_STRIDE + 2] == 0) break;
    }
    if (err) return fail(KBISIM_EINTERNAL);
    if ((rc = sched_finish(c, g->row_ptr, c->sched, gcap, c->narrow ? HUB_STAGED_MAX : HUB_STAGED_MAX_WIDE, host,
                           c->nzv)))
      return fail(rc);
  }
  if ((rc = sort_long_rows(c, c->sched))) return fail(rc);
  // a load of at most 1/4 (within the planned table): shorter probe runs measured
  // faster than a smaller, more cache-resident span
  c->tmask_steps = std::min<u64>(pow2_at_least(4 * (uint64_t)std::max<int64_t>(c->sched.nonempty, 1)), plan.tslots) - 1;
  *out = c;
  return KBISIM_OK;
}

}  // namespace

extern "C" {

int kbisim_workspace_bytes(const kbisim_graph *g, int kmax, size_t *bytes) {
  int rc = check_sizes(g);
  if (rc) return rc;
  if (!bytes || kmax < 0 || kmax > (1 << 20)) return KBISIM_EINVAL;
  *bytes = make_plan(g->n, g->m, g->vlabel_ptr ? g->nlabels : 0, kmax, 0).total;
  return KBISIM_OK;
}

int kbisim_create(const kbisim_graph *g, int kmax, void *workspace, size_t ws_bytes, void *stream, kbisim_ctx **out) {
  return create_impl(g, kmax, nullptr, workspace, ws_bytes, stream, 0, nullptr, out);
}

int kbisim_create_tuned(const kbisim_graph *g, int kmax, const kbisim_tuning *tuning, void *workspace,
                        size_t ws_bytes, void *stream, kbisim_ctx **out) {
  return create_impl(g, kmax, tuning, workspace, ws_bytes, stream, 0, nullptr, out);
}

int kbisim_initial(kbisim_ctx *c, int32_t *out_ids, int64_t *out_count) {
  if (!c || !out_count || (c->g.n > 0 && !out_ids)) return KBISIM_EINVAL;
  if (c->g.n > 0) {
    k_copy_i32<<<std::min<unsigned>(blocks_for(c->g.n, 256), 65536), 256, 0, c->stream>>>(out_ids, c->p0, c->g.n);
    LAUNCH_CHECK();
    HIP_TRY(hipStreamSynchronize(c->stream));
  }
  *out_count = c->p0_count;
  return KBISIM_OK;
}

int kbisim_refine(kbisim_ctx *c, int k, int32_t *const *out_block_ids, int64_t *out_counts) {
  if (c && c->num_graphs > 0) return KBISIM_EINVAL;
  return refine_impl(c, nullptr, k, out_block_ids, out_counts);
}

int kbisim_refine_from(kbisim_ctx *c, const int32_t *pid_i, int k, int32_t *const *out_block_ids,
                       int64_t *out_counts) {
  if (!c || c->num_graphs > 0 || (c->g.n > 0 && !pid_i)) return KBISIM_EINVAL;
  if (c->g.n > 0) {
    int rc0 = fill_i32(c, (int *)c->err, 1, 0);
    if (rc0) return rc0;
    validate_vals(c->stream, c->g.n, pid_i, c->g.n, c->err, ERR_BAD_PID);
    LAUNCH_CHECK();
    u32 err = 0;
    int rc = read_err(c, &err);
    if (rc) return rc;
    if (err) return KBISIM_EINVAL;
  }
  return refine_impl(c, pid_i, k, out_block_ids, out_counts);
}

// Single steps.  Step i reads P_i (prev, P0 for i = 0; a batch keeps its own
// global-id copy) and writes P_{i+1} into out; the rank-ordered copy of the
// partition left by step i-1 is reused, so steps of one context go in order.
int step_async_impl(kbisim_ctx *c, int i, const int32_t *prev, int32_t *out) {
  if (!c || i < 0 || i >= c->kmax) return KBISIM_EINVAL;
  const bool batch = c->num_graphs > 0;
  if (c->g.n == 0) return KBISIM_OK;
  if (!out || (!batch && i > 0 && !prev) || (const int32_t *)out == prev) return KBISIM_EINVAL;
  const int32_t *p = i == 0 ? c->p0 : (batch ? c->ibuf[(i - 1) & 1] : prev);
  int rc = 0;
  if (c->incr) c->incr_k = 0;  // single steps do not keep a chain for updates
  std::vector<int32_t *> o((size_t)i + 1, out);  // indexed by step number
  return enqueue_steps(c, p, i, i + 1, o.data(), false, c->kmax, i == 0, i == 0);
}

int step_result_impl(kbisim_ctx *c, int i, const int32_t *prev, int32_t *out) {
  if (!c || i < 0 || i >= c->kmax) return KBISIM_EINVAL;
  const bool batch = c->num_graphs > 0;
  if (c->g.n == 0) return KBISIM_OK;
  if (!out || (!batch && i > 0 && !prev)) return KBISIM_EINVAL;
  const int32_t *p = i == 0 ? c->p0 : (batch ? c->ibuf[(i - 1) & 1] : prev);
  int left = 0;
  u32 err = 0;
  HIP_TRY(hipMemcpyAsync(&left, c->counters + CNT_STRIDE * i + 2, sizeof(int), hipMemcpyDeviceToHost, c->stream));
  HIP_TRY(hipMemcpyAsync(&err, c->err, sizeof err, hipMemcpyDeviceToHost, c->stream));
  HIP_TRY(hipStreamSynchronize(c->stream));
  prof_collect(c);
  if (err) return KBISIM_EINTERNAL;
  if (left) {
    std::vector<int32_t *> o((size_t)i + 1, out);
    int rc = enqueue_steps(c, p, i, i + 1, o.data(), true, c->kmax, true);
    if (rc) return rc;
    HIP_TRY(hipMemcpyAsync(&err, c->err, sizeof err, hipMemcpyDeviceToHost, c->stream));
    HIP_TRY(hipStreamSynchronize(c->stream));
    prof_collect(c);
    if (err) return KBISIM_EINTERNAL;
  }
  return KBISIM_OK;
}

int kbisim_step_async(kbisim_ctx *c, int i, const int32_t *prev, int32_t *out) {
  if (!c || c->num_graphs > 0) return KBISIM_EINVAL;
  return step_async_impl(c, i, prev, out);
}

int kbisim_step_result(kbisim_ctx *c, int i, const int32_t *prev, int32_t *out, int64_t *count) {
  if (!c || c->num_graphs > 0 || !count) return KBISIM_EINVAL;
  int rc = step_result_impl(c, i, prev, out);
  if (rc) return rc;
  if (c->g.n == 0) {
    *count = 0;
    return KBISIM_OK;
  }
  HIP_TRY(hipMemcpyAsync(count, &c->dcounts[i], 8, hipMemcpyDeviceToHost, c->stream));
  HIP_TRY(hipStreamSynchronize(c->stream));
  return KBISIM_OK;
}

int kbisim_work_efficient(kbisim_ctx *c, int enable, int *last_steps) {
  if (!c) return KBISIM_EINVAL;
  if (enable > 0 && c->incr) return KBISIM_EINVAL;  // updates need every step of the chain cached
  if (last_steps) *last_steps = c->we_steps;
  if (enable >= 0) c->work_eff = enable != 0;
  return KBISIM_OK;
}

int kbisim_use_graphs(kbisim_ctx *c, int enable) {
  if (!c) return KBISIM_EINVAL;
  if (enable && c->stream == nullptr) return KBISIM_EINVAL;  // the null stream cannot be captured
  c->use_graphs = enable != 0;
  return KBISIM_OK;
}

int kbisim_set_stream(kbisim_ctx *c, void *stream) {
  if (!c) return KBISIM_EINVAL;
  hipStream_t s = (hipStream_t)stream;
  if (c->use_graphs && s == nullptr) return KBISIM_EINVAL;
  if (s == c->stream) return KBISIM_OK;
  hipEvent_t e = nullptr;
  HIP_TRY(hipEventCreateWithFlags(&e, hipEventDisableTiming));
  hipError_t r = hipEventRecord(e, c->stream);
  if (r == hipSuccess) r = hipStreamWaitEvent(s, e, 0);
  (void)hipEventDestroy(e);
  if (r != hipSuccess) return hip_fail(r);
  c->stream = s;
  return KBISIM_OK;
}

int kbisim_incr_state_bytes(const kbisim_graph *g, int kmax, size_t *bytes) {
  int rc = check_sizes(g);
  if (rc) return rc;
  if (!bytes || kmax < 1 || kmax > (1 << 20)) return KBISIM_EINVAL;
  *bytes = incr_plan(g->n, g->m, kmax).total;
  return KBISIM_OK;
}

int kbisim_incr_enable(kbisim_ctx *c, void *state, size_t bytes) { return incr_enable_impl(c, state, bytes); }

int kbisim_incr_update(kbisim_ctx *c, const kbisim_graph *g_new, const int32_t *rows, int64_t nrows, int k,
                       int32_t *const *out_block_ids, int64_t *out_counts) {
  return update_impl(c, g_new, rows, nrows, k, out_block_ids, out_counts);
}

int kbisim_destroy(kbisim_ctx *c) {
  if (c) {
    for (hipEvent_t e : c->ev_pool) (void)hipEventDestroy(e);
    for (auto &kv : c->graphs) (void)hipGraphExecDestroy(kv.second);
  }
  delete c;
  return KBISIM_OK;
}

int kbisim_profile_enable(kbisim_ctx *c, int enable) {
  if (!c) return KBISIM_EINVAL;
  HIP_TRY(hipStreamSynchronize(c->stream));
  prof_collect(c);
  c->prof = enable != 0;
  for (int i = 0; i < KBISIM_NKERNELS; ++i) {
    c->prof_ms[i] = 0.0;
    c->prof_n[i] = 0;
  }
  return KBISIM_OK;
}

int kbisim_profile_select(kbisim_ctx *c, uint32_t kinds) {
  if (!c) return KBISIM_EINVAL;
  c->prof_mask = kinds;
  return KBISIM_OK;
}

int kbisim_profile_read(kbisim_ctx *c, double *ms, int64_t *launches) {
  if (!c) return KBISIM_EINVAL;
  HIP_TRY(hipStreamSynchronize(c->stream));
  prof_collect(c);
  for (int i = 0; i < KBISIM_NKERNELS; ++i) {
    if (ms) ms[i] = c->prof_ms[i];
    if (launches) launches[i] = c->prof_n[i];
  }
  return KBISIM_OK;
}

const char *kbisim_kernel_name(int kind) {
  static const char *names[KBISIM_NKERNELS] = {"k_sig_range", "k_sig_row", "k_hub_stage", "k_hub_reduce",
                                               "k_hub_final", "k_lookup",    "k_verify",    "k_res_*",
                                               "k_scan",      "k_assign",    "k_fill_*"};
  return (kind >= 0 && kind < KBISIM_NKERNELS) ? names[kind] : nullptr;
}

int kbisim_schedule_info(kbisim_ctx *c, int64_t *info) {
  if (!c || !info) return KBISIM_EINVAL;
  for (int i = 0; i < 8; ++i) info[i] = c->sched.info[i];
  return KBISIM_OK;
}

int kbisim_copy_probe(void *dst, const void *src, size_t bytes, void *stream) {
  if (!dst || !src || bytes % 16) return KBISIM_EINVAL;
  const int64_t n16 = (int64_t)(bytes / 16);
  if (n16 == 0) return KBISIM_OK;
  const unsigned g = (unsigned)std::min<int64_t>((n16 + 255) / 256, 1 << 20);
  k_copy16<<<g, 256, 0, (hipStream_t)stream>>>((uint4 *)dst, (const uint4 *)src, n16);
  HIP_TRY(hipGetLastError());
  return KBISIM_OK;
}

int kbisim_gather_probe(kbisim_ctx *c, const int32_t *pid, int reps, double *ms) {
  if (!c || !pid || reps < 1 || !ms) return KBISIM_EINVAL;
  *ms = 0.0;
  const int64_t n = c->g.n, m = c->g.m;
  if (m == 0) return KBISIM_OK;
  k_scatter_rank<<<blocks_for(n, 256), 256, 0, c->stream>>>((int)n, pid, c->rank, c->gpid[0]);
  HIP_TRY(hipGetLastError());
  u32 slots = 1;  // output words: a power of two, at most 1024 and at most n
  while (slots < 1024 && (int64_t)slots * 2 <= n) slots *= 2;
  int rc = fill_i32(c, c->vlist, slots, 0);
  if (rc) return rc;
  // the probe reads the same gather index and pairs as the signature kernels
  const unsigned grid = (unsigned)std::min<int64_t>((m + 1023) / 1024, 1 << 20);
  const GraphSrcT<true> sep{c->g.row_ptr, c->gcol, sep_labels(c), c->gpid[0], pid, c->pb, c->rbits};
  const GraphSrcT<false> pk{c->g.row_ptr, c->gcol, nullptr, c->gpid[0], pid, c->pb, c->rbits};
  const bool s2 = separate_labels(c);
  auto probe = [&]() {
    if (s2) k_gather_probe<<<grid, 256, 0, c->stream>>>(sep, m, (u32 *)c->vlist, slots - 1);
    else k_gather_probe<<<grid, 256, 0, c->stream>>>(pk, m, (u32 *)c->vlist, slots - 1);
  };
  hipEvent_t e0 = nullptr, e1 = nullptr;
  HIP_TRY(hipEventCreate(&e0));
  if (hipEventCreate(&e1) != hipSuccess) {
    (void)hipEventDestroy(e0);
    return KBISIM_EHIP;
  }
  probe();  // warm-up
  (void)hipEventRecord(e0, c->stream);
  for (int r = 0; r < reps; ++r) probe();
  (void)hipEventRecord(e1, c->stream);
  hipError_t e = hipStreamSynchronize(c->stream);
  float t = 0.f;
  if (e == hipSuccess) e = hipEventElapsedTime(&t, e0, e1);
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
  if (e != hipSuccess) return hip_fail(e);
  *ms = (double)t / reps;
  return KBISIM_OK;
}

int kbisim_batch_workspace_bytes(const kbisim_graph *u, int64_t num_graphs, int kmax, size_t *bytes) {
  int rc = check_sizes(u);
  if (rc) return rc;
  if (!bytes || num_graphs < 1 || num_graphs >= (int64_t(1) << 31) || kmax < 0 || kmax > (1 << 20))
    return KBISIM_EINVAL;
  *bytes = make_plan(u->n, u->m, u->vlabel_ptr ? u->nlabels : 0, kmax, num_graphs).total;
  return KBISIM_OK;
}

int kbisim_batch_create(const kbisim_graph *u, int64_t num_graphs, const int64_t *vert_off, int kmax,
                        const kbisim_tuning *tuning, void *workspace, size_t ws_bytes, void *stream,
                        kbisim_batch **out) {
  if (!out || num_graphs < 1 || num_graphs >= (int64_t(1) << 31) || !vert_off) return KBISIM_EINVAL;
  *out = nullptr;
  kbisim_ctx *c = nullptr;
  int rc = create_impl(u, kmax, tuning, workspace, ws_bytes, stream, num_graphs, vert_off, &c);
  if (rc) return rc;
  kbisim_batch *b = new (std::nothrow) kbisim_batch();
  if (!b) {
    kbisim_destroy(c);
    return KBISIM_EINTERNAL;
  }
  b->c = c;
  *out = b;
  return KBISIM_OK;
}

int kbisim_batch_refine(kbisim_batch *b, int k, int32_t *const *out_ids, int64_t *out_counts) {
  if (!b) return KBISIM_EINVAL;
  return refine_impl(b->c, nullptr, k, out_ids, out_counts);
}

int kbisim_batch_step_async(kbisim_batch *b, int i, int32_t *out_ids) {
  if (!b) return KBISIM_EINVAL;
  return step_async_impl(b->c, i, nullptr, out_ids);
}

int kbisim_batch_step_result(kbisim_batch *b, int i, int32_t *out_ids, int64_t *out_counts) {
  if (!b || !out_counts) return KBISIM_EINVAL;
  kbisim_ctx *c = b->c;
  int rc = step_result_impl(c, i, nullptr, out_ids);
  if (rc) return rc;
  const int64_t G = c->num_graphs;
  if (c->g.n == 0) {
    for (int64_t g = 0; g < G; ++g) out_counts[g] = 0;
    return KBISIM_OK;
  }
  // column i of the [graph][kmax] count table
  HIP_TRY(hipMemcpy2DAsync(out_counts, sizeof(int64_t), c->bcounts + i, sizeof(int64_t) * (size_t)c->kmax,
                           sizeof(int64_t), (size_t)G, hipMemcpyDeviceToHost, c->stream));
  HIP_TRY(hipStreamSynchronize(c->stream));
  return KBISIM_OK;
}

int kbisim_batch_context(kbisim_batch *b, kbisim_ctx **ctx) {
  if (!b || !ctx) return KBISIM_EINVAL;
  *ctx = b->c;
  return KBISIM_OK;
}

int kbisim_batch_destroy(kbisim_batch *b) {
  if (b) kbisim_destroy(b->c);
  delete b;
  return KBISIM_OK;
}

namespace {
// Numbers of entries that are sorted.  Below, the sort's extra launches cost
// more than the scatter's atomics (500k entries: 160 against 129 us; 5M: 276
// against 725 us); above, its two arrays of keys (16 bytes per entry) would
// take too much of the memory that a caller has beside the graph.
constexpr int64_t TRANSPOSE_SORT_MIN = (int64_t)1 << 20, TRANSPOSE_SORT_MAX = (int64_t)1 << 31;
struct TransposePlan {
  size_t off_cnt, off_tiles, off_cursor, total;
  size_t off_ka, off_kb, off_hist, off_offs, off_htiles, sort_total;  // sorting
  int64_t ntiles, rtiles, hist_n;
};
TransposePlan transpose_plan(int64_t n, int64_t m) {
  TransposePlan p{};
  size_t at = 0;
  auto take = [&](size_t bytes) {
    size_t o = at;
    at = align_up(at + std::max<size_t>(bytes, 1));
    return o;
  };
  p.ntiles = (std::max<int64_t>(n, 1) + SCAN_TILE - 1) / SCAN_TILE;
  p.off_cnt = take(4 * (size_t)std::max<int64_t>(n, 1));
  p.off_tiles = take(8 * (size_t)p.ntiles);
  p.off_cursor = take(8 * (size_t)std::max<int64_t>(n, 1));
  p.total = p.sort_total = at;
  if (n > 0 && m >= TRANSPOSE_SORT_MIN && m <= TRANSPOSE_SORT_MAX) {
    p.rtiles = (m + RADIX_TILE - 1) / RADIX_TILE;
    p.hist_n = 256 * p.rtiles;
    p.off_ka = take(8 * (size_t)m);
    p.off_kb = take(8 * (size_t)m);
    p.off_hist = take(4 * (size_t)p.hist_n);
    p.off_offs = take(8 * (size_t)(p.hist_n + 1));
    p.off_htiles = take(8 * (size_t)((p.hist_n + SCAN_TILE - 1) / SCAN_TILE));
    p.sort_total = at;
  }
  return p;
}
}  // namespace

int kbisim_transpose_workspace_bytes(int64_t n, int64_t m, size_t *bytes) {
  if (!bytes || n < 0 || m < 0) return KBISIM_EINVAL;
  if (n >= (int64_t(1) << 31)) return KBISIM_ERANGE;
  *bytes = transpose_plan(n, m).total;
  return KBISIM_OK;
}

int kbisim_transpose_sort_bytes(int64_t n, int64_t m, size_t *bytes) {
  if (!bytes || n < 0 || m < 0) return KBISIM_EINVAL;
  if (n >= (int64_t(1) << 31)) return KBISIM_ERANGE;
  *bytes = transpose_plan(n, m).sort_total;
  return KBISIM_OK;
}

int kbisim_transpose(int64_t n, int64_t m, const int64_t *row_ptr, const int32_t *col, const int32_t *elabel,
                     int64_t *out_row_ptr, int32_t *out_col, int32_t *out_elabel, void *workspace, size_t ws_bytes,
                     void *stream) {
  if (n < 0 || m < 0 || !row_ptr || !out_row_ptr || (m > 0 && (!col || !out_col))) return KBISIM_EINVAL;
  if (n >= (int64_t(1) << 31)) return KBISIM_ERANGE;
  const TransposePlan p = transpose_plan(n, m);
  if (!workspace || ws_bytes < p.total) return KBISIM_ENOSPACE;
  hipStream_t s = (hipStream_t)stream;
  char *w = (char *)workspace;
  int *cnt = (int *)(w + p.off_cnt);
  int64_t *tiles = (int64_t *)(w + p.off_tiles);
  unsigned long long *cursor = (unsigned long long *)(w + p.off_cursor);
  u32 *err = (u32 *)(w + p.off_tiles);  // scratch words (error bits, largest label), reused by the scan afterwards
  if (n == 0) {
    if (m > 0) return KBISIM_EGRAPH;
    k_fill_u64<<<1, 64, 0, s>>>((u64 *)out_row_ptr, 1, 0);
    HIP_TRY(hipGetLastError());
    HIP_TRY(hipStreamSynchronize(s));
    return KBISIM_OK;
  }
  // validate the input (row offsets monotone from 0 to m, targets in range); the
  // largest label is asked for only where entries may be sorted (it takes 5 us)
  const bool sortable = p.sort_total > p.total && ws_bytes >= p.sort_total;
  k_fill_i32<<<1, 64, 0, s>>>((int *)err, 2, 0);
  k_validate_rows<<<blocks_for(n + 1, 256), 256, 0, s>>>(n, m, row_ptr, err, ERR_GRAPH_ROWPTR);
  if (m > 0) {
    validate_vals(s, m, col, n, err, ERR_GRAPH_COL);
    if (elabel) validate_vals(s, m, elabel, -1, err, ERR_GRAPH_ELABEL, sortable ? err + 1 : nullptr);
  }
  HIP_TRY(hipGetLastError());
  u32 bad[2] = {0, 0};
  HIP_TRY(hipMemcpyAsync(bad, err, sizeof bad, hipMemcpyDeviceToHost, s));
  HIP_TRY(hipStreamSynchronize(s));
  if (bad[0]) return KBISIM_EGRAPH;
  k_fill_i32<<<blocks_for(n, 256), 256, 0, s>>>(cnt, n, 0);
  // Sorted by target when the workspace holds the keys and (target, label,
  // source) fit 64 bits: entries move in runs, where the scatter pays a
  // device-wide atomic and two stray writes per entry (40M entries: 1.0 ms
  // against 6.1).
  const u32 sb = (u32)std::max(1, bit_width((uint64_t)(n - 1)));
  const u32 lb = elabel && out_elabel ? (u32)bit_width(bad[1]) : 0u;
  if (sortable && 2 * sb + lb <= 64) {
    u64 *ka = (u64 *)(w + p.off_ka), *kb = (u64 *)(w + p.off_kb);
    k_transpose_keys<<<blocks_for(m, TKEY_CHUNK), 256, 0, s>>>(n, m, row_ptr, col, lb ? elabel : nullptr, sb, lb, ka);
    HIP_TRY(hipGetLastError());
    int rc = radix_sort(s, m, ka, kb, (int)(sb + lb), (int)(2 * sb + lb), p.rtiles, (int *)(w + p.off_hist),
                        (int64_t *)(w + p.off_htiles), (int64_t *)(w + p.off_offs));
    if (rc) return rc;
    k_transpose_unpack<<<blocks_for(m, 256), 256, 0, s>>>(m, ka, sb, lb, out_col, out_elabel, cnt);
    HIP_TRY(hipGetLastError());
    if ((rc = scan64(s, n, cnt, tiles, out_row_ptr))) return rc;
    HIP_TRY(hipStreamSynchronize(s));
    return KBISIM_OK;
  }
  if (m > 0) k_indegree<<<(unsigned)std::min<int64_t>(blocks_for(m, INDEG_CHUNK), 65536), 256, 0, s>>>(m, col, cnt);
  k_sum_tiles64<<<(unsigned)p.ntiles, 256, 0, s>>>(n, cnt, tiles);
  k_scan_tiles64<<<1, 256, 0, s>>>(p.ntiles, tiles);
  k_write_ptr64<false><<<(unsigned)p.ntiles, 256, 0, s>>>(n, cnt, tiles, out_row_ptr, cursor);
  if (m > 0)
    k_transpose_scatter<<<(unsigned)std::min<int64_t>(blocks_for(n * WAVE, 256), 65536), 256, 0, s>>>(
        n, row_ptr, col, elabel, cursor, out_col, out_elabel);
  HIP_TRY(hipGetLastError());
  HIP_TRY(hipStreamSynchronize(s));
  return KBISIM_OK;
}

namespace {
struct QuotientPlan {
  size_t off_a, off_b, off_hist, off_offs, off_tiles, off_count, off_pos, off_word, off_tgt, total;
  int64_t rtiles, hist_n, htiles, runs;
};
QuotientPlan quotient_plan(int64_t n, int64_t m) {
  QuotientPlan p{};
  size_t at = 0;
  auto take = [&](size_t bytes) {
    size_t o = at;
    at = align_up(at + std::max<size_t>(bytes, 1));
    return o;
  };
  const int64_t M = std::max<int64_t>(m, 1);
  p.rtiles = (M + RADIX_TILE - 1) / RADIX_TILE;
  p.hist_n = 256 * p.rtiles;
  p.htiles = (p.hist_n + SCAN_TILE - 1) / SCAN_TILE;
  p.runs = (M + RUN_TILE - 1) / RUN_TILE;  // at most hist_n: their scan fits the sort's tiles
  p.off_a = take(8 * (size_t)M);
  p.off_b = take(8 * (size_t)M);
  p.off_hist = take(4 * (size_t)p.hist_n);
  p.off_offs = take(8 * (size_t)(p.hist_n + 1));
  p.off_tiles = take(8 * (size_t)p.htiles);
  p.off_count = take(4 * (size_t)p.runs);
  p.off_pos = take(8 * (size_t)(p.runs + 1));
  p.off_word = take(16);
  p.off_tgt = take(4 * (size_t)std::max<int64_t>(n, 1));
  p.total = at;
  return p;
}

// One summary key per CSR entry, over the degree schedule of the context.
extern "C++" template <class Src>
int quotient_keys(kbisim_ctx *c, const Src &src, const int32_t *src_pid, const int32_t *tgt, QKey q, u64 *keys) {
  const Schedule &S = c->sched;
  hipStream_t st = c->stream;
  if (S.nranges) {
    if (S.range_edges == 1024)
      k_quotient_range<Src, 1024><<<(unsigned)S.nranges, 256, 0, st>>>(src, c->ranges, c->nzv, c->nzrow, src_pid, tgt, q,
                                                                      keys);
    else
      k_quotient_range<Src, 2048><<<(unsigned)S.nranges, 256, 0, st>>>(src, c->ranges, c->nzv, c->nzrow, src_pid, tgt, q,
                                                                      keys);
  }
  const int nrows = S.nbig + S.nrow8 + S.nrow20;
  if (nrows) k_quotient_rows<Src><<<(unsigned)nrows, 256, 0, st>>>(src, c->ranges + S.nranges, src_pid, tgt, q, keys);
  const int *hubs = c->lists + S.hub_off;
  if (S.nchunks)
    k_quotient_hubs<Src, HubChunk><<<(unsigned)S.nchunks, 256, 0, st>>>(src, c->chunks, hubs, src_pid, tgt, q, keys);
  if (S.ngchunks)
    k_quotient_hubs<Src, HubGChunk><<<(unsigned)S.ngchunks, 256, 0, st>>>(src, c->gchunks, hubs, src_pid, tgt, q,
                                                                          keys);
  HIP_TRY(hipGetLastError());
  return 0;
}

}  // namespace

int kbisim_quotient_workspace_bytes(kbisim_ctx *c, size_t *bytes) {
  if (!c || !bytes || c->num_graphs > 0) return KBISIM_EINVAL;
  *bytes = quotient_plan(c->g.n, c->g.m).total;
  return KBISIM_OK;
}

int kbisim_quotient(kbisim_ctx *c, const int32_t *src_pid, const int32_t *dst_pid, int32_t *out_src,
                    int32_t *out_label, int32_t *out_dst, int64_t *out_count, void *workspace, size_t ws_bytes) {
  if (!c || c->num_graphs > 0 || !src_pid || !dst_pid || !out_count) return KBISIM_EINVAL;
  const int64_t n = c->g.n, m = c->g.m;
  *out_count = 0;
  if (m == 0) return KBISIM_OK;
  if (!out_src || !out_label || !out_dst) return KBISIM_EINVAL;
  const QuotientPlan p = quotient_plan(n, m);
  if (!workspace || ws_bytes < p.total) return KBISIM_ENOSPACE;
  hipStream_t s = c->stream;
  char *w = (char *)workspace;
  u64 *ka = (u64 *)(w + p.off_a), *kb = (u64 *)(w + p.off_b);
  int *hist = (int *)(w + p.off_hist);
  int64_t *offs = (int64_t *)(w + p.off_offs), *tiles = (int64_t *)(w + p.off_tiles);
  int *count = (int *)(w + p.off_count);
  int64_t *pos = (int64_t *)(w + p.off_pos);
  u32 *word = (u32 *)(w + p.off_word);  // [0] error bits, [1] max source id, [2] max target id
  int rc = 0;
  // both partitions must hold ids in [0, n)
  k_fill_i32<<<1, 64, 0, s>>>((int *)word, 4, 0);
  validate_vals(s, n, src_pid, n, word, ERR_BAD_PID, word + 1);
  validate_vals(s, n, dst_pid, n, word, ERR_BAD_PID, word + 2);
  HIP_TRY(hipGetLastError());
  u32 hw[3] = {0, 0, 0};
  HIP_TRY(hipMemcpyAsync(hw, word, sizeof hw, hipMemcpyDeviceToHost, s));
  HIP_TRY(hipStreamSynchronize(s));
  if (hw[0]) return KBISIM_EINVAL;
  QKey q;
  q.db = (u32)std::max(1, bit_width(hw[2]));
  q.lb = c->g.elabel ? (u32)bit_width(c->max_label) : 0u;
  const int sbits = std::max(1, bit_width(hw[1]));
  const int total_bits = sbits + (int)q.lb + (int)q.db;
  if (total_bits > 64) return KBISIM_ERANGE;
  // target blocks in rank order, then one key per entry over the schedule
  int32_t *tgt = (int32_t *)(w + p.off_tgt);
  k_scatter_rank<<<blocks_for(n, 256), 256, 0, s>>>((int)n, dst_pid, c->rank, tgt);
  HIP_TRY(hipGetLastError());
  const int32_t *lab = separate_labels(c) ? sep_labels(c) : nullptr;
  if (lab) rc = quotient_keys(c, GraphSrcT<true>{c->g.row_ptr, c->gcol, lab, tgt, src_pid, c->pb, c->rbits}, src_pid,
                             tgt, q, ka);
  else rc = quotient_keys(c, GraphSrcT<false>{c->g.row_ptr, c->gcol, nullptr, tgt, src_pid, c->pb, c->rbits}, src_pid,
                         tgt, q, ka);
  if (rc) return rc;
  if ((rc = radix_sort(s, m, ka, kb, 0, total_bits, p.rtiles, hist, tiles, offs))) return rc;
  k_run_count<<<(unsigned)p.runs, 256, 0, s>>>(m, ka, count);
  HIP_TRY(hipGetLastError());
  if ((rc = scan64(s, p.runs, count, tiles, pos))) return rc;
  k_quotient_write<<<(unsigned)p.runs, 256, 0, s>>>(m, ka, pos, q, out_src, out_label, out_dst);
  HIP_TRY(hipGetLastError());
  HIP_TRY(hipMemcpyAsync(out_count, pos + p.runs, 8, hipMemcpyDeviceToHost, s));
  HIP_TRY(hipStreamSynchronize(s));
  return KBISIM_OK;
}

}  // extern "C"

// ---------------------------------------------------------------- no-allocation entry point
// Scratch for kbisim_refine_noalloc: one array per GPU, held from the
// library's load on that GPU until the process ends.  In host code its name
// stands for the symbol only; its device address comes from
// hipGetSymbolAddress, once per device, with that device current.
constexpr size_t NOALLOC_SCRATCH_BYTES = size_t(128) << 20;
static __device__ __align__(256) unsigned char scratch[NOALLOC_SCRATCH_BYTES];

namespace {
constexpr int NOALLOC_MAX_DEVICES = 64;
void *g_scratch_ptr[NOALLOC_MAX_DEVICES] = {};
std::mutex &scratch_mu() {
  static std::mutex *m = new std::mutex();
  return *m;
}

// Device address of the current device's scratch array (looked up on the
// first call on that device).
int scratch_address(void **out) {
  int dev = -1;
  HIP_TRY(hipGetDevice(&dev));
  if (dev < 0 || dev >= NOALLOC_MAX_DEVICES) return KBISIM_EINTERNAL;
  std::lock_guard<std::mutex> lk(scratch_mu());
  if (!g_scratch_ptr[dev]) {
    void *p = nullptr;
    const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return hip_fail(e);
    if (!p) return KBISIM_EINTERNAL;
    g_scratch_ptr[dev] = p;
  }
  *out = g_scratch_ptr[dev];
  return 0;
}
}  // namespace

extern "C" {

size_t kbisim_noalloc_scratch_bytes(void) { return NOALLOC_SCRATCH_BYTES; }

int kbisim_refine_noalloc(const kbisim_graph *g, int k, int32_t *const *out_block_ids, int64_t *out_counts,
                          void *stream) {
  int rc = check_sizes(g);
  if (rc) return rc;
  if (k < 0 || k > (1 << 20)) return KBISIM_EINVAL;
  if (k > 0 && (!out_block_ids || !out_counts)) return KBISIM_EINVAL;
  const size_t need = make_plan(g->n, g->m, g->vlabel_ptr ? g->nlabels : 0, k, 0).total;
  if (need > NOALLOC_SCRATCH_BYTES) return KBISIM_ENOSPACE;
  void *ws = nullptr;
  if ((rc = scratch_address(&ws))) return rc;
  kbisim_ctx *c = nullptr;
  if ((rc = create_impl(g, k, nullptr, ws, NOALLOC_SCRATCH_BYTES, stream, 0, nullptr, &c))) return rc;
  rc = refine_impl(c, nullptr, k, out_block_ids, out_counts);
  kbisim_destroy(c);
  return rc;
}

const char *kbisim_strerror(int code) {
  switch (code) {
    case KBISIM_OK: return "ok";
    case KBISIM_EINVAL: return "invalid argument";
    case KBISIM_EGRAPH: return "graph validation failed";
    case KBISIM_ENOSPACE: return "workspace too small";
    case KBISIM_EHIP: return g_hip_msg[0] ? g_hip_msg : "HIP runtime error";
    case KBISIM_ERANGE: return "size out of range";
    case KBISIM_EINTERNAL: return "internal consistency check failed";
    default: return "unknown error";
  }
}

const char *kbisim_version(void) { return "kbisim 0.3 gfx950"; }

}  // extern "C"
