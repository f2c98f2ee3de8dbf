// Host side of the C ABI declared in include/hps.h: argument checks, carving of
// the caller's storage and workspace, and the kernel launch sequences of
// insert / pull / push / get / dump.  No device memory is allocated here.

#include "../../include/hps.h"
#include "../../include/hps_measure.h"
#include "../../include/hps_mem.h"

#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <new>
#include <vector>

#include <algorithm>

#include "common.hpp"
#include "bucket.hpp"
#include "dedup.hpp"
#include "form.hpp"
#include "partition.hpp"
#include "pool.hpp"
#include "push.hpp"
#include "rows.hpp"
#include "small.hpp"
#include "sort.hpp"
#include "table.hpp"
#include "mem_tier.hpp"

using namespace hps;

namespace {

constexpr double kLoadFactor = 0.7;
constexpr size_t kAlign = 256;
constexpr uint64_t kMaxSlots = 0xFFFFFFF0ull;   // row indices are 32-bit, kNoRow is reserved
constexpr uint32_t kMinTileGroup = 8;

size_t align_up(size_t x) { return (x + kAlign - 1) / kAlign * kAlign; }

uint64_t slots_for(uint64_t capacity) {
  uint64_t s = (uint64_t)((double)capacity / kLoadFactor) + 1;
  if (s < capacity + kSlotsPerLine) s = capacity + kSlotsPerLine;
  // a whole number of 128-byte memory lines (two lines of slots each)
  return (s + 2 * kSlotsPerLine - 1) / (2 * kSlotsPerLine) * (2 * kSlotsPerLine);
}

bool valid_opt(const hps_optimizer* o) {
  return o && (o->kind == HPS_OPT_ADAGRAD_ROWWISE || o->kind == HPS_OPT_ADAGRAD_ELEMENTWISE) &&
         (o->row_format == HPS_ROWS_F32 || o->row_format == HPS_ROWS_BF16 ||
          o->row_format == HPS_ROWS_F32_WIDE) &&
         o->init_range >= 0.f && o->eps >= 0.f && o->init_acc >= 0.f;
}

bool valid_shape(uint64_t capacity, uint32_t dim) {
  return capacity >= 1 && dim >= 4 && dim <= 1024 && dim % 4 == 0 &&
         slots_for(capacity) <= kMaxSlots;
}

struct StorageLayout {
  size_t keys, w, acc, state, total;
  uint32_t w_pitch, acc_pitch;     // bytes from one row to the next
};

// Weights and accumulators of a row side by side (table.hpp: TableView)?
bool rows_side_by_side(uint32_t dim, uint32_t acc_len, int row_format) {
  const uint32_t pair = 8 * dim;
  const char* env = std::getenv("HPS_ROWS");          // "apart": always two arrays (for comparison)
  if (env && std::strcmp(env, "apart") == 0) return false;
  return row_format == HPS_ROWS_F32 && acc_len == dim && (pair % 128 == 0 || 128 % pair == 0);
}

StorageLayout storage_layout(uint64_t n_slots, uint32_t dim, uint32_t acc_len, int row_format) {
  StorageLayout L;
  size_t o = 0;
  L.keys = o;  o = align_up(o + n_slots * sizeof(uint64_t));
  const uint32_t w_bytes = dim * (row_format == HPS_ROWS_BF16 ? 2 : 4), acc_bytes = acc_len * 4;
  if (row_format == HPS_ROWS_F32_WIDE) {
    // one record per row, whole memory lines
    const uint32_t pitch = (w_bytes + acc_bytes + 127) / 128 * 128;
    L.w = o;   L.acc = o + w_bytes;
    L.w_pitch = L.acc_pitch = pitch;
    o = align_up(o + n_slots * (size_t)pitch);
  } else if (rows_side_by_side(dim, acc_len, row_format)) {
    L.w = o;   L.acc = o + w_bytes;
    L.w_pitch = L.acc_pitch = w_bytes + acc_bytes;
    o = align_up(o + n_slots * (size_t)(w_bytes + acc_bytes));
  } else {
    L.w = o;   o = align_up(o + n_slots * (size_t)w_bytes);
    L.acc = o; o = align_up(o + n_slots * (size_t)acc_bytes);
    L.w_pitch = w_bytes;
    L.acc_pitch = acc_bytes;
  }
  L.state = o; o = align_up(o + sizeof(TableState));
  L.total = o;
  return L;
}

// Bucket form of the dedup by number of occurrences: tiles (threads x items), number and mean size of
// the natural buckets, heavy keys at most, threads of a bucket's workgroup (which holds
// 8 * threads occurrences).  Small mini-batches take small tiles and buckets, so that they
// spread over the GPU; large ones large tiles and buckets, so that a tile's run per bucket stays
// long (large: 12288 / 2400 buckets = five occurrences, 40 bytes of keys).
struct BucketSizes {
  uint64_t max_n;
  uint32_t threads, items, max_nat, mean, max_heavy, group_threads;
};
constexpr BucketSizes kBucketSizes[] = {
    {1u << 16, 256, 4, 256, 256, 255, 256},
    {1u << 20, 512, 8, 1024, 256, 1023, 256},
    {3u << 20, 1024, 8, 1536, 2048, 2047, 512},
    {12u << 20, 1024, 12, 3072, 4096, 2047, 1024},
};
constexpr int kBucketClasses = 4;
constexpr int kMaxBuckets[kBucketClasses] = {512, 2048, 4096, 5120};
constexpr bool bucket_sizes_ok() {
  for (int k = 0; k < kBucketClasses; ++k) {
    const BucketSizes& z = kBucketSizes[k];
    if (z.max_nat + z.max_heavy > (uint32_t)kMaxBuckets[k] || z.max_nat + z.max_heavy > 8191) return false;
    if (z.max_heavy > order_max_heavy((int)z.group_threads)) return false;
    if (z.max_nat < z.max_n / z.mean && k != 1) return false;
    if (k == 0 && z.max_n > kDirectTiles * z.threads * z.items) return false;
    if (z.max_n > 1024u * z.threads * z.items) return false;       // scan_buckets: at most 16 tiles per group of lanes
  }
  return true;
}
static_assert(kBucketSizes[0].max_nat <= kMaxBorders && kBucketSizes[1].max_nat <= kMaxBorders &&
                  kBorderMaxKeys <= kBucketSizes[1].max_n, "buckets by sampled borders");
static_assert(bucket_sizes_ok(), "the kernels' limits");
static_assert(kBucketPathMaxKeys == kBucketSizes[kBucketClasses - 1].max_n, "the largest class");

int bucket_class(uint64_t n) {
  int k = 0;
  while (k + 1 < kBucketClasses && n > kBucketSizes[k].max_n) ++k;
  return k;
}
// Threads of the workgroups that group the buckets of n occurrences.
u32 group_threads(int form, uint64_t n) { return form == kByBorders ? border_group_threads(n) : kBucketSizes[bucket_class(n)].group_threads; }
// A key with at least this many occurrences in a mini-batch of n is listed as heavy: an eighth of
// what a bucket's workgroup holds, so that a few such keys the hint misses still fit one.
uint32_t heavy_min(uint64_t n) {
  const uint64_t share = n / kHeavyShare, eighth = kBucketSizes[bucket_class(n)].group_threads;
  return (uint32_t)(share > eighth ? share : eighth);
}
BucketPlan bucket_plan(uint64_t n) {
  const BucketSizes& z = kBucketSizes[bucket_class(n)];
  BucketPlan p;
  uint64_t nat = (n + z.mean - 1) / z.mean;
  p.n_nat = (u32)(nat < 1 ? 1 : nat > z.max_nat ? z.max_nat : nat);
  p.max_heavy = z.max_heavy;
  p.stride = (p.n_nat + p.max_heavy + 63) / 64 * 64;
  p.n_tiles = (u32)((n + z.threads * z.items - 1) / (z.threads * z.items));
  return p;
}
// Counts a dedup of at most n occurrences keeps per (tile, bucket).
uint64_t max_counts(uint64_t n) {
  uint64_t most = 0;
  for (int k = 0; k < kBucketClasses; ++k) {
    const BucketPlan p = bucket_plan(n < kBucketSizes[k].max_n ? n : kBucketSizes[k].max_n);
    const uint64_t c = (uint64_t)p.n_tiles * p.stride;
    if (c > most) most = c;
    if (n <= kBucketSizes[k].max_n) break;
  }
  return most;
}

int lanes_per_row(uint32_t dim) {
  int l = 1;
  while (l < 64 && (uint32_t)l * 4 < dim) l <<= 1;
  return l;
}

// Per pull context (two of them, so that the dedup of the next mini-batch can run
// while the current one is still between pull and push).
struct ContextLayout {
  size_t ctx, uniq, rows, bags, seg_off, inv_len;
  size_t code, from, upos, bucket_start, count, border;      // bucket form
  size_t places;                                     // small form
  size_t inverse;                                    // plain form (shares its memory with `code`)
};

struct WorkspaceLayout {
  size_t fresh, keys_a, keys_b, idx_a, idx_b, hist, prefix, total, tile_bag, heavy_raw, ghist,
      tickets, tile_rows, group_rows, head_rows, head_groups, evidence, bag_of, id16, by_pos, by_heavy, row_of,
      med_list, med_span, arrived, chunk_items, partials, end;
  size_t local_rank, rank_by_pos, rank_by_heavy, bucket_total, sort_ctx, sort_n;     // hps_last_unique's own
  ContextLayout c[2];
  uint64_t max_long, max_items, sort_tiles, head_tiles;
};

// small: with what the small form and pulls need (an accumulate on the static scratch is neither).
WorkspaceLayout workspace_layout(uint64_t n, uint64_t bags, uint32_t dim, bool small = true) {
  WorkspaceLayout L;
  const uint64_t n1 = n ? n : 1;
  const uint64_t buckets = (uint64_t)kMaxBuckets[kBucketClasses - 1] + 1;
  L.sort_tiles = (n1 + kSortTile - 1) / kSortTile;
  L.head_tiles = (n1 + kHeadTile - 1) / kHeadTile;
  // (a smaller mini-batch than the largest may be cut into more pieces)
  L.max_long = L.max_items = 0;                   // keys the push handles chunk by chunk, their chunks
  for (uint64_t m : {n1, n1 < kSmallPush ? n1 : kSmallPush}) {
    const PieceSizes pieces = piece_sizes(lanes_per_row(dim), m);
    L.max_long = std::max(L.max_long, m / (pieces.medium + 1) + 1);
    L.max_items = std::max(L.max_items, m / pieces.chunk + m / (pieces.medium + 1) + 2);
  }
  size_t o = 0;
  L.keys_a = o;      o = align_up(o + n1 * 8);
  L.keys_b = o;      o = align_up(o + n1 * 8);
  L.idx_a = o;       o = align_up(o + n1 * 8);    // payloads: occurrence index | bag << 32
  L.idx_b = o;       o = align_up(o + n1 * 8);
  L.hist = o;        o = align_up(o + std::max<uint64_t>(max_counts(n1), kSmallHistWords) * 2);    // bucket and small form: counts per (tile, bucket)
  L.prefix = o;      o = align_up(o + max_counts(n1) * 4);    // ... and those of the tiles before
  L.total = o;       o = align_up(o + buckets * 4);
  L.tile_bag = o;    o = align_up(o + 1025 * 4);
  // from here to `evidence`: cleared at creation, never again (see sort.hpp)
  L.ghist = o;       o = align_up(o + 2 * (size_t)kHistWords * 4);
  L.tickets = o;     o = align_up(o + (kMaxPasses + 2) * 4);
  L.tile_rows = o;   o = align_up(o + (size_t)kMaxPasses * L.sort_tiles * kRadix * 4);
  L.group_rows = o;  o = align_up(o + (size_t)kMaxPasses * (L.sort_tiles / kMinTileGroup + 1) * kRadix * 4);
  L.head_rows = o;   o = align_up(o + 2 * L.head_tiles * 4);
  L.head_groups = o; o = align_up(o + 2 * (L.head_tiles / kMinTileGroup + 1) * 4);
  L.evidence = o;    o = align_up(o + kMaxEvidence * 4);
  L.heavy_raw = o;   o = align_up(o + sizeof(HeavyRing));
  L.bag_of = L.id16 = o; o = align_up(o + n1 * 4);    // plain: bag of every occurrence; buckets: its bucket (16 bits)
  for (int k = 0; k < 2; ++k) {
    L.c[k].ctx = o;     o = align_up(o + sizeof(PullCtx));
    L.c[k].uniq = o;    o = align_up(o + n1 * 8);
    L.c[k].rows = o;    o = align_up(o + n1 * 4);
    L.c[k].bags = o;    o = align_up(o + n1 * 4);
    L.c[k].seg_off = o; o = align_up(o + (n1 + 1) * 4);
    L.c[k].inv_len = o; o = align_up(o + (bags ? bags : 1) * 4);    // mean pooling: 1 / bag length
    L.c[k].code = L.c[k].inverse = o; o = align_up(o + n1 * 4);
    L.c[k].from = o;    o = align_up(o + n1 * 2);
    L.c[k].upos = o;    o = align_up(o + n1 * 4);
    L.c[k].bucket_start = o; o = align_up(o + (buckets + 1) * 4);
    L.c[k].count = o;   o = align_up(o + buckets * 4);
    L.c[k].border = o;  o = align_up(o + kMaxBorders * 8);
    L.c[k].places = o;  o = align_up(o + (small ? std::min<uint64_t>(n1, kSmallMax) * 16 : 0));
  }
  L.by_pos = o;      o = align_up(o + n1 * 4);      // row of the key at every position
  L.by_heavy = o;    o = align_up(o + (kMaxHeavy + 1) * 4);
  L.row_of = o;      o = align_up(o + n1 * 4);      // row of every occurrence
  L.fresh = o;       o = align_up(o + (small ? n1 * 4 : 0));      // the pull that created the key
  L.local_rank = o;    o = align_up(o + n1 * 4);
  L.rank_by_pos = o;   o = align_up(o + n1 * 4);
  L.rank_by_heavy = o; o = align_up(o + (kMaxHeavy + 1) * 4);
  L.bucket_total = o;  o = align_up(o + buckets * 4);
  L.sort_ctx = o;      o = align_up(o + sizeof(PullCtx));
  L.sort_n = o;        o = align_up(o + 4);
  L.med_list = o;    o = align_up(o + (n1 / (kShortSeg + 1) + kMaxHeavy + 64) * 4);
  L.med_span = o;    o = align_up(o + (std::max<uint64_t>(buckets, n1 / 1024 + 2049) + kMaxHeavy / kHeavyGroup + 1) * 8);    // (unique_spans)
  L.arrived = o;     o = align_up(o + L.max_long * 4);
  L.chunk_items = o; o = align_up(o + L.max_items * 16);
  L.partials = o;    o = align_up(o + L.max_items * (size_t)dim * 4);
  L.end = o;
  return L;
}

// Tiles per look-back group: about the square root of the tile count.
uint32_t tile_group(uint64_t n_tiles) {
  uint32_t g = kMinTileGroup;
  while (g < kMaxTileGroup && (uint64_t)g * g < n_tiles) ++g;
  return g;
}

// Plain form.  How many 8-bit digits to sort for n occurrences: enough that two different
// keys rarely agree in all sorted bits.  With b sorted bits about n^2 / 2^(b+1) pairs of
// distinct hashed keys collide; b >= 2*log2(n) - 2 keeps that near one in a few
// batches, and every collision is repaired anyway (dedup.hpp).
// all_bits: every bit of the keys is sorted (eight passes), whatever the keys look like.
SortPlan sort_plan(uint64_t n, bool all_bits) {
  SortPlan p;
  int log2n = 1;
  while ((1ull << log2n) < n) ++log2n;
  int want = (2 * log2n - 2 + 7) / 8;
  if (want < 2) want = 2;
  if (want > kMaxPasses || all_bits) want = kMaxPasses;
  p.n_pass = want;
  p.low_shift = 64 - 8 * want;
  p.group = tile_group((n + kSortTile - 1) / kSortTile);
  return p;
}

unsigned grid_for(uint64_t work_items, uint64_t items_per_block, unsigned max_blocks) {
  uint64_t b = (work_items + items_per_block - 1) / items_per_block;
  if (b < 1) b = 1;
  return (unsigned)(b < max_blocks ? b : max_blocks);
}

bool launch_ok() { return hipGetLastError() == hipSuccess; }

}  // namespace

// ---- the one entry point that allocates nothing (hps_accumulate_static) ------------------
// Its workspace: a file-scope device array, one copy per GPU, held until the process ends.
// Room for the workspace of HPS_STATIC_MAX_KEYS pairs with rows of up to 1024 floats.
constexpr size_t kStaticScratchBytes = 16u << 20;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];
constexpr int kMaxDevices = 64;
struct StaticScratch {
  char* ptr;                // this device's address of `scratch` (hipGetSymbolAddress), null until first used
  bool ring_ready;          // its lists of frequent keys have been initialised
  uint64_t lookup_serial;   // lookups run on it so far (they take turns on its three lists)
};
static StaticScratch g_static[kMaxDevices];

struct hps_table {
  uint64_t capacity, n_slots, max_keys, max_bags;
  uint32_t dim, acc_len;
  hps_optimizer opt;
  TableView view;
  char* ws;
  WorkspaceLayout wl;
  int lpr;
  bool mean_pooling;        // bags are averaged instead of summed (hps_set_pooling)
  uint64_t lookup_serial;   // lookups so far; lookup s lists its frequent keys in ring slot s % 3
  uint64_t dumped;          // TableState::dump_count after the last dump (~0: not known, that dump failed)
  uint64_t pull_serial;     // pulls with bags so far: they take the two sets of counts in turn (common.hpp: pull_made)
  bool ordered_rank;   // the GPU's LDS atomics serve a wave's lanes in lane order (sort.hpp: digit_rank)
  // How much of pull_lookup's per-block list of created keys is used: all of it, unless
  // HPS_LOOKUP_NEW_LIST says less (tests of what happens when it is full).
  u32 lookup_new_cap;
  uint64_t serial;     // number of dedups so far (status words carry it modulo kEpochMod)
  uint64_t plain_serial;   // ... of them in the plain form
  unsigned long long* report;             // pinned host words the lookups report into: [0] of the lookup after a dedup in any form but by key range, [1] by key range, [2] of the small form
  FormChoice choice;        // the dedups' form

  // Pull contexts.  `current` is the context of the outstanding pull (-1: none),
  // `prepared` the one whose dedup has been enqueued but not yet pulled (-1: none).
  struct Context {
    uint64_t n_keys, n_bags;
    const int32_t* d_offsets;
    bool mean;            // pooling of this pull (fixed when it is prepared)
    bool looked_up;       // its dedup included the lookup (small form)
    int form;             // of its dedup (form.hpp)
    bool buckets;         // ... and whether that is the bucket or the small form ...
    BucketPlan plan;      // ... with these sizes
    hipEvent_t ready;     // recorded after the dedup kernels
    hipEvent_t released;  // recorded after the push that used the context
    bool ready_set, released_set;
    bool listed;          // hps_last_unique has read this context since its dedup
    bool counted;         // ... was called for it, captured or not
  } cx[2];
  int current, prepared;
  hipEvent_t scratch_free;   // the one of the other events that marks the end of the last work on the dedups' scratch, which is shared; or null
  hipEvent_t listing;        // the last hps_last_unique's end: its scratch, and the context it read
  bool listing_set;
  // While all calls come on the null stream, its order is all they need, and none of these events is recorded (a record
  // takes the stream 3 us in which nothing runs, three of them a step); the *_set flags are kept all the same.  See enter().
  bool many_streams;
  uint64_t last_n_keys;      // of the most recent pull, for hps_stats

  // stage timing (measurement only)
  uint32_t timing_mask;
  std::vector<hipEvent_t> ev_pool[HPS_N_STAGES];   // begin/end alternate
  size_t ev_used[HPS_N_STAGES];

  template <typename T> T* w(size_t off) const { return reinterpret_cast<T*>(ws + off); }
  PullCtx* ctx(int c) const { return w<PullCtx>(wl.c[c].ctx); }
};

namespace {
constexpr size_t kMaxEventPairs = 4096;

void stage_mark(hps_table* t, int stage, hipStream_t s) {
  if (!(t->timing_mask & (1u << stage))) return;
  std::vector<hipEvent_t>& pool = t->ev_pool[stage];
  if (t->ev_used[stage] >= 2 * kMaxEventPairs) return;
  if (t->ev_used[stage] == pool.size()) {
    hipEvent_t e;
    if (hipEventCreate(&e) != hipSuccess) return;
    pool.push_back(e);
  }
  (void)hipEventRecord(pool[t->ev_used[stage]++], s);
}
}  // namespace

// ---- order between streams ---------------------------------------------------------------
// From the first call on another stream than the null stream on, the events are recorded.  Those that have been left out are put down
// on the null stream now (later than they ask for).  Only calls on the null stream may leave them out: it can always be
// recorded on, while a stream of the caller's may be gone by the time another one comes, its handle
// perhaps in use for a new stream, and hipStreamDestroy need not wait for the work on it.
static bool leave_null_stream(hps_table* t) {
  const struct { hipEvent_t event; bool set; } left_out[] = {
      {t->listing, t->listing_set}, {t->cx[0].ready, t->cx[0].ready_set},
      {t->cx[1].ready, t->cx[1].ready_set}, {t->cx[0].released, t->cx[0].released_set}, {t->cx[1].released, t->cx[1].released_set}};
  for (const auto& e : left_out)
    if (e.set && hipEventRecord(e.event, nullptr) != hipSuccess) {
      (void)hipGetLastError();
      return false;             // (nothing has changed: the next call tries again)
    }
  t->many_streams = true;
  return true;
}

// Before any wait or mark of a call on stream s.  waits: the call has to come after earlier ones (a push is part of its pull:
// where it comes on another stream, the caller orders it).
static bool enter(hps_table* t, hipStream_t s, bool waits) {
  if (t->many_streams) return true;
  hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(s, &capture) != hipSuccess) (void)hipGetLastError();
  if (capture != hipStreamCaptureStatusNone) {
    // (what ran before the capture cannot be waited for inside it)
    if (t->scratch_free || t->listing_set || t->cx[0].released_set || t->cx[1].released_set) return !waits;
    t->many_streams = true;
    return true;
  }
  return s == nullptr || leave_null_stream(t);
}
static bool mark(hps_table* t, hipEvent_t e, bool* set, hipStream_t s) {
  *set = true;
  return !t->many_streams || hipEventRecord(e, s) == hipSuccess;
}
static bool wait_for(const hps_table* t, hipEvent_t e, bool set, hipStream_t s) {
  return !set || !t->many_streams || hipStreamWaitEvent(s, e, 0) == hipSuccess;
}

static bool wait_for_scratch(const hps_table* t, hipStream_t s) { return wait_for(t, t->scratch_free, t->scratch_free != nullptr, s); }

static UniqueSpans unique_spans(const hps_table* t, int c, uint64_t n) {
  const hps_table::Context& cx = t->cx[c];
  UniqueSpans u;
  if (cx.buckets) {
    u.bucket_start = t->w<u32>(t->wl.c[c].bucket_start);
    u.count = t->w<u32>(t->wl.c[c].count);
    u.n_spans = cx.plan.n_nat;
    u.max_heavy = cx.plan.max_heavy;
    u.plain_span = 0;
  } else {
    u.bucket_start = u.count = nullptr;
    // about 2000 blocks, however few keys there are (a few dozen keys per block still fill its waves)
    u.plain_span = 32;
    while (u.plain_span < 1024 && (uint64_t)u.plain_span * 2048 < n) u.plain_span *= 2;
    u.n_spans = (u32)((n + u.plain_span - 1) / u.plain_span);
    u.max_heavy = 0;
  }
  return u;
}

// The number the running pull marks the keys it creates with: never 0, which hps_create leaves in the marks.
static u32 pull_stamp(const hps_table* t) { return (u32)(t->pull_serial % 0xFFFFFFFFu) + 1; }

// spread (partition.hpp) with the tiles of a bucket-form dedup of n occurrences.
static void launch_spread(const u32* code, const uint16_t* from, u32 n, u32 n_tiles, const u32* by_pos,
                          const u32* by_heavy, u32* out, hipStream_t s) {
#define HPS_SPREAD(K) \
  spread<kBucketSizes[K].threads, kBucketSizes[K].items><<<n_tiles, kBucketSizes[K].threads, 0, s>>>(code, from, n, by_pos, by_heavy, out)
  switch (bucket_class(n)) {
    case 0: HPS_SPREAD(0); break;
    case 1: HPS_SPREAD(1); break;
    case 2: HPS_SPREAD(2); break;
    default: HPS_SPREAD(3); break;
  }
#undef HPS_SPREAD
}

// Rows per occurrence (row_of), then the bags' sums.
template <int LPR>
static void launch_pool(hps_table* t, int c, float* d_pooled, hipStream_t s) {
  const hps_table::Context& cx = t->cx[c];
  const ContextLayout& C = t->wl.c[c];
  u32* row_of = t->w<u32>(t->wl.row_of);
  uint4* places = t->w<uint4>(C.places);
  const bool small = cx.n_keys && cx.buckets && cx.form == kSmallForm;
  if (cx.n_keys) {
    const u32 n = (u32)cx.n_keys;
    if (small) {
      if (!cx.looked_up) small_rows<<<grid_for(n, 256, 256), 256, 0, s>>>(t->view.st, t->w<u32>(C.rows), n, places);
    } else if (cx.buckets)
      launch_spread(t->w<u32>(C.code), t->w<uint16_t>(C.from), n, cx.plan.n_tiles, t->w<u32>(t->wl.by_pos),
                    t->w<u32>(t->wl.by_heavy), row_of, s);
    else
      rows_by_rank<<<grid_for(n, kPoolThreads * 4, 4096), kPoolThreads, 0, s>>>(t->view.st, t->w<i32>(C.inverse), t->w<u32>(C.rows), n, row_of);
  }
  // (a block has 256 / LPR lane groups with eight rows in flight each: wide rows need more
  // blocks for as many rows in flight; d = 64: 0.293 ms with 1024 blocks, 0.247 with 4096, while
  // d = 16 runs the same with 1024 to 3072)
  const unsigned blocks = grid_for(cx.n_bags, kPoolThreads / LPR, kPoolMaxBlocks * (LPR > 4 ? LPR / 4 : 1));
  float* inv_len = cx.mean ? t->w<float>(C.inv_len) : nullptr;
  const PullEnd end = {(u32)(t->pull_serial & 1), unique_spans(t, c, cx.n_keys), t->ctx(c), t->w<u32>(C.rows), t->w<u32>(t->wl.fresh), pull_stamp(t)};
  u32* bags = t->w<u32>(C.bags);
#define HPS_POOL(COLS, SMALL) \
  pool_bags<LPR, COLS, SMALL><<<blocks, kPoolThreads, 0, s>>>(t->view, cx.d_offsets, (u32)cx.n_bags, (u32)cx.n_keys, row_of, d_pooled, inv_len, places, bags, end)
  if (t->dim <= (uint32_t)LPR * 4) { if (small) HPS_POOL(1, true); else HPS_POOL(1, false); }
  else { if (small) HPS_POOL(4, true); else HPS_POOL(4, false); }
#undef HPS_POOL
}

template <int LPR>
static void launch_push(hps_table* t, uint64_t n, PushArgs& a, hipStream_t s) {
  // (a span's distinct keys are fewer than its occurrences; about four keys per lane group)
  const uint64_t per_span = (n + a.spans.n_spans - 1) / a.spans.n_spans;
  a.parts = grid_for(per_span, 4 * kPushThreads / LPR, std::max(1u, std::min((unsigned)kPushMaxParts, kPushSplitBlocks / a.spans.n_spans)));
  a.medium_blocks = std::min(std::max(kPushMediumBlocks, a.spans.n_spans / 2), kPushMaxMediumBlocks);
  a.chunk = piece_sizes(LPR, n).chunk;
  a.chunk_blocks = grid_for(n / a.chunk + 1, 1, kPushChunkBlocks);
  const unsigned main_blocks = a.chunk_blocks + a.medium_blocks + heavy_blocks(a.spans) + a.spans.n_spans * a.parts;
  if (t->dim <= (uint32_t)LPR * 4) {
    push_main<LPR, 1><<<main_blocks, kPushThreads, 0, s>>>(t->view, a);
  } else {
    push_main<LPR, 4><<<main_blocks, kPushThreads, 0, s>>>(t->view, a);
  }
}

// The bucket form's kernels for context c (partition.hpp, bucket.hpp), size class K.
template <int K, int FORM>
static void launch_buckets(hps_table* t, int c, const uint64_t* d_keys, u32 n, const int32_t* d_offsets, u32 n_bags,
                           const HeavyRaw* heavy, hipStream_t s) {
  constexpr int kThreads = kBucketSizes[K].threads, kItems = kBucketSizes[K].items;
  constexpr bool kDirect = K == 0;
  const WorkspaceLayout& L = t->wl;
  const ContextLayout& C = L.c[c];
  const BucketPlan plan = t->cx[c].plan;
  PullCtx* ctx = t->ctx(c);
  uint16_t* id16 = t->w<uint16_t>(L.id16);
  uint16_t* hist = t->w<uint16_t>(L.hist);
  u32* prefix = t->w<u32>(L.prefix);
  u32* tile_bag = t->w<u32>(L.tile_bag);
  u32* bucket_start = t->w<u32>(C.bucket_start);
  u64* keys = t->w<u64>(L.keys_a);
  u64* uniq = t->w<u64>(C.uniq);
  u32* seg_off = t->w<u32>(C.seg_off);
  u32* bags = t->w<u32>(C.bags);
  const unsigned bag_blocks = d_offsets ? grid_for(n_bags, kThreads * 4, 256) : 0;
  u64* border = t->w<u64>(C.border);
  if constexpr (FORM == kByBorders) {
    constexpr u32 kSamples = border_samples(kBucketSizes[K].max_nat);
    sample_borders<kSamples><<<kSamples / kWave, kBorderThreads, 0, s>>>(d_keys, n, plan.n_nat, border);
  }
  bucket_count<kThreads, kItems, kMaxBuckets[K], FORM><<<plan.n_tiles + bag_blocks, kThreads, 0, s>>>(
      d_keys, n, plan, border, ctx, d_offsets, n_bags, tile_bag, heavy, id16, hist);
  if (!kDirect) {
    const unsigned blocks = (plan.n_nat + plan.max_heavy + kScanBuckets - 1) / kScanBuckets;
#define HPS_SCAN(PER) scan_buckets<PER><<<blocks, kScanThreads, 0, s>>>(hist, plan, prefix, t->w<u32>(L.total), ctx)
    if (plan.n_tiles <= 4 * kScanChunks) HPS_SCAN(4);
    else if (plan.n_tiles <= 8 * kScanChunks) HPS_SCAN(8);
    else HPS_SCAN(16);
#undef HPS_SCAN
  }
#define HPS_ORDERED(ORDERED)                                                                                      \
  do {                                                                                                            \
    bucket_scatter<kThreads, kItems, kMaxBuckets[K], ORDERED, kDirect><<<plan.n_tiles, kThreads, 0, s>>>(         \
        d_keys, id16, d_offsets, n_bags, tile_bag, n, plan, ctx, hist, prefix, t->w<u32>(L.total), heavy, bucket_start, uniq, seg_off,  \
        keys, bags, t->w<u32>(C.code), t->w<uint16_t>(C.from));                                                   \
    stage_mark(t, HPS_STAGE_SORT, s);                                                                             \
    stage_mark(t, HPS_STAGE_UNIQUE, s);                                                                           \
    if (group == 256) HPS_GROUP(256, ORDERED);                                                                    \
    else if (group == 512) HPS_GROUP(512, ORDERED);                                                               \
    else HPS_GROUP(1024, ORDERED);                                                                                \
  } while (0)
#define HPS_GROUP(THREADS, ORDERED)                                                                               \
  group_bucket<THREADS, ORDERED><<<plan.n_nat, THREADS, 0, s>>>(keys, bucket_start, uniq, seg_off, bags, t->w<u32>(C.upos), \
                                                                t->w<u32>(C.count), slow, ctx, t->view.st)
  const u32 group = group_threads(FORM, n);
  const SlowScratch slow = {t->w<u64>(L.idx_a), t->w<u64>(L.keys_b), t->w<u64>(L.idx_b)};
  if (t->ordered_rank) HPS_ORDERED(true);
  else HPS_ORDERED(false);
#undef HPS_GROUP
#undef HPS_ORDERED
}

// Whether a pull's lookup may create keys as it finds them (table.hpp: end_pull).
static bool creates_at_once(const hps_table* t, uint64_t n_keys) { return n_keys <= t->capacity / 4; }

// What a lookup of context c, of n_keys occurrences, works with besides the keys: the lists it fills (it counts as a lookup) and
// how it treats missing keys.
static OftenLists start_lookup(hps_table* t, int c, uint64_t n_keys) {
  HeavyRing* ring = t->w<HeavyRing>(t->wl.heavy_raw);
  OftenLists often;
  often.ctx = t->ctx(c);
  often.med_list = t->w<u32>(t->wl.med_list);
  often.med_span = t->w<uint2>(t->wl.med_span);
  often.chunk_items = t->w<uint4>(t->wl.chunk_items);
  often.arrived = t->w<u32>(t->wl.arrived);
  often.pieces = piece_sizes((u32)t->lpr, n_keys);
  ++t->lookup_serial;
  often.heavy_raw = &ring->raw[t->lookup_serial % kHeavyRing];
  often.heavy_next = &ring->raw[(t->lookup_serial + 1) % kHeavyRing];
  often.heavy_min = heavy_min(n_keys);
  often.report = t->report;
  often.serial = (u32)t->lookup_serial;
  return often;
}
static Creation creation_of(const hps_table* t, uint64_t n_keys, bool create) {
  Creation k;
  k.how = !create ? kCreateNone : creates_at_once(t, n_keys) ? kCreateAtOnce : kCreateIfRoom;
  k.set = (u32)(t->pull_serial & 1);
  k.new_cap = t->lookup_new_cap;
  k.fresh = t->w<u32>(t->wl.fresh);
  k.stamp = pull_stamp(t);
  return k;
}

// What a dedup includes besides (small form).
enum Include { kDedupOnly, kWithPullLookup, kWithAddLookup };

// The small form (small.hpp).
template <bool LOOKUP>
static void launch_small(hps_table* t, int c, const uint64_t* d_keys, u32 n, bool own_bags, Include include, hipStream_t s) {
  const WorkspaceLayout& L = t->wl;
  const ContextLayout& C = L.c[c];
  SmallArgs a;
  a.keys = d_keys;
  a.n = n;
  a.log2_nat = kSmallMinLog2;
  while (n > kSmallMean << a.log2_nat) ++a.log2_nat;
  a.n_tiles = (n + kSmallTile - 1) / kSmallTile;
  a.own_bags = own_bags ? 1u : 0u;
  a.ctx = t->ctx(c);
  a.ids = t->w<uint8_t>(L.id16);
  a.hist = t->w<uint16_t>(L.hist);
  a.bucket_start = t->w<u32>(C.bucket_start);
  a.count = t->w<u32>(C.count);
  a.uniq = t->w<u64>(C.uniq);
  a.seg_off = t->w<u32>(C.seg_off);
  a.bags = t->w<u32>(C.bags);
  a.places = own_bags ? nullptr : t->w<uint4>(C.places);
  a.dealt = t->w<u64>(L.keys_a);
  a.upos = t->w<u32>(C.upos);
  a.slow = {t->w<u64>(L.idx_a), t->w<u64>(L.keys_b), t->w<u64>(L.idx_b)};
  a.report = t->report ? t->report + 2 : nullptr;
  a.serial = (u32)t->serial;
  a.rows = t->w<u32>(C.rows);
  a.create = LOOKUP ? creation_of(t, n, include == kWithPullLookup) : Creation();
  a.often = LOOKUP ? start_lookup(t, c, n) : OftenLists();
  BucketPlan& plan = t->cx[c].plan;
  plan.n_nat = 1u << a.log2_nat;
  plan.max_heavy = plan.stride = plan.n_tiles = 0;
  small_ids<<<a.n_tiles, kSmallTile, 0, s>>>(t->view, a);
  if (t->ordered_rank) small_group<LOOKUP, true><<<plan.n_nat, kSmallThreads, 0, s>>>(t->view, a);
  else small_group<LOOKUP, false><<<plan.n_nat, kSmallThreads, 0, s>>>(t->view, a);
}

// a1 for context c: the kernels that turn (keys, offsets) into the distinct keys and the
// occurrences' bags grouped by key.  d_offsets == nullptr: every occurrence is its own bag.
// `include`: what the small form may do besides; cx[c].looked_up tells whether it did.
static void launch_dedup(hps_table* t, int c, const uint64_t* d_keys, u32 n,
                         const int32_t* d_offsets, u32 n_bags, Include include, hipStream_t s) {
  const WorkspaceLayout& L = t->wl;
  const ContextLayout& C = L.c[c];
  PullCtx* ctx = t->ctx(c);
  t->cx[c].buckets = t->cx[c].looked_up = t->cx[c].counted = false;
  if (n == 0) {
    set_ctx_empty<<<1, 64, 0, s>>>(ctx, t->w<u32>(C.seg_off));
  } else {
    // a1: order the occurrences by the top bits of their keys
    stage_mark(t, HPS_STAGE_SORT, s);
    ++t->serial;
    const u32 epoch = (u32)(t->serial % kEpochMod) + 1;
    if (epoch == 1 && t->serial >= kEpochMod)   // the epochs start over: forget the old words
      fill_u64<<<1024, 256, 0, s>>>(t->w<u64>(L.tile_rows), (L.evidence - L.tile_rows) / 8, 0);
    // (the other forms' word first: what it tells of came after whatever the range's word then does not tell of)
    FormChoice::Reports reports = {0, 0, 0};
    if (t->report) {
      reports.other = __atomic_load_n(t->report, __ATOMIC_ACQUIRE);
      reports.range = __atomic_load_n(t->report + 1, __ATOMIC_RELAXED);
      reports.small = __atomic_load_n(t->report + 2, __ATOMIC_RELAXED);
    }
    const int form = t->choice.next(n, d_offsets != nullptr, t->serial, t->lookup_serial, reports);
    t->cx[c].form = form;
    t->cx[c].buckets = form != kPlainForm;
    if (form == kSmallForm) {
      t->cx[c].looked_up = include != kDedupOnly;
      if (include == kWithPullLookup) ++t->pull_serial;
      const bool own_bags = d_offsets == nullptr;
      if (include == kDedupOnly) launch_small<false>(t, c, d_keys, n, own_bags, include, s);
      else launch_small<true>(t, c, d_keys, n, own_bags, include, s);
      stage_mark(t, HPS_STAGE_SORT, s);
      stage_mark(t, HPS_STAGE_UNIQUE, s);
      stage_mark(t, HPS_STAGE_UNIQUE, s);
      return;
    }
    if (form != kPlainForm) {
      t->cx[c].plan = bucket_plan(n);
      // the most recent list of frequent keys that is certainly complete (common.hpp)
      const HeavyRaw* heavy = &t->w<HeavyRing>(L.heavy_raw)->raw[(t->lookup_serial + kHeavyRing - 1) % kHeavyRing];
#define HPS_BUCKETS(K, FORM) launch_buckets<K, FORM>(t, c, d_keys, n, d_offsets, n_bags, heavy, s)
#define HPS_BUCKETS3(K)                                    \
  if (form == kByBorders) HPS_BUCKETS(K, kByBorders);      \
  else if (form == kByHash) HPS_BUCKETS(K, kByHash);       \
  else HPS_BUCKETS(K, kByRange)
#define HPS_BUCKETS2(K)                                    \
  if (form == kByHash) HPS_BUCKETS(K, kByHash);            \
  else HPS_BUCKETS(K, kByRange)
      switch (bucket_class(n)) {
        case 0: HPS_BUCKETS3(0); break;
        case 1: HPS_BUCKETS3(1); break;
        case 2: HPS_BUCKETS2(2); break;
        default: HPS_BUCKETS2(3); break;
      }
#undef HPS_BUCKETS2
#undef HPS_BUCKETS3
#undef HPS_BUCKETS
    } else {
      const SortPlan plan = sort_plan(n, t->choice.all_bits(t->serial));
      u64* kcur = t->w<u64>(L.keys_a);
      u64* kalt = t->w<u64>(L.keys_b);
      u64* pcur = t->w<u64>(L.idx_a);
      u64* palt = t->w<u64>(L.idx_b);
      u32* tickets = t->w<u32>(L.tickets);
      const unsigned n_tiles = (n + kSortTile - 1) / kSortTile;
      const unsigned bag_blocks = grid_for(d_offsets ? n_bags : n, kPrepThreads, 256);
      // two sets of digit histograms: a plain dedup counts into one and clears the other for
      // the next plain dedup
      ++t->plain_serial;
      u32* ghist = t->w<u32>(L.ghist) + (t->plain_serial & 1) * kHistWords;
      u32* ghist_next = t->w<u32>(L.ghist) + ((t->plain_serial + 1) & 1) * kHistWords;
      const unsigned hist_blocks = n_tiles < 768 ? n_tiles : 768;
      sort_prepare<<<hist_blocks + bag_blocks, kPrepThreads, 0, s>>>(
          d_keys, n, plan, ghist, ghist_next, tickets, ctx, d_offsets, n_bags, t->w<i32>(L.bag_of),
          hist_blocks, nullptr);
      for (int p = 0; p < plan.n_pass; ++p) {
        u32* tile_rows = t->w<u32>(L.tile_rows) + (size_t)p * L.sort_tiles * kRadix;
        u32* group_rows = t->w<u32>(L.group_rows) + (size_t)p * (L.sort_tiles / kMinTileGroup + 1) * kRadix;
        const int shift = p * kRadixBits;     // within the key's sorted prefix
        if (p == 0) {
          onesweep_pass<true><<<n_tiles, kSortThreads, 0, s>>>(
              d_keys, nullptr, t->w<i32>(L.bag_of), kcur, pcur, n, shift, ghist + p * kRadix, tile_rows,
              group_rows, plan.group, tickets + p, epoch, ctx, nullptr);
        } else {
          onesweep_pass<false><<<n_tiles, kSortThreads, 0, s>>>(
              kcur, pcur, t->w<i32>(L.bag_of), kalt, palt, n, shift, ghist + p * kRadix, tile_rows,
              group_rows, plan.group, tickets + p, epoch, ctx, nullptr);
          u64* tk = kcur; kcur = kalt; kalt = tk;
          tk = pcur; pcur = palt; palt = tk;
        }
      }
      stage_mark(t, HPS_STAGE_SORT, s);
      // a1: unique keys, ranks, grouping; the second unique_emit only acts after a repair
      stage_mark(t, HPS_STAGE_UNIQUE, s);
      const unsigned head_tiles = (n + kHeadTile - 1) / kHeadTile;
      const u32 head_group = tile_group(head_tiles);
      u32* evidence = t->w<u32>(L.evidence);
      unique_emit<false><<<head_tiles, kHeadThreads, 0, s>>>(
          kcur, pcur, n, t->w<u32>(L.head_rows), t->w<u32>(L.head_groups), head_group,
          tickets + kMaxPasses, epoch, n_bags, t->w<u64>(C.uniq),
          t->w<i32>(C.inverse), t->w<u32>(C.bags), t->w<u32>(C.seg_off), ctx, evidence, t->view.st);
      fix_mixed_runs<<<1, kFixThreads, 0, s>>>(kcur, pcur, kalt, palt, n, ctx, evidence);
      unique_emit<true><<<head_tiles, kHeadThreads, 0, s>>>(
          kcur, pcur, n, t->w<u32>(L.head_rows) + L.head_tiles,
          t->w<u32>(L.head_groups) + (L.head_tiles / kMinTileGroup + 1), head_group,
          tickets + kMaxPasses + 1, epoch, n_bags, t->w<u64>(C.uniq),
          t->w<i32>(C.inverse), t->w<u32>(C.bags), t->w<u32>(C.seg_off), ctx, evidence, t->view.st);
    }
    stage_mark(t, HPS_STAGE_UNIQUE, s);
  }
}

// What a lookup of context c hands on besides rows[]: the rows by position (bucket form, for the
// pooling; an accumulate has none).
static RowsByPosition rows_by_position_args(const hps_table* t, int c, bool pull) {
  const hps_table::Context& cx = t->cx[c];
  RowsByPosition out;
  out.upos = pull && cx.buckets && cx.form != kSmallForm ? t->w<u32>(t->wl.c[c].upos) : nullptr;
  out.by_pos = t->w<u32>(t->wl.by_pos);
  out.by_heavy = t->w<u32>(t->wl.by_heavy);
  return out;
}

// a2 for context c: rows of the distinct keys (kNoRow for a key the table does not hold and, unless
// `create`, does not get) and the push's work lists.
static void launch_lookup(hps_table* t, int c, uint64_t n_keys, bool create, hipStream_t s) {
  const ContextLayout& C = t->wl.c[c];
  if (t->cx[c].looked_up) return;
  const OftenLists often = start_lookup(t, c, n_keys);
  const Creation creation = creation_of(t, n_keys, create);
  const UniqueSpans spans = unique_spans(t, c, n_keys);
  const RowsByPosition out = rows_by_position_args(t, c, create);
  pull_lookup<<<span_blocks(spans) + 1, kProbeThreads, 0, s>>>(t->view, t->w<u64>(C.uniq), t->w<u32>(C.seg_off), spans,
                                                           t->w<u32>(C.rows), out, creation, often);
  if (creation.how == kCreateIfRoom)
    pull_missing<<<span_blocks(spans), kProbeThreads, 0, s>>>(t->view, t->w<u64>(C.uniq), spans, t->ctx(c), t->w<u32>(C.rows), out, creation.set);
}

static void fill_push_args(hps_table* t, int c, uint64_t n_keys, const float* d_rows, int kind, PushArgs& a) {
  const WorkspaceLayout& L = t->wl;
  a.spans = unique_spans(t, c, n_keys);
  a.seg_off = t->w<u32>(L.c[c].seg_off);
  a.bags = t->w<u32>(L.c[c].bags);
  a.rows = t->w<u32>(L.c[c].rows);
  a.grads = d_rows;
  a.inv_len = nullptr;
  a.ctx = t->ctx(c);
  a.med_list = t->w<u32>(L.med_list);
  a.med_span = t->w<uint2>(L.med_span);
  a.chunk_items = t->w<uint4>(L.chunk_items);
  a.arrived = t->w<u32>(L.arrived);
  a.partials = t->w<float>(L.partials);
  a.lr = t->opt.lr;
  a.eps = t->opt.eps;
  a.kind = kind;
}

// Whether the GPU's LDS atomics serve the lanes of one instruction in ascending lane order
// (sort.hpp: digit_rank), measured once per device: 0 not yet, 1 yes, 2 no.  uses the table's (not yet
// initialised) state block for the result; waits for the stream.  HPS_RANK=ballot / ordered overrides
// the measurement (comparison runs, tests).
static int g_lane_order[64];

static bool lane_order_holds(TableState* st, hipStream_t s) {
  static_assert(offsetof(TableState, pad) % 8 == 0 &&
                    offsetof(TableState, probe_bad) == offsetof(TableState, pad) + 4,
                "the two words are cleared as one");
  u32* word = &st->probe_bad;
  const char* force = std::getenv("HPS_RANK");
  if (force && std::strcmp(force, "ballot") == 0) return false;
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) { (void)hipGetLastError(); return false; }
  int state = __atomic_load_n(&g_lane_order[dev], __ATOMIC_ACQUIRE);
  if (state == 0) {
    u32 bad = 1;
    fill_u64<<<1, 64, 0, s>>>(reinterpret_cast<u64*>(&st->pad), 1, 0);
    probe_lane_order<<<256, kSortThreads, 0, s>>>(64, word);
    if (hipMemcpyAsync(&bad, word, sizeof(bad), hipMemcpyDeviceToHost, s) != hipSuccess ||
        hipStreamSynchronize(s) != hipSuccess) {
      (void)hipGetLastError();
      return false;
    }
    state = bad == 0 ? 1 : 2;
    __atomic_store_n(&g_lane_order[dev], state, __ATOMIC_RELEASE);
  }
  return state == 1;
}

#define HPS_DISPATCH_LPR(lpr, CALL)            \
  switch (lpr) {                               \
    case 1: CALL(1); break;                    \
    case 2: CALL(2); break;                    \
    case 4: CALL(4); break;                    \
    case 8: CALL(8); break;                    \
    case 16: CALL(16); break;                  \
    case 32: CALL(32); break;                  \
    default: CALL(64); break;                  \
  }

extern "C" {

const char* hps_strerror(hps_status s) {
  switch (s) {
    case HPS_OK: return "ok";
    case HPS_EINVAL: return "invalid argument";
    case HPS_EFULL: return "table full";
    case HPS_ERESERVED: return "reserved key 0xFFFFFFFFFFFFFFFF in input";
    case HPS_ESTATE: return "call not valid in this state";
    case HPS_EDEVICE: return "HIP call failed or no usable GPU";
    case HPS_ENOMEM: return "buffer too small";
  }
  return "unknown status";
}

size_t hps_table_bytes(uint64_t capacity_keys, uint32_t dim, const hps_optimizer* opt) {
  if (!valid_opt(opt) || !valid_shape(capacity_keys, dim)) return 0;
  const uint32_t acc_len = opt->kind == HPS_OPT_ADAGRAD_ELEMENTWISE ? dim : 1;
  return storage_layout(slots_for(capacity_keys), dim, acc_len, opt->row_format).total;
}

size_t hps_workspace_bytes(uint64_t max_keys, uint64_t max_bags, uint32_t dim) {
  if (max_keys >= (1ull << 30) || max_bags >= (1ull << 31) || dim < 4 || dim > 1024 || dim % 4)
    return 0;
  return workspace_layout(max_keys, max_bags, dim).end;
}

hps_status hps_create(hps_table** out, uint64_t capacity_keys, uint32_t dim,
                      const hps_optimizer* opt, void* d_storage, size_t storage_bytes,
                      void* d_workspace, size_t workspace_bytes, uint64_t max_keys,
                      uint64_t max_bags, void* stream) {
  if (!out) return HPS_EINVAL;
  *out = nullptr;
  if (!valid_opt(opt) || !valid_shape(capacity_keys, dim)) return HPS_EINVAL;
  if (!d_storage || !d_workspace) return HPS_EINVAL;
  if ((uintptr_t)d_storage % kAlign || (uintptr_t)d_workspace % kAlign) return HPS_EINVAL;
  if (max_keys >= (1ull << 30) || max_bags >= (1ull << 31)) return HPS_EINVAL;
  const uint32_t acc_len = opt->kind == HPS_OPT_ADAGRAD_ELEMENTWISE ? dim : 1;
  const uint64_t n_slots = slots_for(capacity_keys);
  const StorageLayout sl = storage_layout(n_slots, dim, acc_len, opt->row_format);
  const WorkspaceLayout wl = workspace_layout(max_keys, max_bags, dim);
  if (storage_bytes < sl.total || workspace_bytes < wl.end) return HPS_ENOMEM;
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess) { (void)hipGetLastError(); return HPS_EDEVICE; }

  hps_table* t = new (std::nothrow) hps_table();
  if (!t) return HPS_ENOMEM;
  t->capacity = capacity_keys;
  t->n_slots = n_slots;
  t->max_keys = max_keys;
  t->max_bags = max_bags;
  t->dim = dim;
  t->acc_len = acc_len;
  t->opt = *opt;
  char* base = static_cast<char*>(d_storage);
  t->view.keys = reinterpret_cast<u64*>(base + sl.keys);
  t->view.w = base + sl.w;
  t->view.acc = base + sl.acc;
  t->view.w_pitch = sl.w_pitch;
  t->view.acc_pitch = sl.acc_pitch;
  t->view.st = reinterpret_cast<TableState*>(base + sl.state);
  t->view.n_lines = n_slots / kSlotsPerLine;
  t->view.capacity = capacity_keys;
  t->view.dim = dim;
  t->view.acc_len = acc_len;
  t->view.init_acc = opt->init_acc;
  t->view.init_range = opt->init_range;
  t->view.init_seed = opt->init_seed;
  t->view.bf16 = opt->row_format == HPS_ROWS_BF16 ? 1u : 0u;
  t->ws = static_cast<char*>(d_workspace);
  t->wl = wl;
  t->lpr = lanes_per_row(dim);
  t->current = t->prepared = -1;
  t->last_n_keys = 0;
  t->scratch_free = nullptr;
  t->listing_set = false;
  t->many_streams = false;
  bool events_ok = hipEventCreateWithFlags(&t->listing, hipEventDisableTiming) == hipSuccess;
  for (int k = 0; k < 2; ++k) {
    t->cx[k].n_keys = t->cx[k].n_bags = 0;
    t->cx[k].d_offsets = nullptr;
    t->cx[k].buckets = t->cx[k].looked_up = false;
    t->cx[k].ready_set = t->cx[k].released_set = t->cx[k].listed = t->cx[k].counted = false;
    events_ok = events_ok &&
                hipEventCreateWithFlags(&t->cx[k].ready, hipEventDisableTiming) == hipSuccess &&
                hipEventCreateWithFlags(&t->cx[k].released, hipEventDisableTiming) == hipSuccess;
  }
  t->report = nullptr;
  if (!events_ok) { (void)hipGetLastError(); hps_destroy(t); return HPS_EDEVICE; }
  t->timing_mask = 0;
  for (int i = 0; i < HPS_N_STAGES; ++i) t->ev_used[i] = 0;
  t->serial = 0;
  t->plain_serial = 0;
  t->mean_pooling = false;
  t->lookup_serial = t->pull_serial = t->dumped = 0;
  t->choice = FormChoice();
  t->report = nullptr;
  if (hipHostMalloc(reinterpret_cast<void**>(&t->report), 64, hipHostMallocDefault) != hipSuccess) {
    (void)hipGetLastError();
    hps_destroy(t);
    return HPS_EDEVICE;
  }
  t->report[0] = t->report[1] = t->report[2] = 0;
  {
    // HPS_DEDUP=radix / bucket / borders / hashed / small pins the dedup to one of its forms (comparison runs, tests)
    const char* mode = std::getenv("HPS_DEDUP");
    t->choice.mode = !mode ? 0 : std::strcmp(mode, "radix") == 0 ? 1 : std::strcmp(mode, "bucket") == 0 ? 2
                    : std::strcmp(mode, "borders") == 0 ? 3 : std::strcmp(mode, "hashed") == 0 ? 4
                    : std::strcmp(mode, "small") == 0 ? 5 : 0;
  }

  t->lookup_new_cap = kNewLdsCap;
  if (const char* cap = std::getenv("HPS_LOOKUP_NEW_LIST")) {
    const unsigned n = (unsigned)std::strtoul(cap, nullptr, 10);
    t->lookup_new_cap = n < kNewLdsCap ? n : kNewLdsCap;
  }
  hipStream_t s = static_cast<hipStream_t>(stream);
  t->ordered_rank = lane_order_holds(t->view.st, s);
  fill_u64<<<4096, 256, 0, s>>>(t->view.keys, n_slots, kEmptyKey);
  // look-back status words, digit histograms and the lists of frequent keys start at zero
  fill_u64<<<1024, 256, 0, s>>>(t->w<u64>(wl.ghist), (wl.bag_of - wl.ghist) / 8, 0);
  fill_u64<<<1024, 256, 0, s>>>(t->w<u64>(wl.fresh), (wl.local_rank - wl.fresh) / 8, 0);      // (aligned to kAlign)
  reset_state<<<1, 64, 0, s>>>(t->view.st);
  fill_u64<<<1, 64, 0, s>>>(reinterpret_cast<u64*>(&t->view.st->dump_count), 1, 0);
  for (int k = 0; k < 2; ++k)
    set_ctx_empty<<<1, 64, 0, s>>>(t->ctx(k), t->w<u32>(wl.c[k].seg_off));
  if (!launch_ok()) { hps_destroy(t); return HPS_EDEVICE; }
  *out = t;
  return HPS_OK;
}

hps_status hps_destroy(hps_table* t) {
  if (!t) return HPS_EINVAL;
  for (int i = 0; i < HPS_N_STAGES; ++i)
    for (hipEvent_t e : t->ev_pool[i]) (void)hipEventDestroy(e);
  // (a table whose creation failed half way holds null handles)
  if (t->listing) (void)hipEventDestroy(t->listing);
  for (int k = 0; k < 2; ++k) {
    if (t->cx[k].ready) (void)hipEventDestroy(t->cx[k].ready);
    if (t->cx[k].released) (void)hipEventDestroy(t->cx[k].released);
  }
  if (t->report) (void)hipHostFree(t->report);     // waits for the device: no lookup still writes to it
  delete t;
  return HPS_OK;
}

hps_status hps_clear(hps_table* t, void* stream) {
  if (!t) return HPS_EINVAL;
  if (t->current >= 0 || t->prepared >= 0) return HPS_ESTATE;
  hipStream_t s = static_cast<hipStream_t>(stream);
  // rows and accumulators need no clearing: a slot's row is written when its key is
  // claimed, and the marks of updated rows live in the accumulators
  fill_u64<<<4096, 256, 0, s>>>(t->view.keys, t->n_slots, kEmptyKey);
  reset_state<<<1, 64, 0, s>>>(t->view.st);
  return launch_ok() ? HPS_OK : HPS_EDEVICE;
}

hps_status hps_insert(hps_table* t, const uint64_t* d_keys, uint64_t n, const float* d_weights,
                      const float* d_acc, void* stream) {
  if (!t || (n && !d_keys) || (d_acc && !d_weights)) return HPS_EINVAL;
  hipStream_t s = static_cast<hipStream_t>(stream);
  if (n) {
    const unsigned blocks = grid_for(n, kProbeGroups, kProbeMaxBlocks);
    const unsigned row_blocks = grid_for(n, kRowThreads, kRowMaxBlocks);
    check_keys<<<grid_for(n, kRowThreads * 4, 2048), kRowThreads, 0, s>>>(d_keys, n, t->view.st);
#define HPS_INSERT(BF16, VALUES) \
    insert_rows<BF16, VALUES><<<row_blocks, kRowThreads, 0, s>>>(t->view, d_keys, n, d_weights, d_acc)
    if (t->view.bf16) { if (d_weights) HPS_INSERT(true, true); else HPS_INSERT(true, false); }
    else { if (d_weights) HPS_INSERT(false, true); else HPS_INSERT(false, false); }
#undef HPS_INSERT
    insert_missing<<<blocks, kProbeThreads, 0, s>>>(t->view, d_keys, n, d_weights, d_acc);
  }
  commit_insert<<<1, 64, 0, s>>>(t->view.st);
  return launch_ok() ? HPS_OK : HPS_EDEVICE;
}

static bool mini_batch_ok(const hps_table* t, const uint64_t* d_keys, uint64_t n_keys,
                          const int32_t* d_offsets, uint32_t n_examples, uint32_t n_slots) {
  if (!t || !d_offsets || (n_keys && !d_keys)) return false;
  if (n_keys > t->max_keys || (uint64_t)n_examples * n_slots > t->max_bags) return false;
  if (n_keys && (uint64_t)n_examples * n_slots == 0) return false;      // keys, but no bag to hold them
  return (uintptr_t)d_keys % 8 == 0 && (uintptr_t)d_offsets % 4 == 0;
}

// Orders a dedup into context c after the hps_last_unique that read what the context held before.
static bool after_listing(hps_table* t, int c, hipStream_t s) {
  if (!wait_for(t, t->listing, t->cx[c].listed, s)) return false;
  t->cx[c].listed = false;
  return true;
}

// include: kDedupOnly, or kWithPullLookup where hps_pull_prepared follows on the same stream at once.
static hps_status prepare(hps_table* t, const uint64_t* d_keys, uint64_t n_keys,
                          const int32_t* d_offsets, uint32_t n_examples, uint32_t n_slots,
                          Include include, void* stream) {
  if (!mini_batch_ok(t, d_keys, n_keys, d_offsets, n_examples, n_slots)) return HPS_EINVAL;
  const uint64_t n_bags = (uint64_t)n_examples * n_slots;
  hipStream_t s = static_cast<hipStream_t>(stream);
  const int c = t->current == 0 ? 1 : 0;        // the context the outstanding pull does not use
  hps_table::Context& cx = t->cx[c];
  const u32 n = (u32)n_keys;
  // order after the push that last read this context, and after the previous dedup
  // (the sort scratch is shared); both may have run on other streams
  if (!enter(t, s, true)) return HPS_EDEVICE;
  if (!wait_for(t, cx.released, cx.released_set, s) || !wait_for_scratch(t, s)) return HPS_EDEVICE;
  if (!after_listing(t, c, s)) return HPS_EDEVICE;
  // (a lookup among it: what hps_pull_prepared orders it after)
  const hps_table::Context& other = t->cx[1 - c];
  if (include != kDedupOnly && !wait_for(t, other.released, other.released_set, s)) return HPS_EDEVICE;

  launch_dedup(t, c, d_keys, n, d_offsets, (u32)n_bags, include, s);
  if (!launch_ok()) return HPS_EDEVICE;
  if (!mark(t, cx.ready, &cx.ready_set, s)) return HPS_EDEVICE;
  t->scratch_free = cx.ready;
  cx.n_keys = n_keys;
  cx.n_bags = n_bags;
  cx.d_offsets = d_offsets;
  cx.mean = t->mean_pooling;
  t->prepared = c;
  return HPS_OK;
}

hps_status hps_prepare(hps_table* t, const uint64_t* d_keys, uint64_t n_keys,
                       const int32_t* d_offsets, uint32_t n_examples, uint32_t n_slots,
                       void* stream) {
  return prepare(t, d_keys, n_keys, d_offsets, n_examples, n_slots, kDedupOnly, stream);
}

hps_status hps_pull_prepared(hps_table* t, float* d_pooled, void* stream) {
  if (!t) return HPS_EINVAL;
  if (t->prepared < 0 || t->current >= 0) return HPS_ESTATE;
  const int c = t->prepared;
  const hps_table::Context& cx = t->cx[c];
  if (cx.n_bags && !d_pooled) return HPS_EINVAL;
  if ((uintptr_t)d_pooled % 16) return HPS_EINVAL;
  hipStream_t s = static_cast<hipStream_t>(stream);
  if (!enter(t, s, true) || !wait_for(t, cx.ready, cx.ready_set, s)) return HPS_EDEVICE;
  // the lookup rewrites the work lists that both contexts share and the pooling reads rows: order
  // them after the push of the mini-batch before, should that have run on another stream
  const hps_table::Context& other = t->cx[1 - c];
  if (!wait_for(t, other.released, other.released_set, s)) return HPS_EDEVICE;
  // a2: look up every unique key, create the missing ones
  if (cx.n_bags && !cx.looked_up) ++t->pull_serial;
  stage_mark(t, HPS_STAGE_LOOKUP, s);
  if (cx.n_keys) launch_lookup(t, c, cx.n_keys, true, s);
  if (!cx.n_bags) commit_insert<<<1, 64, 0, s>>>(t->view.st);   // else the pooling kernel does it
  stage_mark(t, HPS_STAGE_LOOKUP, s);
  // a3: gather rows and pool per bag
  if (cx.n_bags) {
    stage_mark(t, HPS_STAGE_POOL, s);
#define CALL(LPR) launch_pool<LPR>(t, c, d_pooled, s)
    HPS_DISPATCH_LPR(t->lpr, CALL)
#undef CALL
    stage_mark(t, HPS_STAGE_POOL, s);
  }
  if (!launch_ok()) return HPS_EDEVICE;
  t->current = c;
  t->prepared = -1;
  t->last_n_keys = cx.n_keys;
  return HPS_OK;
}

hps_status hps_pull(hps_table* t, const uint64_t* d_keys, uint64_t n_keys,
                    const int32_t* d_offsets, uint32_t n_examples, uint32_t n_slots,
                    float* d_pooled, void* stream) {
  if ((uint64_t)n_examples * n_slots && !d_pooled) return HPS_EINVAL;
  if ((uintptr_t)d_pooled % 16) return HPS_EINVAL;
  if (!mini_batch_ok(t, d_keys, n_keys, d_offsets, n_examples, n_slots)) return HPS_EINVAL;
  if (t->current >= 0) return HPS_ESTATE;
  const Include include = creates_at_once(t, n_keys) ? kWithPullLookup : kDedupOnly;
  const hps_status rc = prepare(t, d_keys, n_keys, d_offsets, n_examples, n_slots, include, stream);
  return rc != HPS_OK ? rc : hps_pull_prepared(t, d_pooled, stream);
}

hps_status hps_push(hps_table* t, const float* d_pooled_grads, void* stream) {
  if (!t) return HPS_EINVAL;
  if (t->current < 0) return HPS_ESTATE;
  const int c = t->current;
  hps_table::Context& cx = t->cx[c];
  if (cx.n_bags && cx.n_keys && !d_pooled_grads) return HPS_EINVAL;
  if ((uintptr_t)d_pooled_grads % 16) return HPS_EINVAL;
  hipStream_t s = static_cast<hipStream_t>(stream);
  if (!enter(t, s, false)) return HPS_EDEVICE;
  t->current = -1;
  if (cx.n_keys && cx.n_bags) {
    PushArgs a;
    fill_push_args(t, c, cx.n_keys, d_pooled_grads,
                   t->opt.kind == HPS_OPT_ADAGRAD_ELEMENTWISE ? kStepElementwise : kStepRowwise, a);
    if (cx.mean) a.inv_len = t->w<float>(t->wl.c[c].inv_len);
    stage_mark(t, HPS_STAGE_PUSH, s);
#define CALL(LPR) launch_push<LPR>(t, cx.n_keys, a, s)
    HPS_DISPATCH_LPR(t->lpr, CALL)
#undef CALL
    stage_mark(t, HPS_STAGE_PUSH, s);
    if (!launch_ok()) return HPS_EDEVICE;
  }
  return mark(t, cx.released, &cx.released_set, s) ? HPS_OK : HPS_EDEVICE;
}

hps_status hps_set_pooling(hps_table* t, int mean) {
  if (!t || (mean != 0 && mean != 1)) return HPS_EINVAL;
  if (t->current >= 0 || t->prepared >= 0) return HPS_ESTATE;
  t->mean_pooling = mean != 0;
  return HPS_OK;
}

// The kernels of an accumulate on context 0 of whatever workspace the table currently points to.
static hps_status accumulate_launches(hps_table* t, const uint64_t* d_keys, uint64_t n,
                                      const float* d_values, hipStream_t s) {
  const int c = 0;
  // every (key, value row) pair is a bag of its own: the dedup groups the pairs by key,
  // the push kernels sum each group's value rows and add the sum onto the row
  launch_dedup(t, c, d_keys, (u32)n, nullptr, (u32)n, kWithAddLookup, s);
  if (n) {
    launch_lookup(t, c, n, false, s);
    PushArgs a;                      // (its kernel also books the keys that were not found)
    fill_push_args(t, c, n, d_values, kStepAdd, a);
#define CALL(LPR) launch_push<LPR>(t, n, a, s)
    HPS_DISPATCH_LPR(t->lpr, CALL)
#undef CALL
  } else {
    commit_absent<<<1, 64, 0, s>>>(t->view.st);
  }
  return launch_ok() ? HPS_OK : HPS_EDEVICE;
}

hps_status hps_accumulate(hps_table* t, const uint64_t* d_keys, uint64_t n, const float* d_values,
                          void* stream) {
  if (!t || (n && (!d_keys || !d_values))) return HPS_EINVAL;
  if (n > t->max_keys || (uintptr_t)d_keys % 8 || (uintptr_t)d_values % 16) return HPS_EINVAL;
  if (t->current >= 0 || t->prepared >= 0) return HPS_ESTATE;
  hipStream_t s = static_cast<hipStream_t>(stream);
  hps_table::Context& cx = t->cx[0];
  if (!enter(t, s, true)) return HPS_EDEVICE;
  for (int k = 0; k < 2; ++k)      // after the last push of either context (shared work lists, table rows)
    if (!wait_for(t, t->cx[k].released, t->cx[k].released_set, s)) return HPS_EDEVICE;
  if (!wait_for_scratch(t, s)) return HPS_EDEVICE;
  if (!after_listing(t, 0, s)) return HPS_EDEVICE;
  const hps_status rc = accumulate_launches(t, d_keys, n, d_values, s);
  if (rc != HPS_OK) return rc;
  if (!mark(t, cx.released, &cx.released_set, s)) return HPS_EDEVICE;
  t->scratch_free = cx.released;
  return HPS_OK;
}

hps_status hps_accumulate_static(hps_table* t, const uint64_t* d_keys, uint64_t n,
                                 const float* d_values, void* stream) {
  if (!t || (n && (!d_keys || !d_values))) return HPS_EINVAL;
  if (n > HPS_STATIC_MAX_KEYS || (uintptr_t)d_keys % 8 || (uintptr_t)d_values % 16) return HPS_EINVAL;
  if (t->current >= 0 || t->prepared >= 0) return HPS_ESTATE;
  const WorkspaceLayout wl = workspace_layout(HPS_STATIC_MAX_KEYS, HPS_STATIC_MAX_KEYS, t->dim, false);
  if (wl.end > kStaticScratchBytes) return HPS_EINVAL;       // rows too wide for the static array
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) { (void)hipGetLastError(); return HPS_EDEVICE; }
  StaticScratch& ss = g_static[dev];
  hipStream_t s = static_cast<hipStream_t>(stream);
  if (!ss.ptr) {
    // this device's copy of the array: the name itself is no device address on the host
    void* p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) { (void)hipGetLastError(); return HPS_EDEVICE; }
    ss.ptr = static_cast<char*>(p);
    ss.ring_ready = false;
  }
  // The table works on the static array for the length of this call: its own workspace, and
  // what the host keeps about it, stay as they are.
  struct Saved {
    char* ws; WorkspaceLayout wl; uint64_t serial, plain_serial, lookup_serial;
    FormChoice choice; unsigned long long* report; uint32_t timing_mask;
  } keep = {t->ws, t->wl, t->serial, t->plain_serial, t->lookup_serial, t->choice, t->report, t->timing_mask};
  t->ws = ss.ptr;
  t->wl = wl;
  t->serial = t->plain_serial = 0;            // the status words are cleared below: any epoch will do
  t->lookup_serial = ss.lookup_serial;
  t->choice.mode = 1;                          // plain passes ...
  t->choice.full_until = ~0ull;                // ... over all 64 key bits: exact whatever the keys, no history needed
  t->report = nullptr;
  t->timing_mask = 0;
  // what must start at zero: digit histograms, tickets, status words; once per device: the lists of frequent keys
  fill_u64<<<256, 256, 0, s>>>(t->w<u64>(wl.ghist), (wl.heavy_raw - wl.ghist) / 8, 0);
  if (!ss.ring_ready) {
    fill_u64<<<64, 256, 0, s>>>(t->w<u64>(wl.heavy_raw), (wl.bag_of - wl.heavy_raw) / 8, 0);
    ss.ring_ready = true;
  }
  set_ctx_empty<<<1, 64, 0, s>>>(t->ctx(0), t->w<u32>(wl.c[0].seg_off));
  const hps_status rc = accumulate_launches(t, d_keys, n, d_values, s);
  ss.lookup_serial = t->lookup_serial;
  t->ws = keep.ws;
  t->wl = keep.wl;
  t->serial = keep.serial;
  t->plain_serial = keep.plain_serial;
  t->lookup_serial = keep.lookup_serial;
  t->choice = keep.choice;
  t->report = keep.report;
  t->timing_mask = keep.timing_mask;
  return rc;
}

// Buckets by hash: puts the distinct keys of context c in order (into d_uniq_out, if wanted) and notes every key's rank
// (local_rank), with the plain form's passes over all 64 bits, in the dedups' scratch.  The number of distinct keys is only
// known on the device.  The status words and histograms are clear before and after, so that neither this call's
// sequence of kernels, which a graph may replay, nor a plain dedup meets words of the other.
static void sort_uniques(hps_table* t, int c, u32 n, uint64_t* d_uniq_out, hipStream_t s) {
  const WorkspaceLayout& L = t->wl;
  const ContextLayout& C = L.c[c];
  const SortPlan plan = sort_plan(n, true);
  PullCtx* ctx = t->w<PullCtx>(L.sort_ctx);
  u32* n_dev = t->w<u32>(L.sort_n);
  u64* in = t->w<u64>(L.keys_b);
  u64* kout = t->w<u64>(L.keys_a);
  u64* pin = nullptr;
  u64* pout = t->w<u64>(L.idx_a);
  u32* tickets = t->w<u32>(L.tickets);
  u32* ghist = t->w<u32>(L.ghist);
  const u32 n_nat = t->cx[c].plan.n_nat;
  const unsigned n_tiles = (n + kSortTile - 1) / kSortTile, hist_blocks = n_tiles < 768 ? n_tiles : 768;
  constexpr u32 kEpoch = 1;
  fill_u64<<<1024, 256, 0, s>>>(t->w<u64>(L.ghist), (L.heavy_raw - L.ghist) / 8, 0);
  gather_uniques<<<n_nat + 1, kOrderThreads, 0, s>>>(t->w<u64>(C.uniq), t->w<u32>(C.bucket_start), t->w<u32>(C.count), n_nat,
                                                     t->ctx(c), in, t->w<u32>(L.bag_of), n_dev);
  sort_prepare<<<hist_blocks, kPrepThreads, 0, s>>>(in, n, plan, ghist, ghist + kHistWords, tickets, ctx, nullptr, 0, nullptr, hist_blocks, n_dev);
  for (int p = 0; p < plan.n_pass; ++p) {
    u32* tile_rows = t->w<u32>(L.tile_rows) + (size_t)p * L.sort_tiles * kRadix;
    u32* group_rows = t->w<u32>(L.group_rows) + (size_t)p * (L.sort_tiles / kMinTileGroup + 1) * kRadix;
    if (p == 0)
      onesweep_pass<true><<<n_tiles, kSortThreads, 0, s>>>(in, pin, t->w<i32>(L.bag_of), kout, pout, n, 0, ghist, tile_rows, group_rows,
                                                           plan.group, tickets, kEpoch, ctx, n_dev);
    else
      onesweep_pass<false><<<n_tiles, kSortThreads, 0, s>>>(in, pin, t->w<i32>(L.bag_of), kout, pout, n, p * kRadixBits, ghist + p * kRadix,
                                                            tile_rows, group_rows, plan.group, tickets + p, kEpoch, ctx, n_dev);
    u64* x = in; in = kout; kout = x;
    x = pin ? pin : t->w<u64>(L.idx_b); pin = pout; pout = x;
  }
  take_ranks<<<grid_for(n, kOrderThreads * 4, 1024), kOrderThreads, 0, s>>>(in, pin, n_dev, ctx, t->view.st, d_uniq_out, t->w<u32>(L.local_rank));
  fill_u64<<<1024, 256, 0, s>>>(t->w<u64>(L.ghist), (L.heavy_raw - L.ghist) / 8, 0);
}

// The kernels and copies of an hps_last_unique of context c.  They read what its dedup wrote and nothing
// else, and write scratch of their own (buckets by hash: and the dedups').
static hps_status list_unique(hps_table* t, int c, uint64_t* d_uniq_out, int32_t* d_inverse_out, hipStream_t s) {
  const WorkspaceLayout& L = t->wl;
  const ContextLayout& C = L.c[c];
  const hps_table::Context& cx = t->cx[c];
  const uint64_t n = cx.n_keys;
  if (cx.buckets) {
    u32* local_rank = t->w<u32>(L.local_rank);
    u32* bucket_total = t->w<u32>(L.bucket_total);
    u32* by_pos = d_inverse_out ? t->w<u32>(L.rank_by_pos) : nullptr;
    u32* by_heavy = d_inverse_out ? t->w<u32>(L.rank_by_heavy) : nullptr;
    const u32* start = t->w<u32>(C.bucket_start);
    const u32* count = t->w<u32>(C.count);
    const u64* border = cx.form == kByBorders ? t->w<u64>(C.border) : nullptr;
    if (cx.form == kSmallForm) {
      sort_uniques(t, c, (u32)n, d_uniq_out, s);
      if (d_inverse_out)
        small_ranks<<<grid_for(n, 256, 256), 256, 0, s>>>(t->w<uint4>(C.places), local_rank, (u32)n, reinterpret_cast<u32*>(d_inverse_out));
      return launch_ok() ? HPS_OK : HPS_EDEVICE;
    }
    if (cx.form == kByHash) {
      sort_uniques(t, c, (u32)n, d_uniq_out, s);
      if (d_inverse_out)
        emit_uniques<<<cx.plan.n_nat, kOrderThreads, 0, s>>>(t->w<u64>(C.uniq), start, count, t->w<u32>(C.upos), cx.plan.n_nat,
                                                             border, t->ctx(c), local_rank, nullptr, nullptr, by_pos, by_heavy);
    } else {
#define HPS_ORDER(GROUP) \
  order_uniques<GROUP><<<cx.plan.n_nat, order_threads(GROUP), 0, s>>>(t->w<u64>(C.uniq), start, count, cx.plan.n_nat, border, t->ctx(c), local_rank, bucket_total)
    if (group_threads(cx.form, n) == 256) HPS_ORDER(256);
    else HPS_ORDER(1024);
#undef HPS_ORDER
    emit_uniques<<<cx.plan.n_nat, kOrderThreads, 0, s>>>(t->w<u64>(C.uniq), start, count, t->w<u32>(C.upos), cx.plan.n_nat,
                                                         border, t->ctx(c), local_rank, bucket_total, d_uniq_out, by_pos, by_heavy);
    }
    if (d_inverse_out)
      launch_spread(t->w<u32>(C.code), t->w<uint16_t>(C.from), (u32)n, cx.plan.n_tiles, by_pos, by_heavy,
                    reinterpret_cast<u32*>(d_inverse_out), s);
    return launch_ok() ? HPS_OK : HPS_EDEVICE;
  }
  // U <= n is only known on the device: copy n entries, the caller reads the first U.
  if (d_uniq_out &&
      hipMemcpyAsync(d_uniq_out, t->w<u64>(C.uniq), n * 8, hipMemcpyDeviceToDevice, s) != hipSuccess)
    return HPS_EDEVICE;
  if (d_inverse_out &&
      hipMemcpyAsync(d_inverse_out, t->w<i32>(C.inverse), n * 4, hipMemcpyDeviceToDevice, s) != hipSuccess)
    return HPS_EDEVICE;
  return HPS_OK;
}

hps_status hps_last_unique(hps_table* t, uint64_t* d_uniq_out, int32_t* d_inverse_out,
                           void* stream) {
  if (!t) return HPS_EINVAL;
  if (t->current < 0) return HPS_ESTATE;
  hipStream_t s = static_cast<hipStream_t>(stream);
  const int c = t->current;
  hps_table::Context& cx = t->cx[c];
  if (cx.n_keys == 0 || (!d_uniq_out && !d_inverse_out)) return HPS_OK;
  if (!cx.counted) t->choice.listed();          // (listed again: that tells nothing new)
  cx.counted = true;
  // On any stream: after the dedup whose results it lists and after the call before it (the ranks'
  // scratch); the next dedup into this context waits for it (after_listing).  Events that were recorded outside a
  // capture cannot be waited for inside one: what is captured here, the caller orders.
  hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(s, &capture) != hipSuccess) (void)hipGetLastError();
  if (capture != hipStreamCaptureStatusNone) {
    t->choice.captured(cx.n_keys, cx.form);
    return list_unique(t, c, d_uniq_out, d_inverse_out, s);
  }
  if (!enter(t, s, true) || !wait_for(t, cx.ready, cx.ready_set, s) || !wait_for(t, t->listing, t->listing_set, s)) return HPS_EDEVICE;
  const bool sorts = cx.buckets && (cx.form == kByHash || cx.form == kSmallForm);       // in the scratch of the dedups
  if (sorts && !wait_for_scratch(t, s)) return HPS_EDEVICE;
  const hps_status rc = list_unique(t, c, d_uniq_out, d_inverse_out, s);
  if (!mark(t, t->listing, &t->listing_set, s)) return HPS_EDEVICE;
  if (sorts) t->scratch_free = t->listing;
  cx.listed = true;
  return rc;
}

static hps_status get_impl(hps_table* t, bool zero, const uint64_t* d_keys, uint64_t n, float* d_weights_out,
                           float* d_acc_out, uint8_t* d_found_out, void* stream) {
  if (!t || (n && (!d_keys || !d_weights_out || !d_acc_out || !d_found_out))) return HPS_EINVAL;
  if (n == 0) return HPS_OK;
  hipStream_t s = static_cast<hipStream_t>(stream);
  const unsigned blocks = grid_for(n, kRowThreads, kRowMaxBlocks);
#define HPS_GET(BF16, ZERO) \
  get_rows<BF16, ZERO><<<blocks, kRowThreads, 0, s>>>(t->view, d_keys, n, d_weights_out, d_acc_out, d_found_out)
  if (t->view.bf16) { if (zero) HPS_GET(true, true); else HPS_GET(true, false); }
  else { if (zero) HPS_GET(false, true); else HPS_GET(false, false); }
#undef HPS_GET
  return launch_ok() ? HPS_OK : HPS_EDEVICE;
}

hps_status hps_get(hps_table* t, const uint64_t* d_keys, uint64_t n, float* d_weights_out,
                   float* d_acc_out, uint8_t* d_found_out, void* stream) {
  return get_impl(t, false, d_keys, n, d_weights_out, d_acc_out, d_found_out, stream);
}

hps_status hps_get_or_zero(hps_table* t, const uint64_t* d_keys, uint64_t n, float* d_weights_out,
                           float* d_acc_out, uint8_t* d_found_out, void* stream) {
  return get_impl(t, true, d_keys, n, d_weights_out, d_acc_out, d_found_out, stream);
}

static hps_status dump_impl(hps_table* t, bool dirty, uint64_t* d_keys_out, float* d_weights_out,
                            float* d_acc_out, uint64_t max_rows, uint64_t* h_n_rows, void* stream) {
  if (!t || !h_n_rows) return HPS_EINVAL;
  if (max_rows && (!d_keys_out || !d_weights_out || !d_acc_out)) return HPS_EINVAL;
  hipStream_t s = static_cast<hipStream_t>(stream);
  if (t->dumped == ~0ull) {
    fill_u64<<<1, 64, 0, s>>>(reinterpret_cast<u64*>(&t->view.st->dump_count), 1, 0);
    t->dumped = 0;
  }
  const uint64_t counted = t->dumped;
  t->dumped = ~0ull;
#define HPS_DUMP(DIRTY, ROUNDS)                                                                                     \
  dump_rows<DIRTY, ROUNDS><<<grid_for(t->n_slots, kDumpSlots * ROUNDS, kDumpMaxBlocks), kRowThreads, 0, s>>>(        \
      t->view, d_keys_out, d_weights_out, d_acc_out, max_rows, &t->view.st->dump_count, counted)
  if (t->n_slots < kDumpSmall) { if (dirty) HPS_DUMP(true, 1); else HPS_DUMP(false, 1); }
  else { if (dirty) HPS_DUMP(true, kDumpRounds); else HPS_DUMP(false, kDumpRounds); }
#undef HPS_DUMP
  if (!launch_ok()) return HPS_EDEVICE;
  unsigned long long count = 0;
  if (hipMemcpyAsync(&count, &t->view.st->dump_count, sizeof(count), hipMemcpyDeviceToHost, s) != hipSuccess)
    return HPS_EDEVICE;
  if (hipStreamSynchronize(s) != hipSuccess) return HPS_EDEVICE;
  t->dumped = count;
  count -= counted;
  *h_n_rows = count;
  return count > max_rows ? HPS_ENOMEM : HPS_OK;
}

hps_status hps_dump(hps_table* t, uint64_t* d_keys_out, float* d_weights_out, float* d_acc_out,
                    uint64_t max_rows, uint64_t* h_n_rows, void* stream) {
  return dump_impl(t, false, d_keys_out, d_weights_out, d_acc_out, max_rows, h_n_rows, stream);
}

hps_status hps_dump_dirty(hps_table* t, uint64_t* d_keys_out, float* d_weights_out,
                          float* d_acc_out, uint64_t max_rows, uint64_t* h_n_rows, void* stream) {
  if (t && t->current >= 0) return HPS_ESTATE;
  return dump_impl(t, true, d_keys_out, d_weights_out, d_acc_out, max_rows, h_n_rows, stream);
}

hps_status hps_stats(hps_table* t, hps_stats_t* h_out, void* stream) {
  if (!t || !h_out) return HPS_EINVAL;
  hipStream_t s = static_cast<hipStream_t>(stream);
  TableState st;
  PullCtx ctx;
  if (hipMemcpyAsync(&st, t->view.st, sizeof(st), hipMemcpyDeviceToHost, s) != hipSuccess)
    return HPS_EDEVICE;
  const int which = t->current >= 0 ? t->current : (t->prepared >= 0 ? t->prepared : 0);
  if (hipMemcpyAsync(&ctx, t->ctx(which), sizeof(ctx), hipMemcpyDeviceToHost, s) != hipSuccess)
    return HPS_EDEVICE;
  if (hipStreamSynchronize(s) != hipSuccess) return HPS_EDEVICE;
  h_out->size = st.size;
  h_out->capacity = t->capacity;
  h_out->n_slots = t->n_slots;
  h_out->last_n_keys = t->last_n_keys;
  h_out->last_n_unique = ctx.n_unique;
  if (ctx.by_id) {
    h_out->last_n_unique = 0;
    for (int k = 0; k < kCountShards; ++k) h_out->last_n_unique += ctx.uniq_shard[k];
  }
  h_out->last_n_inserted = st.inserted;
  h_out->last_n_absent = (uint64_t)st.absent;
  h_out->n_plain_fallbacks = t->choice.n_fallbacks;
  h_out->n_full_fallbacks = t->choice.n_full_fallbacks;
  h_out->load_factor = (double)st.size / (double)t->n_slots;
  h_out->error = st.error;
  h_out->pull_outstanding = t->current >= 0 ? 1 : 0;
  return HPS_OK;
}

hps_status hps_probe_lengths(hps_table* t, double* h_mean, uint64_t* h_max, void* stream) {
  if (!t || !h_mean || !h_max) return HPS_EINVAL;
  hipStream_t s = static_cast<hipStream_t>(stream);
  clear_probe_lengths<<<1, 1, 0, s>>>(t->view.st);
  probe_length_scan<<<4096, 256, 0, s>>>(t->view);
  if (!launch_ok()) return HPS_EDEVICE;
  TableState st;
  if (hipMemcpyAsync(&st, t->view.st, sizeof(st), hipMemcpyDeviceToHost, s) != hipSuccess ||
      hipStreamSynchronize(s) != hipSuccess)
    return HPS_EDEVICE;
  *h_mean = st.size ? (double)st.probe_sum / (double)st.size : 0.0;
  *h_max = st.probe_max;
  return HPS_OK;
}

hps_status hps_set_stage_timing(hps_table* t, uint32_t stage_mask) {
  if (!t || stage_mask >= (1u << HPS_N_STAGES)) return HPS_EINVAL;
  t->timing_mask = stage_mask;
  for (int i = 0; i < HPS_N_STAGES; ++i) t->ev_used[i] = 0;
  return HPS_OK;
}

hps_status hps_stage_times(hps_table* t, double* h_ms_sum, uint32_t* h_count) {
  if (!t || !h_ms_sum || !h_count) return HPS_EINVAL;
  hps_status rc = HPS_OK;
  for (int st = 0; st < HPS_N_STAGES; ++st) {
    h_ms_sum[st] = 0.0;
    h_count[st] = 0;
    const size_t pairs = t->ev_used[st] / 2;
    for (size_t p = 0; p < pairs; ++p) {
      float ms = 0.f;
      if (hipEventSynchronize(t->ev_pool[st][2 * p + 1]) != hipSuccess ||
          hipEventElapsedTime(&ms, t->ev_pool[st][2 * p], t->ev_pool[st][2 * p + 1]) != hipSuccess) {
        (void)hipGetLastError();
        rc = HPS_EDEVICE;
        continue;
      }
      h_ms_sum[st] += ms;
      h_count[st] += 1;
    }
    t->ev_used[st] = 0;
  }
  return rc;
}

hps_status hps_probe_random_rows(const void* d_rows, uint64_t n_rows, uint32_t row_bytes,
                                 uint64_t n_accesses, float* d_sink, void* stream) {
  if (!d_rows || !d_sink || n_rows == 0 || (uintptr_t)d_rows % 16) return HPS_EINVAL;
  if (row_bytes != 64 && row_bytes != 256) return HPS_EINVAL;
  const unsigned blocks = kPoolMaxBlocks;
  const uint64_t groups = (uint64_t)blocks * (kPoolThreads / (row_bytes / 16));
  uint64_t per_group = (n_accesses + groups - 1) / groups;
  per_group = (per_group + kPoolInFlight - 1) / kPoolInFlight * kPoolInFlight;
  if (per_group == 0 || per_group > 0xFFFFFFF0ull) return HPS_EINVAL;
  hipStream_t s = static_cast<hipStream_t>(stream);
  if (row_bytes == 64)
    random_row_probe<4><<<blocks, kPoolThreads, 0, s>>>(static_cast<const float4*>(d_rows), n_rows,
                                                        (u32)per_group, d_sink);
  else
    random_row_probe<16><<<blocks, kPoolThreads, 0, s>>>(static_cast<const float4*>(d_rows), n_rows,
                                                         (u32)per_group, d_sink);
  return launch_ok() ? HPS_OK : HPS_EDEVICE;
}

hps_status hps_clear_error(hps_table* t, void* stream) {
  if (!t) return HPS_EINVAL;
  clear_error<<<1, 64, 0, static_cast<hipStream_t>(stream)>>>(t->view.st);
  // While the status was set the kernels of a pull did nothing: what its context holds
  // (row numbers above all) may be an earlier mini-batch's, and a push must not use it.
  t->current = t->prepared = -1;
  return launch_ok() ? HPS_OK : HPS_EDEVICE;
}

// ---- the host-memory cache behind the table (include/hps_mem.h) --------------------------
struct hps_mem {
  hps::MemTier tier;
  hps_mem(uint32_t dim, uint32_t acc_len, uint64_t lru, uint64_t lfu) : tier(dim, acc_len, lru, lfu) {}
};

hps_status hps_mem_create(hps_mem** out, uint32_t dim, uint32_t acc_len, uint64_t lru_capacity,
                          uint64_t lfu_capacity) {
  if (!out) return HPS_EINVAL;
  *out = nullptr;
  if (dim == 0 || dim > 1024 || (acc_len != 1 && acc_len != dim)) return HPS_EINVAL;
  hps_mem* m = new (std::nothrow) hps_mem(dim, acc_len, lru_capacity, lfu_capacity);
  if (!m) return HPS_ENOMEM;
  *out = m;
  return HPS_OK;
}

hps_status hps_mem_fetch(hps_mem* m, const uint64_t* h_keys, uint64_t n, uint64_t batch, float* h_w,
                         float* h_acc, uint8_t* h_found) {
  if (!m || (n && (!h_keys || !h_w || !h_acc || !h_found))) return HPS_EINVAL;
  try { m->tier.fetch(h_keys, n, batch, h_w, h_acc, h_found); } catch (const std::bad_alloc&) { return HPS_ENOMEM; }
  return HPS_OK;
}

hps_status hps_mem_store(hps_mem* m, const uint64_t* h_keys, uint64_t n, const float* h_w,
                         const float* h_acc, uint64_t batch, int visit) {
  if (!m || (n && (!h_keys || !h_w || !h_acc)) || (visit != 0 && visit != 1)) return HPS_EINVAL;
  try { m->tier.store(h_keys, n, h_w, h_acc, batch, visit != 0); } catch (const std::bad_alloc&) { return HPS_ENOMEM; }
  return HPS_OK;
}

hps_status hps_mem_complete_batch(hps_mem* m, uint64_t batch) {
  if (!m) return HPS_EINVAL;
  try { m->tier.complete_batch(batch); } catch (const std::bad_alloc&) { return HPS_ENOMEM; }
  return HPS_OK;
}

hps_status hps_mem_take_evicted(hps_mem* m, uint64_t* h_keys, float* h_w, float* h_acc,
                                uint64_t max_rows, uint64_t* h_n) {
  if (!m || !h_n || (max_rows && (!h_keys || !h_w || !h_acc))) return HPS_EINVAL;
  *h_n = m->tier.take_evicted(h_keys, h_w, h_acc, max_rows);
  return m->tier.evicted_waiting() ? HPS_ENOMEM : HPS_OK;
}

hps_status hps_mem_list(hps_mem* m, int which, uint64_t* h_keys, uint64_t max, uint64_t* h_n) {
  if (!m || !h_n || (which != 0 && which != 1) || (max && !h_keys)) return HPS_EINVAL;
  *h_n = m->tier.list(which, h_keys, max);
  return HPS_OK;
}

hps_status hps_mem_stats(hps_mem* m, hps_mem_stats_t* h_out) {
  if (!m || !h_out) return HPS_EINVAL;
  h_out->lru_size = m->tier.lru_size();
  h_out->lfu_size = m->tier.lfu_size();
  h_out->pinned = m->tier.pinned();
  h_out->evicted_waiting = m->tier.evicted_waiting();
  h_out->hits = m->tier.hits();
  h_out->misses = m->tier.misses();
  return HPS_OK;
}

hps_status hps_mem_destroy(hps_mem* m) {
  if (!m) return HPS_EINVAL;
  delete m;
  return HPS_OK;
}

}  // extern "C"
