// The HBM hash table: open addressing over 64-byte lines of 8 slots, linear
// probing line by line from an even line on, lock-free insertion by 64-bit compare-and-swap on the
// slot's key.  Lookups take four lanes per key, which look at two lines (a 128-byte bucket) at once; the kernels
// that create keys after a lookup (pull_missing, insert_missing) eight, one slot of a line each.
//
// Layout (structure of arrays, row index = slot index; TableView has the variants):
//   keys[n_slots]            u64, kEmptyKey when free
//   w[n_slots][dim]          f32 or bf16
//   acc[n_slots][acc_len]    f32
//
// A pull's lookup creates missing keys as it finds them.  Whether all of them fitted is known when it is over: the
// pooling kernel behind it adds up what was created and, if the table ended above its capacity, takes all of it out
// again (end_pull).  That takes slots for them in the meantime: capacity is 0.7 of the slots, so a mini-batch of up to a
// quarter of it leaves one slot in eight free.  For larger ones, and in a bulk insert, keys are created on the spot only if the
// table has room even if every one were new.  Otherwise creating them is a second kernel: the lookup counts
// the missing keys into sharded counters, pull_missing or insert_missing (every block reads the same total)
// claims slots only if all of them fit.  commit_insert adds an insert's count of created rows to the table size.
// rows.hpp: the entry points that move rows by key or by slot (insert, get, dump).
#pragma once

#include "common.hpp"
#include "form.hpp"

namespace hps {

struct TableView {
  u64* keys;
  // Row r's weights start w_pitch * r bytes after w, its accumulator(s) acc_pitch * r bytes
  // after acc.  Two layouts: weights and accumulators in arrays of their own, or (float32
  // rows with one accumulator per element, where a row's 8 * dim bytes divide the 128-byte
  // memory line or are a multiple of it) side by side, acc = w + 4 * dim and both pitches
  // 8 * dim: the push then finds a row's accumulators in the line(s) it fetched for the
  // weights, and the pooling fetches a full line per 64-byte row either way.
  char* w;
  char* acc;
  u32 w_pitch;
  u32 acc_pitch;
  TableState* st;
  u64 n_lines;      // n_slots / 8
  u64 capacity;
  u32 dim;
  u32 acc_len;
  float init_acc;
  float init_range;
  u64 init_seed;
  u32 bf16;         // 1: w holds bfloat16 values (2 bytes each) instead of float32
};

// ---- weights as stored --------------------------------------------------------------
// Rows hold float32 or bfloat16 values (the upper half of a float32; stored with
// round-to-nearest, ties to even); all arithmetic is float32 either way.
__device__ __forceinline__ float bf16_value(u32 h) { return __uint_as_float(h << 16); }
__device__ __forceinline__ u32 bf16_nearest(float f) {
  const u32 u = __float_as_uint(f);
  if ((u & 0x7FFFFFFFu) > 0x7F800000u) return (u >> 16) | 0x40u;     // NaN stays NaN
  return (u + 0x7FFFu + ((u >> 16) & 1u)) >> 16;
}
__device__ __forceinline__ char* w_row(const TableView& t, u64 row) { return t.w + row * t.w_pitch; }
// The accumulator(s) of row `row`.
__device__ __forceinline__ float* acc_row(const TableView& t, u64 row) {
  return reinterpret_cast<float*>(t.acc + row * t.acc_pitch);
}
// Element j of row `row`.
__device__ __forceinline__ void store_w(const TableView& t, u64 row, u32 j, float v) {
  if (t.bf16) reinterpret_cast<unsigned short*>(w_row(t, row))[j] = (unsigned short)bf16_nearest(v);
  else reinterpret_cast<float*>(w_row(t, row))[j] = v;
}
// Elements 4*col4 .. 4*col4+3 of row `row` (dim is a multiple of 4: one 16- or 8-byte access).
// Loops that keep several loads in flight take the format as a template argument and
// separate the load from the conversion (a test of t.bf16, or a conversion, between the
// loads makes the compiler wait for each load before it issues the next).
template <bool BF16> struct StoredW4;
template <> struct StoredW4<false> {
  float4 raw = make_float4(0.f, 0.f, 0.f, 0.f);
  __device__ __forceinline__ float4 value() const { return raw; }
};
template <> struct StoredW4<true> {
  uint2 raw = make_uint2(0u, 0u);
  __device__ __forceinline__ float4 value() const {
    return make_float4(bf16_value(raw.x & 0xFFFFu), bf16_value(raw.x >> 16), bf16_value(raw.y & 0xFFFFu),
                       bf16_value(raw.y >> 16));
  }
};
template <bool BF16>
__device__ __forceinline__ StoredW4<BF16> load_stored_w4(const TableView& t, u64 row, u32 col4) {
  StoredW4<BF16> s;
  s.raw = reinterpret_cast<const decltype(s.raw)*>(w_row(t, row))[col4];
  return s;
}
template <bool BF16>
__device__ __forceinline__ float4 load_w4_as(const TableView& t, u64 row, u32 col4) {
  return load_stored_w4<BF16>(t, row, col4).value();
}
__device__ __forceinline__ float4 load_w4(const TableView& t, u64 row, u32 col4) {
  return t.bf16 ? load_w4_as<true>(t, row, col4) : load_w4_as<false>(t, row, col4);
}
template <bool BF16>
__device__ __forceinline__ void store_w4_as(const TableView& t, u64 row, u32 col4, float4 v) {
  if (BF16)
    reinterpret_cast<uint2*>(w_row(t, row))[col4] = make_uint2(bf16_nearest(v.x) | (bf16_nearest(v.y) << 16),
                                                   bf16_nearest(v.z) | (bf16_nearest(v.w) << 16));
  else
    reinterpret_cast<float4*>(w_row(t, row))[col4] = v;
}
__device__ __forceinline__ void store_w4(const TableView& t, u64 row, u32 col4, float4 v) {
  if (t.bf16) store_w4_as<true>(t, row, col4, v);
  else store_w4_as<false>(t, row, col4, v);
}
// Elements 4*col4 .. 4*col4+3 of the initial row of the key whose mixed seed is `base`.
__device__ __forceinline__ float4 init_weight4(u64 base, u32 col4, float range) {
  return make_float4(init_weight(base, 4 * col4, range), init_weight(base, 4 * col4 + 1, range),
                     init_weight(base, 4 * col4 + 2, range), init_weight(base, 4 * col4 + 3, range));
}

constexpr int kProbeThreads = 256;
constexpr int kProbeGroups = kProbeThreads / kSlotsPerLine;   // insert: 8-lane groups per block
// Lookups take four lanes per key, each reading two of the line's eight slots with one
// 16-byte load: a wave's load instruction then asks for sixteen lines instead of eight, and
// the rate at which lines come back follows the lines asked for per instruction.
constexpr int kLookupLanes = 4;
// Keys a group of the pull's lookup has in flight, a multiple of the lanes of a group (two, four
// and eight were measured: two and four run alike, eight needs too many registers: 158, three
// waves per SIMD, a third slower; forcing five or six waves per SIMD by spilling gains nothing).
constexpr int kPullInFlight = 4;
static_assert(kPullInFlight % kLookupLanes == 0, "every lane of a group owns the same number of keys");
constexpr int kProbeMaxBlocks = 1024;
constexpr u32 kNewLdsCap = 1024;         // created keys a block of the lookup lists for its common initialisation
constexpr u32 kLongLdsCap = 64;          // very frequent keys whose chunk items whole waves write (>= kHeavyGroup)
constexpr u32 kRowsLdsCap = 2048;        // distinct keys whose rows it keeps to hand them on by position
constexpr u32 kShortSeg = 16;            // occurrences handled serially by one lane group

// How the push shares out the occurrences of a key with more than kShortSeg, by lanes per row: up to
// `medium` go to one wave, the others in pieces of `chunk` to one block each.  Wide rows leave fewer
// lane groups (64 / lpr a wave, 256 / lpr a block), each with eight rows in flight, so that
// the same piece takes more round trips to memory one after the other: 512 occurrences at 32 lanes
// a row are 32 trips of one wave.  Where the mini-batch is small the whole push waits for them (40 K
// occurrences, dim 100: 80 us; 28 with these sizes and kPushMaxParts together), so there a piece is
// about four trips.  In large ones they lie under other work, while more pieces cost more entries in the
// lists and more partial sums (8.4 M occurrences, dim 64: lookup 49 -> 71, push 320 -> 384 us).
struct PieceSizes { u32 medium, chunk; };
constexpr u64 kSmallPush = 1u << 19;
__host__ constexpr PieceSizes piece_sizes(u32 lpr, u64 n) {
  return lpr <= 4 || n > kSmallPush ? PieceSizes{512, 1024} : lpr == 8 ? PieceSizes{256, 1024} : lpr == 16 ? PieceSizes{128, 512}
         : lpr == 32 ? PieceSizes{64, 256} : PieceSizes{64, 128};
}

// Where the distinct keys of a mini-batch lie in uniq / seg_off / rows.  Bucket form (bucket.hpp): natural
// bucket c's in [bucket_start[c], + count[c]), heavy key h at bucket_start[n_spans + h] if that
// bucket is not empty.  Plain form (bucket_start == null): all in [0, ctx->n_unique), taken in
// spans of plain_span.  A block of the kernels that go through the distinct keys takes up to kHeavyGroup
// heavy keys (the first blocks: theirs is the longest work) or one span.
struct UniqueSpans {
  const u32* bucket_start;
  const u32* count;
  u32 n_spans;
  u32 max_heavy;         // bucket form: heavy buckets there may be
  u32 plain_span;        // plain form
};
constexpr u32 kHeavyGroup = 64;
__host__ __device__ __forceinline__ u32 heavy_blocks(const UniqueSpans& s) { return (s.max_heavy + kHeavyGroup - 1) / kHeavyGroup; }
__host__ __device__ __forceinline__ u32 span_blocks(const UniqueSpans& s) { return heavy_blocks(s) + s.n_spans; }
__device__ __forceinline__ void unique_span(const UniqueSpans& s, const PullCtx* ctx, u32 c, u32* first, u32* count) {
  if (s.bucket_start) {
    *first = s.bucket_start[c];
    *count = s.count[c] & 0x7FFFFFFFu;
  } else {
    const u32 u = ctx->n_unique;
    *first = c * s.plain_span;
    *count = u > *first ? min(s.plain_span, u - *first) : 0u;
  }
}

// What the lookup leaves for the push about keys that occur often (push.hpp): keys with
// kShortSeg < occurrences <= pieces.medium are listed, keys with more are cut into
// chunks of pieces.chunk positions.  Every block has its part of the list, with room for as many such keys as its
// occurrences could be (their count goes to med_span, beside where the part starts): with one counter for all, two thousand blocks
// queued up at it for 8 ns each.
struct OftenLists {
  PullCtx* ctx;
  u32* med_list;
  uint2* med_span;      // per block of a span or group of heavy keys: first entry, entries
  uint4* chunk_items;   // (unique index, chunk number, number of the chunked key, its first chunk item)
  u32* arrived;         // per chunked key: chunks the push has summed (cleared here)
  PieceSizes pieces;
  HeavyRaw* heavy_raw;  // keys with at least heavy_min occurrences are listed for the next dedup
  u32 heavy_min;
  HeavyRaw* heavy_next; // the list the next lookup will fill: emptied
  // Host memory (or null) that receives serial | flags << 32 about the dedup before this
  // lookup, in its second word if that went by key range, else in its first: kReportStandIn = it went by borders or by hash, kReportSlow = and more than 1/8 of
  // the occurrences lay in buckets that had to be ordered through global memory,
  // kReportOneKey = most of them in buckets that one key fills at least half of (keys
  // that turned frequent without warning, which the next hint will list; otherwise the
  // keys do not suit the buckets); kReportUneven = a bucket by range holds far more distinct keys than the mean,
  // kReportCrowded = so many that it costs several times the others' time (report_dedup); kReportMixed = it took the plain form and more places
  // than fix_mixed_runs can note had different keys agreeing in all sorted bits (keys in
  // clusters far apart), so that one workgroup had to put the whole array in order.  The host looks at it when it chooses the form of a later dedup, without
  // waiting for it.
  unsigned long long* report;
  u32 serial;
};

// "Updated since the last dirty dump" is kept in the sign bit of a row's first
// accumulator element: accumulators are sums of squares, never negative, so the bit
// is free, and the push rewrites that element anyway -- marking costs no traffic.
// Every reader takes the absolute value.
__device__ __forceinline__ float acc_value(float stored) { return fabsf(stored); }
__device__ __forceinline__ float acc_marked(float value) {
  return __uint_as_float(__float_as_uint(value) | 0x80000000u);
}
__device__ __forceinline__ bool acc_is_marked(float stored) {
  return (__float_as_uint(stored) & 0x80000000u) != 0;
}

// Bits of a wave-wide ballot that belong to this lane's 8-lane group.
__device__ __forceinline__ u32 group_bits(u64 ballot) {
  return (u32)(ballot >> (lane_id() & ~7u)) & 0xFFu;
}

__device__ __forceinline__ u64 load_slot_key(const u64* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Fill kernels (no memset nodes: safe to capture in a graph).
__global__ void __launch_bounds__(256) fill_u64(u64* __restrict__ p, u64 n, u64 v) {
  for (u64 i = (u64)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (u64)gridDim.x * blockDim.x)
    p[i] = v;
}
__device__ __forceinline__ void clear_counts(TableState* st) {
  if (threadIdx.x < kCountShards)
    st->miss_shard[threadIdx.x] = st->made_shard[threadIdx.x] = st->pull_made[0][threadIdx.x] = st->pull_made[1][threadIdx.x] = 0;
}
// (not dump_count: the host counts on from it, and a captured hps_clear runs when the host does not see it)
__global__ void __launch_bounds__(64) reset_state(TableState* st) {
  if (threadIdx.x == 0) {
    st->size = 0;
    st->inserted = 0;
    st->error = 0;
    st->absent = 0;
    st->size_before = 0;
    st->tight = 0;
  }
  clear_counts(st);
}
__global__ void __launch_bounds__(64) clear_error(TableState* st) {
  if (threadIdx.x == 0) st->error = 0;
  clear_counts(st);
}
__global__ void __launch_bounds__(64) set_ctx_empty(PullCtx* ctx, u32* seg_off) {
  if (threadIdx.x == 0) {
    ctx->n_unique = 0;
    ctx->n_long = 0;
    ctx->n_chunk_items = 0;
    ctx->n_evidence = 0;
    ctx->sort_error = 0;
    ctx->n_slow = 0;
    ctx->n_slow_one_key = 0;
    ctx->n_heavy = 0;
    ctx->n_total = 0;
    ctx->by_id = 0;
    seg_off[0] = 0;
  }
  if (threadIdx.x < kCountShards) ctx->uniq_shard[threadIdx.x] = 0;
}

// After an insert's kernels: adds the rows that were created to the table size and clears the counters.
__global__ void __launch_bounds__(64) commit_insert(TableState* st) {
  const u32 lane = lane_id();
  u32 made = lane < kCountShards ? st->made_shard[lane] : 0;
#pragma unroll
  for (int d = 1; d < kWave; d <<= 1) made += __shfl_xor(made, d, kWave);
  if (lane < kCountShards) st->miss_shard[lane] = st->made_shard[lane] = 0;
  if (lane == 0) {
    st->size += made;
    st->inserted = made;
  }
}

// After a lookup that creates nothing (accumulate): the number of keys not found
// goes to st->absent, the counters are cleared.  One wave; of the push, or where there is nothing to push a kernel.
__device__ __forceinline__ void commit_absent_wave(TableState* st) {
  const u32 lane = lane_id();
  u32 missing = lane < kCountShards ? st->miss_shard[lane] : 0;
#pragma unroll
  for (int d = 1; d < kWave; d <<= 1) missing += __shfl_xor(missing, d, kWave);
  if (lane < kCountShards) st->miss_shard[lane] = 0;
  if (lane == 0) st->absent = (int)missing;
}
__global__ void __launch_bounds__(64) commit_absent(TableState* st) { commit_absent_wave(st); }

// Where a key's probe sequence starts: an even line (n_lines is even), so that a 128-byte
// memory line holds the first two lines of the sequence.
__device__ __forceinline__ u64 home_line(const TableView& t, u64 key) {
  return 2 * __umul64hi(slot_hash(key), t.n_lines >> 1);
}

// The same for a group of kLookupLanes lanes: lane `sub` holds slots 2 * sub and 2 * sub + 1 of
// the line in `pair`.
__device__ __forceinline__ u32 group4_bits(u64 ballot) {
  return (u32)(ballot >> (lane_id() & ~3u)) & 0xFu;
}
__device__ __forceinline__ ulonglong2 load_slot_pair(const TableView& t, u64 line, u32 sub) {
  return reinterpret_cast<const ulonglong2*>(t.keys)[line * (kSlotsPerLine / 2) + sub];
}

// Finds the key or claims a free slot for it.  *created tells which.
__device__ __forceinline__ u32 probe_find_or_claim(const TableView& t, u64 key, u32 sub, u64 line,
                                                   u64 slot_key, bool* created) {
  *created = false;
  for (u64 step = 0; step < 2 * t.n_lines; ++step) {
    const u32 hit = group_bits(__ballot(slot_key == key));
    if (hit) return (u32)(line * kSlotsPerLine + (__ffs(hit) - 1));
    const u32 free_slots = group_bits(__ballot(slot_key == kEmptyKey));
    if (free_slots) {
      const u32 target = __ffs(free_slots) - 1;
      u64 seen = 0;
      if (sub == target)
        seen = atomicCAS((unsigned long long*)&t.keys[line * kSlotsPerLine + target],
                         (unsigned long long)kEmptyKey, (unsigned long long)key);
      seen = __shfl(seen, (int)((lane_id() & ~7u) + target), kWave);
      if (seen == kEmptyKey) { *created = true; return (u32)(line * kSlotsPerLine + target); }
      if (seen == key) return (u32)(line * kSlotsPerLine + target);
      slot_key = load_slot_key(&t.keys[line * kSlotsPerLine + sub]);   // another key took it
      continue;
    }
    line = line + 1 == t.n_lines ? 0 : line + 1;
    slot_key = load_slot_key(&t.keys[line * kSlotsPerLine + sub]);
  }
  return kNoRow;
}

// For a group of kLookupLanes lanes, after search_keys has found a key absent: claims a free slot
// for it, starting at `line` (whose slots may be out of date, the compare-and-swap decides).
// `seen` is what a first compare-and-swap on slot `target` of the line returned (issued by the
// caller, so that several keys' first attempts are in flight together).  *created tells whether
// this group created the key.  DISTINCT: no other group creates the same key at the same time
// (the keys of a pull), so only the free slot is raced for.  Otherwise another group may have put
// the key there meanwhile: slots of a line are only ever claimed in one order (slot_of_bit) and
// never freed, so whoever comes second meets the key before the next free slot.
template <bool DISTINCT>
__device__ __forceinline__ u32 claim_after4(const TableView& t, u64 key, u32 sub, u64 line, u32 target,
                                            u64 seen, bool* created) {
  *created = true;
  if (seen == kEmptyKey) return (u32)(line * kSlotsPerLine + target);
  if (!DISTINCT && seen == key) { *created = false; return (u32)(line * kSlotsPerLine + target); }
  for (u64 step = 0; step < 2 * t.n_lines; ++step) {
    // another key took the slot, or the line is full: look at the line as it is now
    const u64 x = load_slot_key(&t.keys[line * kSlotsPerLine + 2 * sub]);
    const u64 y = load_slot_key(&t.keys[line * kSlotsPerLine + 2 * sub + 1]);
    if (!DISTINCT) {
      const u32 hit = group4_bits(__ballot(x == key)) | (group4_bits(__ballot(y == key)) << 4);
      if (hit) {
        const u32 h = __ffs(hit) - 1;
        *created = false;
        return (u32)(line * kSlotsPerLine + 2 * (h & 3u) + (h >> 2));
      }
    }
    const u32 free_slots = group4_bits(__ballot(x == kEmptyKey)) | (group4_bits(__ballot(y == kEmptyKey)) << 4);
    if (!free_slots) { line = line + 1 == t.n_lines ? 0 : line + 1; continue; }
    const u32 b = __ffs(free_slots) - 1;
    const u32 slot = 2 * (b & 3u) + (b >> 2);
    u64 got = 0;
    if (sub == (b & 3u))
      got = atomicCAS((unsigned long long*)&t.keys[line * kSlotsPerLine + slot],
                      (unsigned long long)kEmptyKey, (unsigned long long)key);
    got = __shfl(got, (int)((lane_id() & ~3u) + (b & 3u)), kWave);
    if (got == kEmptyKey) return (u32)(line * kSlotsPerLine + slot);
    if (!DISTINCT && got == key) { *created = false; return (u32)(line * kSlotsPerLine + slot); }
  }
  *created = false;
  return kNoRow;
}

// ---- the pull's lookup -------------------------------------------------------------------
// A key's probe sequence starts at an even line, so that its first two lines are one 128-byte
// memory line (what a miss fetches anyway): four lanes look at those 16 slots at once.
struct BucketSlots {
  ulonglong2 a, b;      // lane sub: slots 2 sub and 2 sub + 1 of the even line (a) and of the odd one (b)
};
__device__ __forceinline__ BucketSlots load_bucket(const TableView& t, u64 line, u32 sub) {
  BucketSlots s;
  s.a = load_slot_pair(t, line, sub);
  s.b = load_slot_pair(t, line + 1, sub);
  return s;
}
__device__ __forceinline__ u32 slot_of_bit(u32 b) { return 2 * (b & 3u) + (b >> 2); }

// Data movement inside a group of four lanes (a quad): full-rate DPP moves, no LDS.
template <int CTRL> __device__ __forceinline__ u32 quad_perm(u32 v) {
  return (u32)__builtin_amdgcn_mov_dpp((int)v, CTRL, 0xF, 0xF, true);
}
// The value lane k of the quad holds (k = 0..3, a constant after unrolling).
__device__ __forceinline__ u32 quad_lane(u32 v, int k) {
  switch (k) {
    case 0: return quad_perm<0x00>(v);
    case 1: return quad_perm<0x55>(v);
    case 2: return quad_perm<0xAA>(v);
    default: return quad_perm<0xFF>(v);
  }
}
__device__ __forceinline__ u64 quad_lane(u64 v, int k) {
  return (u64)quad_lane((u32)v, k) | ((u64)quad_lane((u32)(v >> 32), k) << 32);
}
// Bitwise or over the quad, in every lane.
__device__ __forceinline__ u32 quad_or(u32 v) {
  v |= quad_perm<0xB1>(v);      // lanes 1 0 3 2
  v |= quad_perm<0x4E>(v);      // lanes 2 3 0 1
  return v;
}

// What a bucket holds for a key, as one word in every lane of the group: byte 0 = slots of the
// even line that hold the key, byte 1 = free slots of the even line, bytes 2 and 3 the same for
// the odd line; within a byte, bit b stands for slot 2 * (b & 3) + (b >> 2) (slot_of_bit).
__device__ __forceinline__ u32 bucket_bits(const BucketSlots& s, u64 key, u32 sub) {
  const u32 lo = 1u << sub, hi = 16u << sub;
  u32 m = (s.a.x == key ? lo : 0u) | (s.a.y == key ? hi : 0u);
  m |= (s.a.x == kEmptyKey ? lo << 8 : 0u) | (s.a.y == kEmptyKey ? hi << 8 : 0u);
  m |= (s.b.x == key ? lo << 16 : 0u) | (s.b.y == key ? hi << 16 : 0u);
  m |= (s.b.x == kEmptyKey ? lo << 24 : 0u) | (s.b.y == kEmptyKey ? hi << 24 : 0u);
  return quad_or(m);
}

// Searches for the K keys a group of four lanes has in flight.  Key k is owned by lane k % 4 (as
// its number k / 4): that lane keeps the key and, here, where its search stands (line) and what
// came of it (row, or kNoRow); the group fetches them from it when needed.  Every phase runs for
// all K keys before the next phase starts: a wave waits for memory once per round, not once per
// key (16 groups share a wave, and nearly always one of them has a key that needs another
// bucket).  Keys equal to kEmptyKey are not searched for.  Returns a mask: bit k = key k is absent,
// and its owner's `line` and `free_at` name the first free slot for it (free_at: bit 3 = in the
// line after `line`, bits 0..2 the slot).  The slots are read with plain (cacheable) loads: they
// may be out of date where the same kernel creates keys, and the compare-and-swap decides.
template <int K>
__device__ __forceinline__ u32 search_keys(const TableView& t, const u64* my_key, u64* my_line, u32* my_row,
                                           u32* my_free, u32 sub) {
  constexpr int OWN = K / kLookupLanes;
#pragma unroll
  for (int o = 0; o < OWN; ++o) {
    my_line[o] = home_line(t, my_key[o]);
    my_row[o] = kNoRow;
    my_free[o] = 0;
  }
  u32 open = 0;                 // bit k: key k is still being searched for
  BucketSlots slots[K];
#pragma unroll
  for (int k = 0; k < K; ++k) {
    const u64 key = quad_lane(my_key[k / kLookupLanes], k % kLookupLanes);
    const u64 line = quad_lane(my_line[k / kLookupLanes], k % kLookupLanes);
    if (key != kEmptyKey) {
      open |= 1u << k;
      slots[k] = load_bucket(t, line, sub);
    }
  }
  // rounds: look at the buckets at hand, fetch the next ones for the keys not settled
  u32 to_create = 0;            // bit k: key k is absent; its owner's my_free names the slot for it
  for (u64 step = 0; step < t.n_lines; step += 2) {
#pragma unroll
    for (int k = 0; k < K; ++k) {
      if (!(open >> k & 1u)) continue;
      const int o = k / kLookupLanes;
      const bool mine = sub == (u32)(k % kLookupLanes);
      const u64 key = quad_lane(my_key[o], k % kLookupLanes);
      const u32 bits = bucket_bits(slots[k], key, sub);
      const u32 hit_a = bits & 0xFFu, free_a = (bits >> 8) & 0xFFu;
      const u32 hit_b = (bits >> 16) & 0xFFu, free_b = bits >> 24;
      // (a key sits in the first line of its sequence that had a free slot when it came: if
      // the even line has a free slot the key is not in the odd one)
      if (hit_a) {
        if (mine) my_row[o] = (u32)(my_line[o] * kSlotsPerLine + slot_of_bit(__ffs(hit_a) - 1));
        open &= ~(1u << k);
      } else if (free_a) {
        if (mine) my_free[o] = slot_of_bit(__ffs(free_a) - 1);
        to_create |= 1u << k;
        open &= ~(1u << k);
      } else if (hit_b) {
        if (mine) my_row[o] = (u32)((my_line[o] + 1) * kSlotsPerLine + slot_of_bit(__ffs(hit_b) - 1));
        open &= ~(1u << k);
      } else if (free_b) {
        if (mine) my_free[o] = 8u | slot_of_bit(__ffs(free_b) - 1);
        to_create |= 1u << k;
        open &= ~(1u << k);
      } else if (mine) {
        my_line[o] = my_line[o] + 2 >= t.n_lines ? 0 : my_line[o] + 2;
      }
    }
    if (!__any(open != 0)) break;
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const u64 line = quad_lane(my_line[k / kLookupLanes], k % kLookupLanes);
      if (open >> k & 1u) slots[k] = load_bucket(t, line, sub);
    }
  }
  return to_create;
}

// Bucket form: what the lookup needs besides the spans to hand the rows on by position
// (partition.hpp: spread).
struct RowsByPosition {
  const u32* upos;       // null (plain form, accumulate): nothing is handed on
  u32* by_pos;
  u32* by_heavy;
};

// lds_rows: the rows of the span's keys (null: rows[] has them).
__device__ __forceinline__ void rows_by_position(const UniqueSpans& spans, const RowsByPosition& out, u32 c,
                                                 u32 first, const u32* rows, const u32* lds_rows) {
  const u32 end = spans.bucket_start[c + 1];
  const bool wide = (spans.count[c] & 0x80000000u) != 0;       // (bucket.hpp: upos_at)
  if (lds_rows && !wide) {
    // (two positions a lane and load, four loads in flight: one after the other, with rows[] from the L2, a block spent a fifth
    // of its time here; the whole lookup, 8.4 M occurrences of 0.27 M keys: 52 us, 44 with this; 20 since the blocks have
    // their own parts of the list of medium keys: OftenLists)
    constexpr int kTurns = 4;
    const u32* up = out.upos + first;
    for (u32 e0 = 2 * threadIdx.x; e0 < end - first; e0 += 2 * kProbeThreads * kTurns) {
      u32 w[kTurns];
#pragma unroll
      for (int q = 0; q < kTurns; ++q) {
        const u32 e = e0 + 2 * kProbeThreads * q;
        w[q] = e < end - first ? up[e / 2] : 0;
      }
#pragma unroll
      for (int q = 0; q < kTurns; ++q) {
        const u32 e = e0 + 2 * kProbeThreads * q;
        if (e < end - first) out.by_pos[first + e] = lds_rows[w[q] & 0xFFFFu];
        if (e + 1 < end - first) out.by_pos[first + e + 1] = lds_rows[w[q] >> 16];
      }
    }
    return;
  }
  const uint16_t* up = reinterpret_cast<const uint16_t*>(out.upos + first);
  for (u32 e = threadIdx.x; e < end - first; e += kProbeThreads)
    out.by_pos[first + e] = rows[first + (wide ? out.upos[first + e] : (u32)up[e])];
}

// What the host is told about the dedup (OftenLists::report).  One block.
//
// Buckets by range are uneven if the largest has half as many distinct keys again as the mean (hashed keys stay within a
// tenth; the slack is for small numbers).  Distinct keys are what counts, not occurrences: frequent keys make
// lumps in any form.  A block takes a bucket in the grouping, the lookup and the push, so the largest
// ends late in each: ids whose density rises from none to twice the mean, dim 16, 30 K, 105 K and 520 K
// occurrences a step of 75, 90 and 208 us by range, 65, 76 and 148 by hash.
__device__ __forceinline__ void report_dedup(const UniqueSpans& spans, const OftenLists& often) {
  __shared__ u32 s_sum, s_most;
  const PullCtx* ctx = often.ctx;
  if (threadIdx.x == 0) { often.heavy_next->count = 0; s_sum = s_most = 0; }
  __syncthreads();
  u32 sum = 0, most = 0;
  if (spans.bucket_start)
    for (u32 c = threadIdx.x; c < spans.n_spans; c += kProbeThreads) {
      const u32 u = spans.count[c] & 0x7FFFFFFFu;
      sum += u;
      most = max(most, u);
    }
  atomicAdd(&s_sum, sum);
  atomicMax(&s_most, most);
  __syncthreads();
  if (threadIdx.x != 0 || !often.report) return;
  const u32 mean = s_sum / spans.n_spans;
  const bool uneven = ctx->by_id == 1 && s_most > mean + mean / 2 + 64;
  const bool crowded = uneven && (s_most > 3 * mean + 256 || ctx->n_slow > ctx->n_slow_one_key);
  const u32 flags = (ctx->by_id > 1 ? kReportStandIn : 0u) |
                    (ctx->by_id != kSmallForm + 1 && (u64)ctx->n_slow * 8 > ctx->n_total ? kReportSlow : 0u) |      // (small.hpp reports by itself)
                    ((u64)ctx->n_slow_one_key * 2 >= ctx->n_slow ? kReportOneKey : 0u) |
                    (uneven ? kReportUneven : 0u) | (crowded ? kReportCrowded : 0u) |
                    (!ctx->by_id && ctx->n_evidence > kMaxEvidence ? kReportMixed : 0u);
  __hip_atomic_store(often.report + (ctx->by_id == 1 ? 1 : 0), (unsigned long long)often.serial | ((unsigned long long)flags << 32),
                     __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// How a lookup treats keys the table does not hold.
constexpr u32 kCreateNone = 0, kCreateIfRoom = 1, kCreateAtOnce = 2;
struct Creation {
  u32 how;
  u32 set;         // which of st->pull_made counts the created rows
  u32 new_cap;     // entries used of a block's list of created keys: all, except in tests of what happens when it is full
  // Per distinct key: `stamp`, the pull's number, if this pull created it.  Written where the table might be overfilled.  What is
  // left of other pulls carries their numbers: a block that stops early, at an error, leaves its part as it was.
  u32* fresh;
  u32 stamp;
};
// (the size does not change while a pull's kernels run: every thread decides the same)
__device__ __forceinline__ bool is_tight(const TableView& t, const Creation& create, u32 n) {
  return create.how == kCreateAtOnce && t.st->size + n > t.capacity;
}
// One thread of a pull's lookup: what end_pull decides by.
__device__ __forceinline__ void note_tight(const TableView& t, const Creation& create, bool tight) {
  if (create.how == kCreateNone) return;
  t.st->size_before = t.st->size;
  t.st->tight = tight ? 1u : 0u;
}

// Where in med_list the part of a block starts whose first occurrence (in the grouped order) is `first`; that of a group of heavy
// keys, h0 the first one's number, lies behind those of n occurrences.
__host__ __device__ constexpr u32 med_first(u32 first) { return first / (kShortSeg + 1); }
__host__ __device__ constexpr u32 med_first_heavy(u32 n, u32 h0) { return n / (kShortSeg + 1) + 1 + h0; }

// What the threads of a block that looks up keys gather, to be written out together at the end.
template <u32 NEW, u32 LONG>
struct LookupLds {
  static constexpr u32 kNew = NEW, kLong = LONG;
  u32 missing, n_new, n_med, n_long;
  uint4 long_list[LONG];  // (unique index, first chunk item, chunks, number) of very frequent keys
  u64 new_key[NEW];       // created keys, and their rows
  u32 new_row[NEW];
  __device__ __forceinline__ void clear() { missing = n_new = n_med = n_long = 0; }
};

// The row of my_key (kEmptyKey: none), one key per lane of a group of four; *mine_new: it was created just now.
//
// A group of four lanes looks at a bucket of the table at once and has four keys in flight, one per lane:
// each lane loads and hashes its own key and, at the end, stores its own key's row and lists it
// (one key per lane: full waves); in between the group goes through its four keys together
// (search_keys).
template <typename LDS>
__device__ __forceinline__ u32 lookup_key(const TableView& t, u64 my_key, bool create_here, u32 new_cap, LDS& L, bool* mine_new) {
  constexpr int K = kPullInFlight;            // keys a group has in flight
  static_assert(K == kLookupLanes, "one key per lane");
  const u32 sub = threadIdx.x % kLookupLanes;
  const u32 lane0 = lane_id() & ~3u;          // the group's first lane
  u64 my_line;
  u32 my_row, my_free;
  *mine_new = false;
  const u32 to_create = search_keys<K>(t, &my_key, &my_line, &my_row, &my_free, sub);
  // keys to create: all first attempts in flight together, then whatever is left of each
  if (create_here && __any(to_create != 0)) {
    u64 seen[K];
    my_line += my_free >> 3;        // the line of the free slot
#pragma unroll
    for (int q = 0; q < K; ++q) {
      const u64 key = quad_lane(my_key, q);
      const u64 line = quad_lane(my_line, q);
      const u32 slot = quad_lane(my_free, q) & 7u;
      seen[q] = 0;
      if ((to_create >> q & 1u) && sub == slot >> 1)
        seen[q] = atomicCAS((unsigned long long*)&t.keys[line * kSlotsPerLine + slot],
                            (unsigned long long)kEmptyKey, (unsigned long long)key);
    }
#pragma unroll
    for (int q = 0; q < K; ++q) {
      const u64 key = quad_lane(my_key, q);
      const u64 line = quad_lane(my_line, q);
      const u32 slot = quad_lane(my_free, q) & 7u;
      if (!(to_create >> q & 1u)) continue;
      const u64 got = __shfl(seen[q], (int)(lane0 + (slot >> 1)), kWave);
      bool created;
      const u32 row = claim_after4<true>(t, key, sub, line, slot, got, &created);
      if (row == kNoRow) {
        raise_error(t.st, kErrInternal);            // (cannot happen: the table has room)
        continue;
      }
      // The new row's initial values are left to the end of the kernel, where all lanes of
      // the block share the work (here four lanes of the wave would do it while sixty wait);
      // only a key that finds the block's list full gets them right away.
      u32 at = 0;
      if (sub == (u32)q) {
        my_row = row;
        *mine_new = true;
        at = atomicAdd(&L.n_new, 1u);
        if (at < new_cap) { L.new_key[at] = key; L.new_row[at] = row; }
      }
      if (quad_lane(at, q) >= new_cap) {
        const u64 base = mix64(key ^ t.init_seed);
        for (u32 j = sub; j < t.dim; j += kLookupLanes) store_w(t, row, j, init_weight(base, j, t.init_range));
        float* ar = acc_row(t, row);
        for (u32 j = sub; j < t.acc_len; j += kLookupLanes) ar[j] = t.init_acc;
      }
    }
  }
  return my_row;
}

// Puts distinct key number u into the push's work lists, by its number of occurrences, and into the hint for later dedups.
template <typename LDS>
__device__ __forceinline__ void list_key(const OftenLists& often, u32 med_base, u32 u, u64 key, u32 len, LDS& L) {
  PullCtx* ctx = often.ctx;
  if (len >= often.heavy_min && key != kEmptyKey) {
    const u32 at = atomicAdd(&often.heavy_raw->count, 1u);
    if (at < (u32)kMaxHeavy) often.heavy_raw->keys[at] = key;
  }
  if (len > often.pieces.medium) {
    const u32 n_chunks = (len + often.pieces.chunk - 1) / often.pieces.chunk;
    const u32 item = atomicAdd(&ctx->n_chunk_items, n_chunks);
    const u32 number = atomicAdd(&ctx->n_long, 1u);
    often.arrived[number] = 0;
    // the key's chunk items are written at the end of the kernel by all lanes of a wave
    // (a key that fills thousands of chunks would keep this lane, and its wave, for long)
    const u32 at = atomicAdd(&L.n_long, 1u);
    if (at < LDS::kLong) {
      L.long_list[at] = make_uint4(u, item, n_chunks, number);
    } else {
      for (u32 i = 0; i < n_chunks; ++i) often.chunk_items[item + i] = make_uint4(u, i, number, item);
    }
  } else if (len > kShortSeg) {
    often.med_list[med_base + atomicAdd(&L.n_med, 1u)] = u;
  }
}

// After a barrier: writes out what the block's threads have gathered.
template <int THREADS, typename LDS>
__device__ __forceinline__ void end_lookup(const TableView& t, const OftenLists& often, const Creation& create, u32 med_base, LDS& L) {
  if (threadIdx.x == 0) {
    if (L.n_new) atomicAdd(&t.st->pull_made[create.set][blockIdx.x % kCountShards], L.n_new);
    if (L.missing) atomicAdd(&t.st->miss_shard[blockIdx.x % kCountShards], L.missing);
    often.med_span[blockIdx.x] = make_uint2(med_base, L.n_med);
  }
  {
    const u32 n_long_here = min(L.n_long, LDS::kLong);
    for (u32 e = threadIdx.x / kWave; e < n_long_here; e += THREADS / kWave) {
      const uint4 it = L.long_list[e];
      for (u32 i = lane_id(); i < it.z; i += kWave) often.chunk_items[it.y + i] = make_uint4(it.x, i, it.w, it.y);
    }
  }
  // the initial rows of the keys created above: one float4 of one row per lane and turn
  const u32 n_new = min(L.n_new, min(create.new_cap, LDS::kNew));
  const u32 dim4 = t.dim >> 2;
  for (u32 e = threadIdx.x; e < n_new * dim4; e += THREADS) {
    const u32 i = e / dim4, col = e % dim4;
    store_w4(t, L.new_row[i], col, init_weight4(mix64(L.new_key[i] ^ t.init_seed), col, t.init_range));
  }
  for (u32 e = threadIdx.x; e < n_new * t.acc_len; e += THREADS)
    acc_row(t, L.new_row[e / t.acc_len])[e % t.acc_len] = t.init_acc;
}

// rows[u] = the slot of distinct key u.  Keys the table does not hold:
//  - kCreateNone (accumulate): rows[u] = kNoRow, counted in st->miss_shard;
//  - kCreateAtOnce: the key is created right here, with its initial row (the line is at hand, and so are its free
//    slots), counted in st->pull_made; end_pull takes them all out again if the table ended above its capacity;
//  - kCreateIfRoom (a mini-batch too large beside the table for that): the same if the table has room for all the
//    keys even if every one of them is new, otherwise rows[u] = kNoRow, counted in st->miss_shard, for
//    pull_missing, which creates all of them or none.
// Also sorts the keys into the push's work lists by their number of occurrences, and (bucket form)
// hands the rows on by position.  One span of distinct keys or group of heavy keys per block; the block behind
// them reports on the dedup.
__global__ void __launch_bounds__(kProbeThreads)
pull_lookup(TableView t, const u64* __restrict__ keys, const u32* __restrict__ seg_off, UniqueSpans spans,
            u32* __restrict__ rows, RowsByPosition out, Creation create, OftenLists often) {
  typedef LookupLds<kNewLdsCap, kLongLdsCap> Lds;
  __shared__ Lds L;
  __shared__ u32 s_rows[kRowsLdsCap];
  __shared__ u32 s_unique;
  PullCtx* ctx = often.ctx;
  const bool tight = is_tight(t, create, ctx->n_total);
  if (blockIdx.x == span_blocks(spans)) {
    if (threadIdx.x == 0) note_tight(t, create, tight);
    report_dedup(spans, often);
    return;
  }
  if (ctx->sort_error != 0) {     // the dedup before this lookup failed
    if (threadIdx.x == 0) raise_error(t.st, kErrInternal);
    return;
  }
  if (load_error(t.st) != 0) return;
  const bool heavies = blockIdx.x < heavy_blocks(spans);
  const u32 c = blockIdx.x - heavy_blocks(spans);        // the span
  const u32 h0 = blockIdx.x * kHeavyGroup;               // or the first heavy key
  u32 first = 0, count;
  if (heavies) count = ctx->n_heavy > h0 ? min(kHeavyGroup, ctx->n_heavy - h0) : 0u;
  else unique_span(spans, ctx, c, &first, &count);
  if (count == 0) {
    if (threadIdx.x == 0) often.med_span[blockIdx.x] = make_uint2(0u, 0u);
    return;
  }
  const u32 med_base = heavies ? med_first_heavy(ctx->n_total, h0) : med_first(spans.bucket_start ? first : seg_off[first]);
  if (threadIdx.x == 0) L.clear();
  if (create.how == kCreateIfRoom && threadIdx.x < kWave) {
    // (kCountShards == kWave) distinct keys of the whole mini-batch
    const u32 u = wave_incl_sum(ctx->uniq_shard[threadIdx.x]);
    if (threadIdx.x == kWave - 1) s_unique = ctx->by_id ? u : ctx->n_unique;
  }
  __syncthreads();
  const bool create_here = create.how == kCreateAtOnce || (create.how == kCreateIfRoom && t.st->size + s_unique <= t.capacity);
  u32 missing = 0;
  // (the bound is the same for all lanes of a group, so a group stays together)
  for (u32 k0 = threadIdx.x & ~3u; k0 < count; k0 += kProbeThreads) {
    const u32 k = k0 + threadIdx.x % kLookupLanes;
    u64 my_key = kEmptyKey;
    u32 my_len = 0, u = 0;
    bool on = k < count, mine_new;
    if (heavies) {
      const u32 h = h0 + k;
      if (on) {
        u = spans.bucket_start[spans.n_spans + h];
        const u32 end = spans.bucket_start[spans.n_spans + h + 1];
        my_len = end - u;
        on = my_len != 0;                      // a key the hint named and the mini-batch does not hold
        if (on) my_key = keys[u];
      }
    } else if (on) {
      u = first + k;
      my_key = keys[u];
      my_len = seg_off[u + 1] - seg_off[u];
    }
    const u32 my_row = lookup_key(t, my_key, create_here, create.new_cap, L, &mine_new);
    // every lane: the row of its own key, and the push's work lists
    if (!on) continue;
    rows[u] = my_row;
    if (!heavies && k < kRowsLdsCap) s_rows[k] = my_row;
    if (tight && mine_new) create.fresh[u] = create.stamp;
    if (heavies && out.upos) out.by_heavy[h0 + k] = my_row;
    if (my_row == kNoRow) ++missing;
    list_key(often, med_base, u, my_key, my_len, L);
  }
  if (missing) atomicAdd(&L.missing, missing);
  __syncthreads();
  if (out.upos && !heavies) rows_by_position(spans, out, c, first, rows, count <= kRowsLdsCap ? s_rows : nullptr);      // (this block's own rows[])
  end_lookup<kProbeThreads>(t, often, create, med_base, L);
}

// Whether the keys a lookup found missing (st->miss_shard) may be created: 0 there are none, 1 yes,
// 2 no (the table would overflow; the error is raised).  All threads of the block.
__device__ __forceinline__ u32 may_create(const TableView& t, u32* s_word) {
  if (threadIdx.x < kWave) {
    const u32 total = wave_incl_sum(threadIdx.x < kCountShards ? t.st->miss_shard[threadIdx.x] : 0);
    if (threadIdx.x == kWave - 1) *s_word = total;
  }
  __syncthreads();
  const u32 total = *s_word;
  if (total == 0) return 0;
  // st->size does not change while this kernel runs: every block decides the same
  if (t.st->size + total <= t.capacity) return 1;
  if (threadIdx.x == 0) raise_error(t.st, kErrFull);
  return 2;
}

// Finds or creates `key` (all eight lanes of a group); a new row is given w / acc (null: the
// deterministic initial values / init_acc).
__device__ __forceinline__ u32 find_or_create(const TableView& t, u64 key, u32 sub, const float* w, const float* acc,
                                              bool* created) {
  const u64 line = home_line(t, key);
  const u64 slot_key = load_slot_key(&t.keys[line * kSlotsPerLine + sub]);
  const u32 row = probe_find_or_claim(t, key, sub, line, slot_key, created);
  if (!*created) return row;
  const u64 base = mix64(key ^ t.init_seed);
  for (u32 j = sub; j < t.dim; j += 8) store_w(t, row, j, w ? w[j] : init_weight(base, j, t.init_range));
  float* ar = acc_row(t, row);
  for (u32 j = sub; j < t.acc_len; j += 8) ar[j] = acc ? acc_value(acc[j]) : t.init_acc;
  return row;
}

// Creates the keys that insert_rows found missing and left to it, if the table has room for all of them (a
// key that occurs twice in a bulk insert is counted twice for this check).
__global__ void __launch_bounds__(kProbeThreads)
insert_missing(TableView t, const u64* __restrict__ keys, u64 n_keys, const float* __restrict__ w_in,
               const float* __restrict__ acc_in) {
  __shared__ u32 s_word, s_made;
  if (load_error(t.st) != 0) return;
  if (threadIdx.x == 0) s_made = 0;
  if (may_create(t, &s_word) != 1) return;
  const u32 sub = threadIdx.x & 7;
  u32 made = 0;
  for (u64 u = (u64)blockIdx.x * kProbeGroups + (threadIdx.x >> 3); u < n_keys; u += (u64)gridDim.x * kProbeGroups) {
    bool created;
    (void)find_or_create(t, keys[u], sub, w_in ? w_in + u * t.dim : nullptr,
                         acc_in ? acc_in + u * t.acc_len : nullptr, &created);
    if (created) ++made;
  }
  if (sub == 0 && made) atomicAdd(&s_made, made);
  __syncthreads();
  if (threadIdx.x == 0 && s_made) atomicAdd(&t.st->made_shard[blockIdx.x % kCountShards], s_made);
}

// The same for a pull, whose lookup left rows[u] == kNoRow; hands the rows on by position again.  One span
// of distinct keys or group of heavy keys per block, as the lookup.  The keys to create are
// gathered in LDS first, so that all groups have one at a time (one key in six is a new one: 0.49 M new
// keys of 2.8 M, 140 us; 278 with every group looking for its own).
__global__ void __launch_bounds__(kProbeThreads)
pull_missing(TableView t, const u64* __restrict__ keys, UniqueSpans spans, const PullCtx* __restrict__ ctx,
             u32* __restrict__ rows, RowsByPosition out, u32 set) {
  constexpr u32 kList = 1024;
  __shared__ u32 s_word, s_made, s_n;
  __shared__ u32 s_list[kList];
  if (load_error(t.st) != 0) return;
  if (threadIdx.x == 0) s_made = 0;
  if (may_create(t, &s_word) != 1) return;
  const u32 sub = threadIdx.x & 7;
  const bool heavies = blockIdx.x < heavy_blocks(spans);
  const u32 c = blockIdx.x - heavy_blocks(spans), h0 = blockIdx.x * kHeavyGroup;
  u32 first = 0, count, made = 0;
  if (heavies) count = ctx->n_heavy > h0 ? min(kHeavyGroup, ctx->n_heavy - h0) : 0u;
  else unique_span(spans, ctx, c, &first, &count);
  const u32* start = spans.bucket_start + spans.n_spans + h0;       // (heavy keys)
  u32 k0 = 0;
  while (k0 < count) {
    __syncthreads();
    if (threadIdx.x == 0) s_n = 0;
    __syncthreads();
    for (; k0 < count && s_n <= kList - kProbeThreads; k0 += kProbeThreads) {       // (s_n: read between barriers)
      const u32 k = k0 + threadIdx.x;
      __syncthreads();
      if (k < count && !(heavies && start[k] == start[k + 1]) && rows[heavies ? start[k] : first + k] == kNoRow)
        s_list[atomicAdd(&s_n, 1u)] = k;
      __syncthreads();
    }
    const u32 n = s_n;
    for (u32 e = threadIdx.x >> 3; e < n; e += kProbeGroups) {
      const u32 k = s_list[e], u = heavies ? start[k] : first + k;
      bool created;
      const u32 row = find_or_create(t, keys[u], sub, nullptr, nullptr, &created);
      if (created) ++made;
      if (sub == 0) {
        rows[u] = row;
        if (heavies && out.upos) out.by_heavy[h0 + k] = row;
      }
    }
  }
  if (sub == 0 && made) atomicAdd(&s_made, made);
  __syncthreads();
  if (threadIdx.x == 0 && s_made) atomicAdd(&t.st->pull_made[set][blockIdx.x % kCountShards], s_made);
  if (out.upos && !heavies) rows_by_position(spans, out, c, first, rows, nullptr);
}

// What the pooling kernel, the last one of a pull, needs to end it.
struct PullEnd {
  u32 set;                 // of st->pull_made
  UniqueSpans spans;
  const PullCtx* ctx;
  const u32* rows;
  const u32* fresh;        // (Creation)
  u32 stamp;
};
// All threads of all blocks, before anything else.  Books the rows the lookup created -- or, if the table ended above
// its capacity, raises kErrFull and takes them out of it (nothing else has been put behind them: the table
// is as before).  Every block adds up the same counts, so all come to the same end, whichever raises the error
// first.  What was created stays booked if an error has come from elsewhere meanwhile (a mini-batch being prepared beside this
// pull, with the reserved key in it): the rows are in the table.  Returns false if the pull has failed, now or before.
__device__ __forceinline__ bool end_pull(const TableView& t, const PullEnd& e) {
  static_assert(kCountShards == kWave, "a count per lane");
  const int error = load_error(t.st);
  const u32 tight = t.st->tight, mine = t.st->pull_made[e.set][lane_id()];
  if (!tight && blockIdx.x != 0) return error == 0;
  const u32 made = (u32)__builtin_amdgcn_readlane((int)wave_incl_sum(mine), kWave - 1);
  const bool overfull = tight && t.st->size_before + made > t.capacity;
  if (blockIdx.x == 0 && threadIdx.x < kWave) {
    t.st->pull_made[1 - e.set][threadIdx.x] = 0;
    t.st->miss_shard[threadIdx.x] = 0;
    if (threadIdx.x == 0 && !overfull && (error == 0 || made != 0)) {
      t.st->size += made;
      t.st->inserted = made;
    }
  }
  if (!overfull) return error == 0;
  if (threadIdx.x == 0) raise_error(t.st, kErrFull);
  for (u32 b = blockIdx.x; b < span_blocks(e.spans); b += gridDim.x) {
    const bool heavies = b < heavy_blocks(e.spans);
    const u32 h0 = b * kHeavyGroup;
    u32 first = 0, count;
    if (heavies) count = e.ctx->n_heavy > h0 ? min(kHeavyGroup, e.ctx->n_heavy - h0) : 0u;
    else unique_span(e.spans, e.ctx, b - heavy_blocks(e.spans), &first, &count);
    for (u32 k = threadIdx.x; k < count; k += blockDim.x) {
      u32 u = first + k;
      if (heavies) {
        u = e.spans.bucket_start[e.spans.n_spans + h0 + k];
        if (e.spans.bucket_start[e.spans.n_spans + h0 + k + 1] == u) continue;
      }
      if (e.fresh[u] == e.stamp) t.keys[e.rows[u]] = kEmptyKey;
    }
  }
  return false;
}

// How many buckets (pairs of lines: 128 bytes) a lookup reads to find each stored key (1 = the
// key sits in the bucket its hash names): sum and maximum over all stored keys, into st->probe_sum / probe_max (zero on
// entry).
__global__ void __launch_bounds__(256) probe_length_scan(TableView t) {
  __shared__ unsigned long long s_sum, s_max;
  if (threadIdx.x == 0) { s_sum = 0; s_max = 0; }
  __syncthreads();
  const u64 n_slots = t.n_lines * kSlotsPerLine;
  unsigned long long sum = 0, most = 0;
  for (u64 s = (u64)blockIdx.x * blockDim.x + threadIdx.x; s < n_slots; s += (u64)gridDim.x * blockDim.x) {
    const u64 key = t.keys[s];
    if (key == kEmptyKey) continue;
    const u64 home = home_line(t, key), line = s / kSlotsPerLine;
    const u64 lines = (line >= home ? line - home : line + t.n_lines - home) / 2 + 1;
    sum += lines;
    most = max(most, (unsigned long long)lines);
  }
#pragma unroll
  for (int d = 1; d < kWave; d <<= 1) {
    sum += __shfl_xor(sum, d, kWave);
    most = max(most, (unsigned long long)__shfl_xor(most, d, kWave));
  }
  if (lane_id() == 0) { atomicAdd(&s_sum, sum); atomicMax(&s_max, most); }
  __syncthreads();
  if (threadIdx.x == 0) { atomicAdd(&t.st->probe_sum, s_sum); atomicMax(&t.st->probe_max, s_max); }
}
__global__ void clear_probe_lengths(TableState* st) { st->probe_sum = 0; st->probe_max = 0; }

}  // namespace hps
