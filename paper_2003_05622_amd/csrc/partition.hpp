// Key dedup, bucket form, part 1: the key occurrences are dealt into buckets in one stable pass,
// without any workgroup waiting for another.
//
// A bucket is one of n_nat parts of the mini-batch's keys, a few hundred to a few thousand occurrences each, or
// one frequent ("heavy") key, which a hint from an earlier lookup names (common.hpp): those would make single
// buckets too large for bucket.hpp, and their occurrences need no grouping.  The heavy buckets follow the n_nat
// natural ones in the order of the hint.  The parts are
//   by range    equal parts of the mini-batch's key range (sampled; for hashed keys: of all 64 bits): the usual way;
//   by borders  parts with equal shares of the occurrences, between sampled borders; and
//   by hash     parts of the keys' hashes: for keys that lie unevenly in their range (raw ids), so that equal parts of
//               it would hold very different numbers of them.
// By range and by borders, buckets 0 .. n_nat-1 are in key order, which hps_last_unique builds on.
// Two launches for few tiles, else three, and one more by borders:
//
//   sample_borders   (by borders) the borders of buckets of equal shares;
//   bucket_count     a tile of consecutive occurrences per block: bucket of every key (id16), counts
//                    per bucket (hist[tile][bucket]); further blocks note which bag every tile
//                    starts in;
//   scan_buckets     counts -> for every tile and bucket the occurrences in earlier tiles
//                    (prefix[tile][bucket]), and how many every bucket holds (total); left out
//                    for up to kDirectTiles tiles, where every block of the scatter adds the counts up itself;
//   bucket_scatter   a tile ranks its occurrences per bucket in occurrence order, stages them in LDS
//                    and writes every bucket's run contiguously: the key (not for heavy
//                    buckets), the bag.  It also leaves, per tile in the order of the
//                    destinations, where each occurrence went (code) and which of the tile's it was
//                    (from): what spread() needs to bring per-position results back into
//                    occurrence order with whole runs read, a tile's worth of LDS scattered and whole lines
//                    written (an occurrence's index does not travel with the pair).
//
// One pass with thousands of buckets instead of two 8-bit passes: what a scatter pays for is
// write requests, and a run of five occurrences (one or two requests for its keys, one for its
// bags) costs two requests where the second pass cost a read and a write of every pair.
#pragma once

#include "common.hpp"
#include "form.hpp"
#include "sort.hpp"

namespace hps {

struct BucketPlan {
  u32 n_nat;        // natural buckets
  u32 max_heavy;    // heavy keys that get buckets of their own, at most
  u32 stride;       // words from one tile's counts to the next, >= n_nat + max_heavy
  u32 n_tiles;
};

constexpr u32 kHeavyCode = 0x80000000u;   // code of an occurrence in heavy bucket h: kHeavyCode | h, else its position
constexpr u32 kDirectTiles = 64;
constexpr int kHeavySlots = 4096;         // hash slots for the heavy keys (a power of two)
constexpr u32 kNoHeavy = ~0u;

// Which part of the key range a key lies in.
__device__ __forceinline__ u32 bucket_of(u64 key, const KeyRange& r) {
  const u64 rel = range_rel(key, r);
  return r.direct ? (u32)rel : (u32)(((rel >> r.pre) * r.mult) >> 32);
}
__device__ __forceinline__ KeyRange bucket_range(u64 lo, u64 hi, u32 n_nat) {
  KeyRange r = widened_range(lo, hi);
  r.direct = r.span < n_nat;
  // span >= n_nat here, so the quotient is below 2^32, and parts are numbered below n_nat
  r.mult = r.direct ? 0u : (u32)(((u64)n_nat << 32) / ((r.span >> r.pre) + 1));
  return r;
}

// Sampled borders, for keys that bunch in parts of their range (raw ids, whose frequent ones are often
// neighbours): bucket b holds the keys from border[b - 1] up to border[b], the quantiles of
// evenly spaced samples, so that every bucket gets about the same share wherever the keys lie.  n_nat - 1 borders in ascending order, some perhaps equal (a frequent key).
// Eight samples a bucket: one of s times the mean has fewer than nine where 8 s are expected, a chance of 5e-5 for
// s = 3 (one mini-batch of 1024 buckets in twenty), 1e-7 for s = 4 and 1e-12 for s = 6.  So the workgroups
// are chosen to hold six times the mean in distinct keys and eight times in occurrences (border_group_threads).
// Larger mini-batches would take more samples than one kernel of a few microseconds can rank (with as many, 1 M
// occurrences took 359 to 372 us by borders, 376 to 396 in the plain form, and listing the unique keys costs 50 us more).
constexpr u32 kMaxBorders = 1024;
__host__ constexpr u32 border_group_threads(u64 n) { return n <= (1u << 18) ? 256 : 512; }
constexpr u32 border_samples(u32 max_nat) { return 8 * max_nat; }
__device__ __forceinline__ u32 bucket_by_border(u64 key, const u64* border, u32 n_borders) {
  u32 at = 0;
#pragma unroll
  for (u32 step = kMaxBorders / 2; step; step >>= 1)
    if (at + step <= n_borders && border[at + step - 1] <= key) at += step;
  return at;
}
static_assert(kMaxBorders / 2 * 2 - 1 >= kMaxBorders - 1, "the steps add up to the most borders there are");
// Whether a key lies in natural bucket c (border == null: equal parts of the range).
__device__ __forceinline__ bool in_bucket(u64 key, u32 c, const KeyRange& r, const u64* border, u32 n_nat) {
  if (!border) return bucket_of(key, r) == c;
  return (c == 0 || border[c - 1] <= key) && (c + 1 == n_nat || key < border[c]);
}

// Puts the borders down.  A block holds all samples in LDS and ranks 64 of them, one per lane of each
// wave, against a sixteenth of all per wave (every lane reads the same word: no conflicts); equal keys
// go by their number.  The sample of rank r is border b where b * SAMPLES / n_nat == r.  Ranking takes SAMPLES
// squared comparisons: 28 us for 8192 samples, 9 for the 2048 of up to 2^16 occurrences.
constexpr int kBorderThreads = 1024;
template <u32 SAMPLES>
__global__ void __launch_bounds__(kBorderThreads)
sample_borders(const u64* __restrict__ keys, u32 n, u32 n_nat, u64* __restrict__ border) {
  constexpr u32 kPart = SAMPLES / (kBorderThreads / kWave);
  __shared__ u64 key[SAMPLES];
  __shared__ u32 rank[kWave];
#pragma unroll
  for (u32 j = threadIdx.x; j < SAMPLES; j += kBorderThreads) key[j] = keys[(u64)j * n / SAMPLES];
  if (threadIdx.x < kWave) rank[threadIdx.x] = 0;
  __syncthreads();
  const u32 me = blockIdx.x * kWave + lane_id(), first = threadIdx.x / kWave * kPart;
  const u64 mine = key[me];
  u32 before = 0;
#pragma unroll 8
  for (u32 j = first; j < first + kPart; ++j) before += key[j] < mine || (key[j] == mine && j < me) ? 1u : 0u;
  atomicAdd(&rank[lane_id()], before);
  __syncthreads();
  if (threadIdx.x < kWave) {
    const u32 r = rank[threadIdx.x], b = (r * n_nat + SAMPLES - 1) / SAMPLES;
    if (b >= 1 && b < n_nat && b * SAMPLES / n_nat == r) border[b - 1] = mine;
  }
}

// Hash for the LDS tables (top bits): the two halves of the key through MurmurHash3's 32-bit finaliser
// (Appleby; its last shift leaves the top bits alone).  One multiplication would do for ids and for well-mixed keys, but
// keys that are multiples of some number (ids spread by a multiplication) can meet it with all keys of a
// bucket in a row: 30 K distinct keys that are multiples of the multiplier's inverse, a step of 236 us, 59 with this;
// 1 M that are multiples of a sixteenth of it, 334 and 216 us (of the multiplier itself, which one multiplication
// spreads evenly: 180 and 217).
__device__ __forceinline__ u32 key_hash(u64 key) {
  u32 h = (u32)key ^ (u32)(key >> 32) * 0x9E3779B1u;
  h = (h ^ h >> 16) * 0x85EBCA6Bu;
  return (h ^ h >> 13) * 0xC2B2AE35u;
}

// The heavy keys in LDS: an open-addressing hash from key to its index in the list.
struct HeavyLds {
  u64 keys[kMaxHeavy + 1];
  u32 slot[kHeavySlots];
};
// Step 1 of 2 (a barrier after each): all threads copy the list and clear the slots.
template <int THREADS>
__device__ __forceinline__ void heavy_copy(HeavyLds& H, const HeavyRaw* raw, u32 count) {
  for (u32 i = threadIdx.x; i < count; i += THREADS) H.keys[i] = raw->keys[i];
  if (count)
    for (u32 i = threadIdx.x; i < (u32)kHeavySlots; i += THREADS) H.slot[i] = kNoHeavy;
}
// Step 2: a key that is listed twice goes by its first index, in every block.
template <int THREADS>
__device__ __forceinline__ void heavy_index(HeavyLds& H, u32 count) {
  for (u32 i = threadIdx.x; i < count; i += THREADS) {
    const u64 key = H.keys[i];
    u32 s = key_hash(key) >> 20;
    while (true) {       // (at most kMaxHeavy of the kHeavySlots slots are ever taken)
      const u32 old = atomicCAS(&H.slot[s], kNoHeavy, i);
      if (old == kNoHeavy) break;
      if (H.keys[old] == key) { atomicMin(&H.slot[s], i); break; }
      s = (s + 1) & (kHeavySlots - 1);
    }
  }
}
__device__ __forceinline__ u32 heavy_find(const HeavyLds& H, u64 key) {
  u32 s = key_hash(key) >> 20;
  while (true) {
    const u32 i = H.slot[s];
    if (i == kNoHeavy || H.keys[i] == key) return i;
    s = (s + 1) & (kHeavySlots - 1);
  }
}
static_assert(kHeavySlots == 1 << 12, "a slot is the top 12 bits of the hash");

// First kernel of a bucket-form dedup, one tile of THREADS * ITEMS occurrences per block for the
// first plan.n_tiles blocks; the blocks behind them look through the bag offsets and leave in
// tile_bag[t] the bag that holds occurrence t * tile (offsets == null: every occurrence is its
// own bag, nothing to do).  Block 0 also resets the pull context.
// FORM: kByRange, kByBorders or kByHash.
template <int THREADS, int ITEMS, int MAX_BUCKETS, int FORM>
__global__ void __launch_bounds__(THREADS, 8)
bucket_count(const u64* __restrict__ keys, u32 n, BucketPlan plan, const u64* __restrict__ border, PullCtx* __restrict__ ctx,
             const i32* __restrict__ offsets, u32 n_bags, u32* __restrict__ tile_bag,
             const HeavyRaw* __restrict__ heavy, uint16_t* __restrict__ id16, uint16_t* __restrict__ hist) {
  constexpr u32 kTile = THREADS * ITEMS;
  if (blockIdx.x >= plan.n_tiles) {
    const u32 first = (blockIdx.x - plan.n_tiles) * THREADS + threadIdx.x, step = (gridDim.x - plan.n_tiles) * THREADS;
    for (u32 b = first; b < n_bags; b += step) {
      const u32 lo = (u32)max(offsets[b], 0), hi = min((u32)max(offsets[b + 1], 0), n);
      for (u32 t = (lo + kTile - 1) / kTile; t < plan.n_tiles && t * kTile < hi; ++t) tile_bag[t] = b;
    }
    return;
  }
  __shared__ u32 h[MAX_BUCKETS];
  __shared__ HeavyLds hv;
  __shared__ u64 s_lo[THREADS / kWave], s_hi[THREADS / kWave];
  __shared__ KeyRange s_range;
  __shared__ u64 s_border[FORM == kByBorders ? kMaxBorders : 1];
  // the tile is requested before anything waits for the samples and the list
  const u32 base = blockIdx.x * kTile;
  u64 key[ITEMS];
#pragma unroll
  for (int k = 0; k < ITEMS; ++k) key[k] = keys[min(base + k * THREADS + threadIdx.x, n - 1)];
  const u32 n_heavy = min(heavy->count, plan.max_heavy);
  if (FORM == kByBorders) {
    for (u32 b = threadIdx.x; b + 1 < plan.n_nat; b += THREADS) s_border[b] = border[b];
  } else if (FORM == kByRange) {
    sample_key_range<THREADS>(keys, n, s_lo, s_hi);
  }
  heavy_copy<THREADS>(hv, heavy, n_heavy);
  const u32 n_buckets = plan.n_nat + n_heavy;
  for (u32 b = threadIdx.x; b < n_buckets; b += THREADS) h[b] = 0;
  if (blockIdx.x == 0) reset_ctx(ctx, n, (u32)FORM + 1, n_heavy);
  __syncthreads();
  heavy_index<THREADS>(hv, n_heavy);
  if (FORM == kByRange && threadIdx.x == 0) {
    u64 lo, hi;
    sampled_ends<THREADS>(s_lo, s_hi, &lo, &hi);
    s_range = bucket_range(lo, hi, plan.n_nat);
    if (blockIdx.x == 0) ctx->range = s_range;
  }
  __syncthreads();
  const KeyRange range = s_range;
#pragma unroll
  for (int k = 0; k < ITEMS; ++k) {
    const u32 i = base + k * THREADS + threadIdx.x;
    if (i < n) {
      // (by another hash than the groups' LDS tables: the keys of a bucket share its leading bits)
      u32 id = FORM == kByBorders ? bucket_by_border(key[k], s_border, plan.n_nat - 1)
               : FORM == kByHash  ? __umulhi((u32)(slot_hash(key[k]) >> 32), plan.n_nat)
                                  : bucket_of(key[k], range);
      if (n_heavy) {
        const u32 at = heavy_find(hv, key[k]);
        if (at != kNoHeavy) id = plan.n_nat + at;
      }
      id16[i] = (uint16_t)id;
      atomicAdd(&h[id], 1u);
    }
  }
  __syncthreads();
  uint16_t* row = hist + (u64)blockIdx.x * plan.stride;
  for (u32 b = threadIdx.x; b < n_buckets; b += THREADS) row[b] = (uint16_t)h[b];
}

// prefix[tile][bucket] and total[bucket].  A block takes 16 buckets and shares the tiles out over
// 64 groups of 16 lanes, PER tiles each, kept in registers between the two halves of the scan.  What bounds it
// is latency: few blocks, each with all its loads in flight at once.  The starts of the buckets (a
// scan of the totals) are left to every block of the scatter: the block that is done last
// here could scan them too, but the device-scope fence that takes costs each block a write-back of
// its L2 (9.8 M occurrences: 139 us with it).
constexpr int kScanThreads = 1024;
constexpr int kScanBuckets = 16;
constexpr int kScanChunks = kScanThreads / kScanBuckets;
template <int PER>
__global__ void __launch_bounds__(kScanThreads)
scan_buckets(const uint16_t* __restrict__ hist, BucketPlan plan, u32* __restrict__ prefix,
             u32* __restrict__ total, const PullCtx* __restrict__ ctx) {
  __shared__ u32 sums[kScanThreads / kWave][kScanBuckets];
  const u32 lane = lane_id(), wave = threadIdx.x / kWave, col = lane % kScanBuckets;
  const u32 n_buckets = plan.n_nat + ctx->n_heavy;
  const u32 b = blockIdx.x * kScanBuckets + col;
  const u32 t0 = (threadIdx.x / kScanBuckets) * PER;
  u32 v[PER];
#pragma unroll
  for (int k = 0; k < PER; ++k)
    v[k] = b < n_buckets && t0 + k < plan.n_tiles ? (u32)hist[(u64)(t0 + k) * plan.stride + b] : 0u;
  u32 mine = 0;
#pragma unroll
  for (int k = 0; k < PER; ++k) mine += v[k];
  // prefix over the wave's four groups, then over the waves
  u32 incl = mine;
  u32 up = (u32)__shfl_up((int)incl, kScanBuckets, kWave);
  if (lane >= kScanBuckets) incl += up;
  up = (u32)__shfl_up((int)incl, 2 * kScanBuckets, kWave);
  if (lane >= 2 * kScanBuckets) incl += up;
  if (lane >= kWave - kScanBuckets) sums[wave][col] = incl;
  __syncthreads();
  u32 run = incl - mine, all = 0;
#pragma unroll
  for (u32 w = 0; w < kScanThreads / kWave; ++w) {
    const u32 c = sums[w][col];
    if (w < wave) run += c;
    all += c;
  }
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    if (b < n_buckets && t0 + k < plan.n_tiles) prefix[(u64)(t0 + k) * plan.stride + b] = run;
    run += v[k];
  }
  if (threadIdx.x < kScanBuckets && b < n_buckets) total[b] = all;
}

// Where a tile lies beside more than kSparseBags bags per thread, nearly all of them empty, its occurrences' bags are
// found by a search among the bags' starts: going through them all is a round trip to memory per bag and thread
// (1000 occurrences in 10^6 bags: a step of 899 us, 63 with the search), the search one per halving, of all the
// thread's occurrences together.  Up to about a hundred bags per thread going through them is as fast or faster
// (0.2 M occurrences, 512 threads a tile, 32 bags per thread: 107 us and 117 with the search; 64: 119 and 123; 160: 164 and 143).
constexpr u32 kSparseBags = 96;

// Deals one tile per block out to the buckets.  What bounds it is the write requests of short runs (9.8 M
// occurrences, 2400 buckets: five occurrences a run, 40 bytes of keys, 20 of bags), which start and end
// in the middle of memory lines.  Neighbouring tiles' runs lie side by side, so tiles that follow each other
// go to the same XCD (xcd_piece), whose L2 then puts the pieces of a line together before it
// writes it: 143 -> 107 us (and 46 -> 37 us for spread, which reads the same runs).  The first tile's block also writes bucket_start[0 .. n_nat +
// max_heavy] and the heavy keys' entries of uniq and seg_off (bucket.hpp).  DIRECT: scan_buckets was left out, hist holds all there is.
template <int THREADS, int ITEMS, int MAX_BUCKETS, bool ORDERED, bool DIRECT>
__global__ void __launch_bounds__(THREADS)
bucket_scatter(const u64* __restrict__ keys, const uint16_t* __restrict__ id16, const i32* __restrict__ offsets,
               u32 n_bags, const u32* __restrict__ tile_bag, u32 n, BucketPlan plan, PullCtx* __restrict__ ctx,
               const uint16_t* __restrict__ hist, const u32* __restrict__ prefix, const u32* __restrict__ total,
               const HeavyRaw* __restrict__ heavy_raw, u32* __restrict__ bucket_start, u64* __restrict__ uniq, u32* __restrict__ seg_off,
               u64* __restrict__ keys_out, u32* __restrict__ bags_out, u32* __restrict__ code,
               uint16_t* __restrict__ from) {
  constexpr u32 kTile = THREADS * ITEMS;
  constexpr int kWaves = THREADS / kWave;
  constexpr int kPer = (MAX_BUCKETS + THREADS - 1) / THREADS;    // buckets a thread scans
  constexpr int kIdBits = 13;
  static_assert(MAX_BUCKETS <= 1 << kIdBits && kTile <= 1 << 16, "packed below");
  __shared__ u64 stage[kTile];
  __shared__ u32 first[kPer * THREADS];      // per bucket: count, then first staged place
  __shared__ u32 out[kPer * THREADS];        // per bucket: destination of a staged element - its staged place
  __shared__ u32 scratch[kWaves + 1];
  __shared__ u32 wave_last[kWaves];
  const u32 tid = threadIdx.x, wave = tid / kWave, lane = tid & (kWave - 1);
  const u32 tile = xcd_piece(blockIdx.x, plan.n_tiles), base = tile * kTile;
  const u32 tile_n = min(kTile, n - base);
  const u32 wave_first = wave * (kWave * ITEMS);        // element e of the tile: wave_first + r * 64 + lane
  const u32 n_buckets = plan.n_nat + ctx->n_heavy;

  // Everything the tile needs from memory is requested up front, what is needed last after what is needed
  // first (loads come back in order): bag starts, the buckets' counts, keys and bucket numbers.
  const u32 last_bag = n_bags - 1;
  u32 bag0 = 0, bag_end = 0, bag_lo = 0, bag_hi = 0;
  if (offsets) {
    bag0 = min(tile_bag[tile], last_bag);
    bag_end = tile + 1 < plan.n_tiles ? min(tile_bag[tile + 1], last_bag) : last_bag;
    if (bag0 + 1 + tid <= bag_end) { bag_lo = (u32)offsets[bag0 + 1 + tid]; bag_hi = (u32)offsets[bag0 + 2 + tid]; }
  }
  u32 in_bucket[kPer], in_earlier[kPer];       // of this thread's buckets: occurrences in all tiles, in the tiles before
#pragma unroll
  for (int q = 0; q < kPer; ++q) {
    const u32 b = kPer * tid + q;
    in_bucket[q] = in_earlier[q] = 0;
    if (!DIRECT && b < n_buckets) {
      in_bucket[q] = total[b];
      in_earlier[q] = prefix[(u64)tile * plan.stride + b];
    }
  }
  u64 key[ITEMS];
  u32 id[ITEMS];
#pragma unroll
  for (int r = 0; r < ITEMS; ++r) {
    const u32 i = min(base + wave_first + r * kWave + lane, n - 1);
    key[r] = keys[i];
    id[r] = id16[i];
  }
  if (DIRECT) {
#pragma unroll 8
    for (u32 t = 0; t < plan.n_tiles; ++t) {
#pragma unroll
      for (int q = 0; q < kPer; ++q) {
        const u32 b = kPer * tid + q;
        const u32 v = b < n_buckets ? (u32)hist[(u64)t * plan.stride + b] : 0u;
        in_bucket[q] += v;
        if (t < tile) in_earlier[q] += v;
      }
    }
  }
  // every non-empty bag that starts inside the tile marks its first occurrence
  u32* mark = reinterpret_cast<u32*>(stage);
  for (u32 e = tid; e < kTile; e += THREADS) mark[e] = 0;
#pragma unroll
  for (int q = 0; q < kPer; ++q) first[q * THREADS + tid] = 0;
  __syncthreads();
  const bool sparse = bag_end - bag0 > kSparseBags * THREADS;
  if (offsets && !sparse) {
    for (u32 b = bag0 + 1 + tid; b <= bag_end; b += THREADS) {
      if (bag_lo < bag_hi && bag_lo - base < kTile) mark[bag_lo - base] = b;      // (before the tile: the difference is huge)
      if (b + THREADS <= bag_end) { bag_lo = (u32)offsets[b + THREADS]; bag_hi = (u32)offsets[b + THREADS + 1]; }
    }
  }
  // ranks: the waves take turns, so that a bucket's counter is counted up in occurrence order
  u32 rank[ITEMS];
  const u64 lt = lanemask_lt();
  for (int w = 0; w < kWaves; ++w) {
    if (wave == (u32)w) {
#pragma unroll
      for (int r = 0; r < ITEMS; ++r)
        rank[r] = digit_rank<ORDERED, kIdBits>(&first[id[r]], id[r], wave_first + r * kWave + lane < tile_n, lt);
    }
    __syncthreads();
  }
  // bags: the bag of the last mark at or before the element, in this wave or an earlier one
  u32 bag[ITEMS];
  if (sparse) {
    // the last bag that starts at or before the element
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) bag[r] = bag0;
    for (u32 step = 1u << (31 - __clz((int)(bag_end - bag0))); step; step >>= 1) {
#pragma unroll
      for (int r = 0; r < ITEMS; ++r) {
        const u32 b = bag[r] + step;
        if (b <= bag_end && offsets[b] <= (i32)(base + wave_first + r * kWave + lane)) bag[r] = b;
      }
    }
  } else if (offsets) {
    u32 carry = 0;
    u32 m[ITEMS];
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) m[r] = mark[wave_first + r * kWave + lane];
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) {
      const u64 set = __ballot(m[r] != 0);
      const u64 upto = set & (lt | (1ull << lane));
      const u32 v = (u32)__shfl((int)m[r], upto ? 63 - __clzll((long long)upto) : 0, kWave);
      bag[r] = upto ? v : carry;                 // 0: none in this wave so far
      if (set) carry = (u32)__builtin_amdgcn_readlane((int)m[r], 63 - __clzll((long long)set));
    }
    if (lane == 0) wave_last[wave] = carry;
    __syncthreads();
    u32 before = bag0;
    for (u32 w = 0; w < wave; ++w) before = wave_last[w] ? wave_last[w] : before;
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) bag[r] = bag[r] ? bag[r] : before;
  } else {
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) bag[r] = base + wave_first + r * kWave + lane;
  }
  // per bucket (thread t: buckets kPer * t ...): its first staged place, its run's destination
  {
    u32 c[kPer], start[kPer], sum = 0, bucket_sum = 0, all;
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
      c[q] = first[kPer * tid + q];
      sum += c[q];
      bucket_sum += in_bucket[q];
    }
    u32 at = block_excl_sum<THREADS>(sum, scratch, &all);
    u32 at_all = block_excl_sum<THREADS>(bucket_sum, scratch, &all);
#pragma unroll
    for (int q = 0; q < kPer; ++q) { start[q] = at_all; at_all += in_bucket[q]; }
    if (tile == 0) {
      const u32 n_all = plan.n_nat + plan.max_heavy;
#pragma unroll
      for (int q = 0; q < kPer; ++q) {
        const u32 b = kPer * tid + q;
        if (b < n_all) bucket_start[b] = start[q];
        if (b >= plan.n_nat && in_bucket[q]) {       // a heavy key that occurs
          atomicAdd(&ctx->uniq_shard[b % kCountShards], 1u);
          uniq[start[q]] = heavy_raw->keys[b - plan.n_nat];
          seg_off[start[q]] = start[q];
          seg_off[start[q] + 1] = start[q] + in_bucket[q];
        }
      }
      if (tid == 0) bucket_start[n_all] = all;
    }
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
      const u32 b = kPer * tid + q;
      first[b] = at;
      out[b] = start[q] + in_earlier[q] - at;
      at += c[q];
    }
  }
  __syncthreads();
  // destinations
#pragma unroll
  for (int r = 0; r < ITEMS; ++r) {
    const u32 e = wave_first + r * kWave + lane;
    if (e < tile_n) {
      rank[r] += first[id[r]];                   // now the staged place
      const u32 dest = out[id[r]] + rank[r];
      const u32 c = id[r] >= plan.n_nat ? kHeavyCode | (id[r] - plan.n_nat) : dest;
      stage[rank[r]] = (u64)dest | ((u64)c << 32);
    }
  }
  __syncthreads();
  u32 dest[ITEMS];
  u32 heavy = 0;
#pragma unroll
  for (int k = 0; k < ITEMS; ++k) {
    const u32 j = k * THREADS + tid;
    dest[k] = 0;
    if (j < tile_n) {
      const u64 v = stage[j];
      dest[k] = (u32)v;
      code[base + j] = (u32)(v >> 32);
      if (v >> 63) heavy |= 1u << k;
    }
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < ITEMS; ++r)
    if (wave_first + r * kWave + lane < tile_n) stage[rank[r]] = key[r];
  __syncthreads();
#pragma unroll
  for (int k = 0; k < ITEMS; ++k) {
    const u32 j = k * THREADS + tid;
    if (j < tile_n && !(heavy >> k & 1u)) keys_out[dest[k]] = stage[j];
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < ITEMS; ++r) {
    const u32 e = wave_first + r * kWave + lane;
    if (e < tile_n) stage[rank[r]] = (u64)bag[r] | ((u64)e << 32);
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < ITEMS; ++k) {
    const u32 j = k * THREADS + tid;
    if (j < tile_n) {
      const u64 v = stage[j];
      bags_out[dest[k]] = (u32)v;
      from[base + j] = (uint16_t)(v >> 32);
    }
  }
}

// Brings a value per position (by_pos) or heavy bucket (by_heavy) back into occurrence order:
// out[i] = the value of the position or heavy bucket that occurrence i went to.  One tile per block.
template <int THREADS, int ITEMS>
__device__ __forceinline__ void spread_tile(const u32* __restrict__ code, const uint16_t* __restrict__ from, u32 n,
                                            u32 tile, const u32* __restrict__ by_pos,
                                            const u32* __restrict__ by_heavy, u32* __restrict__ out, u32* lds) {
  constexpr u32 kTile = THREADS * ITEMS;
  const u32 base = tile * kTile, tile_n = min(kTile, n - base);
  u32 c[ITEMS], at[ITEMS];
#pragma unroll
  for (int k = 0; k < ITEMS; ++k) {
    const u32 j = min(base + k * THREADS + threadIdx.x, n - 1);
    c[k] = code[j];
    at[k] = from[j];
  }
  u32 v[ITEMS];
#pragma unroll
  for (int k = 0; k < ITEMS; ++k) v[k] = c[k] & kHeavyCode ? by_heavy[c[k] & ~kHeavyCode] : by_pos[c[k]];
#pragma unroll
  for (int k = 0; k < ITEMS; ++k)
    if (k * THREADS + threadIdx.x < tile_n) lds[at[k]] = v[k];
  __syncthreads();
#pragma unroll
  for (int k = 0; k < ITEMS; ++k) {
    const u32 e = k * THREADS + threadIdx.x;
    if (e < tile_n) out[base + e] = lds[e];
  }
}

template <int THREADS, int ITEMS>
__global__ void __launch_bounds__(THREADS)
spread(const u32* __restrict__ code, const uint16_t* __restrict__ from, u32 n, const u32* __restrict__ by_pos,
       const u32* __restrict__ by_heavy, u32* __restrict__ out) {
  __shared__ u32 lds[THREADS * ITEMS];
  spread_tile<THREADS, ITEMS>(code, from, n, xcd_piece(blockIdx.x, gridDim.x), by_pos, by_heavy, out, lds);
}

}  // namespace hps
