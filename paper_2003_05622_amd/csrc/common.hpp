// Shared device-side definitions of the HBM-PS pull/push kernels (gfx950, wave64).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace hps {

typedef uint32_t u32;
typedef uint64_t u64;
typedef int32_t i32;

constexpr u64 kEmptyKey = ~u64(0);   // marks a free slot; never a legal key
constexpr u32 kNoRow = ~u32(0);      // "this key has no row" (lookup miss / table full)
constexpr int kWave = 64;
constexpr int kSlotsPerLine = 8;     // 8 keys of 8 bytes = one 64-byte line, probed by 8 lanes

// Device-side status values mirror hps_status.
constexpr int kErrFull = -2;
constexpr int kErrReserved = -3;
constexpr int kErrInternal = -5;   // HPS_EDEVICE: a dedup's cross-workgroup wait gave up (never expected)

// Plain form of the dedup: places where different keys agree in all sorted bits that
// fix_mixed_runs can note; beyond that one workgroup puts the whole array in order.
constexpr u32 kMaxEvidence = 1024;

constexpr int kCountShards = 64;   // counters that many blocks add to are spread over this many words

// Lives in the table's storage for the table's whole life.
struct TableState {
  unsigned long long size;      // keys stored
  unsigned long long inserted;  // keys created by the last pull / insert call
  int error;                    // sticky: 0 or a negative status
  int absent;                   // distinct keys the last accumulate did not find
  unsigned long long dump_count;  // rows seen by all dumps since the creation (the host knows how many before the running one)
  // Keys the running lookup found missing and left / rows the running insert created, spread
  // over shards so that blocks do not all hit one address.
  u32 miss_shard[kCountShards];
  u32 made_shard[kCountShards];
  // Rows the running pull has created, in the set pulls take in turn (the end of a pull clears the other
  // one for the next); size before it, and whether it might have overfilled the table (table.hpp: end_pull).
  u32 pull_made[2][kCountShards];
  unsigned long long size_before;
  u32 tight;
  u32 pad2;
  u32 pad;
  u32 probe_bad;                // result word of probe_lane_order (written once, at creation)
  // hps_probe_lengths: lines looked at to find each stored key, summed / the most for one key
  unsigned long long probe_sum;
  unsigned long long probe_max;
};

// Where a mini-batch's keys lie, estimated from a sample of them by the dedup's first kernel.
// The dedup orders keys by rel = clamp(key - lo, 0, span) instead of by the key itself, which
// is the same order, but raw ids that all share their leading bits spread over the
// buckets / digits like hashed keys do (sort.hpp: range_rel; partition.hpp: bucket_of).
struct KeyRange {
  u64 lo;
  u64 span;      // largest rel
  u32 mult;      // bucket form: bucket = ((rel >> pre) * mult) >> 32
  u32 pre;       //   (rel >> pre fits 32 bits)
  u32 direct;    // bucket form: span is below the number of buckets, bucket = rel
  u32 base;      // plain form: the sorted digits start at this bit of rel
};

// Lives in the workspace; describes the outstanding pull.
struct PullCtx {
  u32 n_unique;        // plain form: number of distinct keys (bucket form: the sum of uniq_shard)
  u32 n_long;          // keys the push handles chunk by chunk
  u32 n_slow;          // bucket form: occurrences in buckets that were grouped through global memory
  u32 n_chunk_items;   // (key, chunk) work items of the push
  u32 n_evidence;      // plain form: sorted positions where a run of equal sorted bits mixes keys
  u32 sort_error;      // set if a look-back wait gave up (never expected)
  u32 n_total;         // occurrences of this dedup
  u32 by_id;           // 0: this dedup took the plain form, else 1 + its form (form.hpp)
  u32 n_heavy;         // bucket form: frequent keys with a bucket of their own
  u32 pad[2];
  u32 n_slow_one_key;  // ... of n_slow, in buckets that one key fills at least half of
  KeyRange range;      // plain form: for the kernels after the first
  u32 uniq_shard[kCountShards];   // bucket form: distinct keys, spread over shards
};

// Keys that make up a large share of a mini-batch ("heavy" keys): the bucket form gives each
// of them a bucket of its own.  Which ones they are is a hint, taken from an earlier lookup,
// which lists the keys it sees often in arrival order; readers cope with any content.
// Lookup s (s = 1, 2, ...) fills raw[s % 3] and empties raw[(s + 1) % 3] for the next one.  A dedup
// issued when s lookups have been issued reads raw[(s - 1) % 3]: lookup s - 1 is certainly
// complete (the dedup waits for the push that released its context, which is push s - 1 or a
// later one) and nobody appends to that list again before lookup s + 2, which comes after this
// dedup's pull.  So every block of a dedup sees the same, unchanging list, whatever
// streams the calls were issued on.
constexpr int kMaxHeavy = 2047;
struct HeavyRaw {
  u32 count;
  u32 pad;
  u64 keys[kMaxHeavy + 1];
};
constexpr u32 kHeavyRing = 3;
struct HeavyRing {
  HeavyRaw raw[kHeavyRing];
};

// SplitMix64 output function for state x (Steele, Lea, Flood 2014).  The row
// initialiser is defined on top of it.
__device__ __forceinline__ u64 mix64(u64 x) {
  u64 z = x + 0x9E3779B97F4A7C15ull;
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}

// Slot hash: the 64-bit finaliser of MurmurHash3 (Appleby), so that the table
// does not rely on keys arriving well mixed.
__device__ __forceinline__ u64 slot_hash(u64 k) {
  k ^= k >> 33;
  k *= 0xFF51AFD7ED558CCDull;
  k ^= k >> 33;
  k *= 0xC4CEB9FE1A85EC53ull;
  k ^= k >> 33;
  return k;
}

// Element j of key's initial row: uniform on [-a, a) from 24 random bits, as a
// rounded product followed by a rounded difference.  The two must never be fused
// into one multiply-add (that would round once and change the bits), so
// contraction is switched off for this function.
__device__ __forceinline__ float init_weight(u64 base, u32 j, float a) {
#pragma clang fp contract(off)
  const u64 r = mix64(base + j);
  const float u = (float)(u32)(r >> 40) * 0x1.0p-24f;   // exact
  const float scaled = u * (a * 2.0f);
  return scaled - a;
}

__device__ __forceinline__ u32 lane_id() { return threadIdx.x & (kWave - 1); }

// The value a lane of the wave holds (`lane` the same in all of them).
__device__ __forceinline__ u32 wave_lane(u32 v, int lane) { return (u32)__builtin_amdgcn_readlane((int)v, lane); }
__device__ __forceinline__ u64 wave_lane(u64 v, int lane) { return wave_lane((u32)v, lane) | (u64)wave_lane((u32)(v >> 32), lane) << 32; }

__device__ __forceinline__ u64 lanemask_lt() {
  const u32 l = lane_id();
  return l == 0 ? 0ull : (~0ull >> (64 - l));
}

// One step of a wave-wide scan or reduction in the data-parallel-primitive form: lane l receives
// lane l - 1, - 2, - 4 or - 8 of its row of 16 (CTRL 0x110 + distance), or the last lane of the row
// / of the half before (0x142, 0x143, masked to the rows that need it); zero where there is none.
template <int CTRL, int ROWS>
__device__ __forceinline__ u32 dpp_or_zero(u32 v) {
  return (u32)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROWS, 0xF, false);
}

// The value lane k (a constant after unrolling, below eight) of each group of LPR lanes holds, in all its lanes: full-rate moves.
template <int LPR>
__device__ __forceinline__ u32 group_lane(u32 v, int k) {
  static_assert(LPR == 1 || LPR == 2 || LPR == 4 || LPR == 8 || LPR == 16 || LPR == 32 || LPR == 64, "");
  if (LPR == 1) return v;
  if (LPR == 2) return (u32)(k == 0 ? __builtin_amdgcn_mov_dpp((int)v, 0xA0, 0xF, 0xF, true) : __builtin_amdgcn_mov_dpp((int)v, 0xF5, 0xF, 0xF, true));
#define HPS_LANE(K)                                                                                                           \
  case K:                                                                                                                     \
    if (LPR == 4) return (u32)__builtin_amdgcn_mov_dpp((int)v, (K & 3) * 0x55, 0xF, 0xF, true);             /* within four */  \
    if (LPR == 16) return (u32)__builtin_amdgcn_mov_dpp((int)v, 0x150 + K, 0xF, 0xF, true);                 /* within 16 */    \
    if (LPR == 8)                                                                                           /* half by half */ \
      return (u32)__builtin_amdgcn_update_dpp(__builtin_amdgcn_update_dpp(0, (int)v, 0x150 + K, 0xF, 0x3, false), (int)v, 0x158 + K, 0xF, 0xC, false); \
    break;
  switch (k) { HPS_LANE(0) HPS_LANE(1) HPS_LANE(2) HPS_LANE(3) HPS_LANE(4) HPS_LANE(5) HPS_LANE(6) HPS_LANE(7) }
#undef HPS_LANE
  const u32 low = (u32)__builtin_amdgcn_readlane((int)v, k);
  if (LPR == 64) return low;
  const u32 high = (u32)__builtin_amdgcn_readlane((int)v, 32 + k);
  return lane_id() < 32 ? low : high;
}

// Eight items a group of LPR lanes has in flight, each known to one lane (item j to lane j % LPR, as its number j / LPR): where
// they lie, as byte offsets.
constexpr u64 kNowhere = ~0ull;
template <int LPR>
struct GroupOffsets {
  static constexpr int kOwn = LPR < 8 ? 8 / LPR : 1;
  u64 own[kOwn];
  // The offset of item k; false: there is none.
  __device__ __forceinline__ bool get(int k, u64* offset) const {
    const u64 v = own[k / LPR];
    const u32 high = group_lane<LPR>((u32)(v >> 32), k % LPR);
    *offset = (u64)high << 32 | group_lane<LPR>((u32)v, k % LPR);
    return high != 0xFFFFFFFFu;
  }
};

// Inclusive sum over the 64 lanes of a wave.
__device__ __forceinline__ u32 wave_incl_sum(u32 v) {
  v += dpp_or_zero<0x111, 0xF>(v);
  v += dpp_or_zero<0x112, 0xF>(v);
  v += dpp_or_zero<0x114, 0xF>(v);
  v += dpp_or_zero<0x118, 0xF>(v);
  v += dpp_or_zero<0x142, 0xA>(v);
  v += dpp_or_zero<0x143, 0xC>(v);
  return v;
}

// Exclusive sum over a block of THREADS threads (multiple of 64, at most 1024).
// `scratch` needs THREADS/64 words of LDS.  Returns the exclusive prefix of v
// and the block total in *total.  Contains __syncthreads().
template <int THREADS>
__device__ __forceinline__ u32 block_excl_sum(u32 v, u32* scratch, u32* total) {
  constexpr int NW = THREADS / kWave;
  const u32 incl = wave_incl_sum(v);
  const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
  __syncthreads();   // scratch may still be in use by a previous call
  if (lane_id() == kWave - 1) scratch[w] = incl;
  __syncthreads();
  // every wave adds up the waves' sums for itself
  const u32 c = lane_id() < (u32)NW ? scratch[lane_id()] : 0u;
  const u32 upto = wave_incl_sum(c);
  *total = (u32)__builtin_amdgcn_readlane((int)upto, kWave - 1);
  const u32 before = (u32)__builtin_amdgcn_readlane((int)upto, w) - (u32)__builtin_amdgcn_readlane((int)c, w);
  return before + incl - v;
}

// Which of n consecutive pieces of work block b of n takes, so that neighbours stay together: the GPU
// deals blocks out over its 8 XCDs in turn, each with an L2 of its own, so block b takes the
// (b / 8)-th piece of part b % 8.
constexpr u32 kXcds = 8;
__device__ __forceinline__ u32 xcd_piece(u32 b, u32 n) {
  const u32 part = b % kXcds;
  return part * (n / kXcds) + min(part, n % kXcds) + b / kXcds;
}

__device__ __forceinline__ int load_error(const TableState* st) {
  return __hip_atomic_load(&st->error, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ void raise_error(TableState* st, int code) {
  atomicCAS(&st->error, 0, code);
}

}  // namespace hps
