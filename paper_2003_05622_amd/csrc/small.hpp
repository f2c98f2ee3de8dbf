// Small mini-batches: dedup, and in a pull or an accumulate the lookup too, in two launches.
//
// The bucket form (partition.hpp, bucket.hpp) takes four launches from the keys to the rows, and up to some ten thousand
// occurrences each of them is a chain of round trips to memory with nothing else to do: 7 to 8 us where the work
// itself is a fraction of one.  Here the natural buckets (2^log2_nat, parts of the keys' hashes, of 128 to 256
// occurrences each) have a block each, and nothing is dealt out beforehand:
//
//   small_ids     the bucket of every occurrence, one byte, and how many of each a tile holds;
//   small_group   a block goes through the bytes of ALL occurrences (16 KB to 64 KB, four to an instruction) and takes its own.
//                 A lane takes up to 64 consecutive occurrences, a wave its lanes'; the keys are entered into an LDS hash table and counted
//                 per wave, so that afterwards every wave can place its occurrences in their order without waiting for
//                 the others.  Then the distinct keys are looked up.
//
// 20 and 40 thousand occurrences (dim 8 and 100, a key with an eighth of them): 18 and 25 us in the two launches, 37 and 42 in the
// six (dedup, lookup, missing keys, rows by occurrence) they stand for.  What bounds it is the chain of round trips (ids, keys, slots) and,
// in the block with the most frequent key, that key's occurrences.  (Hashing all keys in every block instead, with no launch
// before it: 24 and 41 us, of which 8 and 12 are the hashes.)
//
// There are no buckets for frequent keys and there is no hint: a bucket may hold every occurrence there is.
// What is left, per occurrence, in one word of 16 bytes (a key with thousands of occurrences has one block write them all, in as
// many lines): the row (with the lookup), the place in the order grouped by key, the number of the key.  The bags of grouped
// positions (what the push reads) are put down by the pooling kernel, which knows every occurrence's
// bag; here they are only made harmless.
#pragma once

#include "common.hpp"
#include "bucket.hpp"
#include "table.hpp"

namespace hps {

constexpr u32 kSmallTile = 1024;           // occurrences and threads of a block of small_ids
constexpr int kSmallThreads = 1024;
constexpr u32 kSmallWaves = kSmallThreads / kWave;
constexpr u32 kSmallSlots = 1024;          // distinct keys of a bucket, at most (beyond: group_slow)
constexpr u32 kSmallSlotBits = 10;
constexpr u32 kSmallMean = 256;            // occurrences of a bucket on average, at most
constexpr u32 kSmallMinLog2 = 1, kSmallMaxLog2 = 8;
constexpr u32 kSmallBuckets = 1u << kSmallMaxLog2;
constexpr u32 kSmallPiece = 8 * kWave;     // occurrences of its bucket a wave lists at a time
// The block of a key that makes up much of the mini-batch places all its occurrences, 9 ns each on end, while the bucket form gives such a
// key a bucket that needs no grouping.  A bucket this long is reported, and the next mini-batches go by hash.  (us a step, dim 8,
// small form and by hash, one key with a share of 3, 12, 30, 50, 95 %: 20 K occurrences 23, 29, 39, 50, 77 and 39 to 41; 40 K 29, 34,
// 51, 74, 132 and 40 to 42; 65 K 34, 45, 68, 105, 196 and 43 to 47; 5 K 20, 23, 28, 34, 41 and 35 to 38.)
constexpr u32 kSmallLong = 7168;
__device__ __forceinline__ bool small_too_long(u32 cnt, u32 n) { return cnt > kSmallLong || (n >= 2048 && cnt > n / 4 * 3); }
constexpr u64 kSmallHistWords = (u64)(kSmallMax / kSmallTile) * kSmallBuckets;
static_assert(kSmallMax <= kSmallMean << kSmallMaxLog2, "a byte per occurrence");
static_assert(kSmallMax <= kSmallThreads * 64, "a bit per occurrence in a lane's mask");
static_assert(kSmallSlots == kSmallThreads && kSmallSlots == 1u << kSmallSlotBits, "a slot per thread");
static_assert(kSmallMax / kSmallTile * (kSmallBuckets / 16) == kSmallThreads, "sixteen of the counts per thread");

struct SmallArgs {
  const u64* keys;
  u32 n, log2_nat, n_tiles;
  u32 own_bags;          // every occurrence is its own bag (accumulate)
  PullCtx* ctx;
  uint8_t* ids;          // (padded to whole words)
  uint16_t* hist;        // [tile][kSmallBuckets]
  u32 *bucket_start, *count;
  u64* uniq;
  u32 *seg_off, *bags;
  uint4* places;         // per occurrence: row, grouped position, number of its key (null: own_bags)
  u64* dealt;            // group_slow: the bucket's keys, upos, its scratch
  u32* upos;
  SlowScratch slow;
  unsigned long long* report;      // host memory (or null): receives `serial`, the dedup's number, if the mini-batch does not suit this form
  u32 serial;
  // with the lookup
  u32* rows;
  Creation create;
  OftenLists often;
};

__global__ void __launch_bounds__(kSmallTile)
small_ids(TableView t, SmallArgs a) {
  __shared__ u32 h[kSmallBuckets];
  const u32 tid = threadIdx.x, i = blockIdx.x * kSmallTile + tid;
  const u64 key = a.keys[min(i, a.n - 1)];
  if (tid < kSmallBuckets) h[tid] = 0;
  if (blockIdx.x == 0) reset_ctx(a.ctx, a.n, (u32)kSmallForm + 1, 0);
  __syncthreads();
  if (i < a.n) {
    const u32 id = key_hash(key) >> (32 - a.log2_nat);
    a.ids[i] = (uint8_t)id;
    atomicAdd(&h[id], 1u);
    if (key == kEmptyKey) raise_error(t.st, kErrReserved);
  }
  __syncthreads();
  if (tid < kSmallBuckets) a.hist[blockIdx.x * kSmallBuckets + tid] = (uint16_t)h[tid];
}

constexpr u32 kSmallNewCap = 256;
struct SmallLds {
  union {
    struct {
      u64 key[kSmallSlots];        // kEmptyKey: free
      u64 ukey[kSmallSlots];       // distinct keys by their number; later their rows
      u32 place[kSmallSlots];      // where the group of the slot's key starts
      u32 uoff[kSmallSlots + 1];   // where the groups start, by the keys' numbers
      uint16_t num[kSmallSlots];   // number of the slot's key
      // per wave and slot (two to a word): occurrences; then those of the waves before, counted up as places are given out
      u32 cnt[kSmallWaves][kSmallSlots / 2];
    };
    SlowLds<kSmallThreads> slow;
  };
  LookupLds<kSmallNewCap, 64> look;
  u32 scratch[kSmallWaves + 1];
  u32 wave_cnt[kSmallWaves], low[kSmallWaves];
  u32 full;
  uint16_t list[kSmallWaves][kSmallPiece];
};

// Where a key's search starts in the LDS table (the leading bits of the hash name the bucket).
__device__ __forceinline__ u32 small_home(u64 key, u32 log2_nat) { return key_hash(key) << log2_nat >> (32 - kSmallSlotBits); }
// The slot of a key that is in the table.
__device__ __forceinline__ u32 small_find(const SmallLds& L, u64 key, u32 log2_nat) {
  u32 s = small_home(key, log2_nat);
  for (u32 step = 0; L.key[s] != key && step < kMaxProbes; ++step) s = (s + 1) & (kSmallSlots - 1);
  return s;
}
// The slot of a key, found or taken; kSmallSlots: none within kMaxProbes steps.
__device__ __forceinline__ u32 small_take(SmallLds& L, u64 key, u32 log2_nat) {
  u32 s = small_home(key, log2_nat);
  for (u32 step = 0; step < kMaxProbes; ++step) {
    u64 seen = L.key[s];
    if (seen == kEmptyKey) {
      seen = atomicCAS((unsigned long long*)&L.key[s], (unsigned long long)kEmptyKey, (unsigned long long)key);
      if (seen == kEmptyKey) return s;
    }
    if (seen == key) return s;
    s = (s + 1) & (kSmallSlots - 1);
  }
  return kSmallSlots;
}

// Lanes that hold the same key as the first lane in use, if they are many: a frequent key's occurrences.  That lane stands for
// all of them where they would queue up at one LDS word (a key with an eighth of 40 K occurrences: the kernel 34 us with every lane
// for itself).
struct SameKey {
  u64 lanes;             // 0: not many
  int first;
};
template <typename T>
__device__ __forceinline__ SameKey same_key(T v, bool on) {
  SameKey k;
  const u64 in_use = __ballot(on);
  k.first = in_use ? __ffsll((unsigned long long)in_use) - 1 : 0;
  k.lanes = __ballot(on && v == wave_lane(v, k.first));
  if (__popcll(k.lanes) < 16) k.lanes = 0;
  return k;
}

// A wave's occurrences of the bucket: bit b of a lane's mask says whether occurrence first + b is one.
struct SmallMine {
  u64 mask;
  u32 first;
};
// Lists those of them numbered p0 .. p0 + kSmallPiece - 1, in order; `before`: how many the lanes before have.  The whole
// wave, which alone reads the list (LDS serves its accesses in order: only the compiler has to keep them so).
__device__ __forceinline__ void small_list(uint16_t* list, const SmallMine& m, u32 before, u32 p0) {
  u32 at = before - p0;
  __builtin_amdgcn_wave_barrier();
  for (u64 b = m.mask; b; b &= b - 1, ++at)       // (before p0: `at` is huge)
    if (at < kSmallPiece) list[at] = (uint16_t)(m.first + (u32)__ffsll((unsigned long long)b) - 1);
  __builtin_amdgcn_wave_barrier();
}

__device__ __forceinline__ void small_report(const SmallArgs& a) {
  if (a.report) __hip_atomic_store(a.report, (unsigned long long)a.serial, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// LOOKUP: with the lookup.  ORDERED: how occurrences are ranked (sort.hpp: digit_rank).
template <bool LOOKUP, bool ORDERED>
__global__ void __launch_bounds__(kSmallThreads)
small_group(TableView t, SmallArgs a) {
  constexpr int K = kSmallPiece / kWave;
  __shared__ SmallLds L;
  const u32 tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane((int)(tid / kWave)), lane = tid & (kWave - 1), c = blockIdx.x;
  const u32 n = a.n;
  const bool look = LOOKUP && load_error(t.st) == 0;
  const bool tight = LOOKUP && is_tight(t, a.create, n);
  // which occurrences are the bucket's
  const u32 vecs = (n + kSmallThreads * 16 - 1) / (kSmallThreads * 16);       // a lane takes 16 * vecs in a row
  SmallMine mine;
  mine.mask = 0;
  mine.first = tid * 16 * vecs;
  const uint4* ids = reinterpret_cast<const uint4*>(a.ids) + tid * vecs;
  uint4 w[4];
#pragma unroll
  for (u32 q = 0; q < 4; ++q) w[q] = q < vecs && mine.first + 16 * q < n ? ids[q] : make_uint4(0, 0, 0, 0);
#pragma unroll
  for (u32 q = 0; q < 4; ++q) {
    const u32 word[4] = {w[q].x, w[q].y, w[q].z, w[q].w};
    u32 bits = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const u32 x = word[k] ^ c * 0x01010101u;
      const u32 z = ~((((x & 0x7F7F7F7Fu) + 0x7F7F7F7Fu) | x) | 0x7F7F7F7Fu) >> 7;       // one per zero byte
      bits |= ((z | z >> 7 | z >> 14 | z >> 21) & 15u) << (4 * k);
    }
    if (q < vecs) mine.mask |= (u64)bits << (16 * q);
  }
  const u32 here_n = mine.first < n ? min(n - mine.first, 16 * vecs) : 0u;
  if (here_n < 64) mine.mask &= (1ull << here_n) - 1;
  // how many come before them
  u32 low = 0;
  if (tid / 16 < a.n_tiles) {
    const uint4* h = reinterpret_cast<const uint4*>(a.hist + tid * 16);
    const uint4 v[2] = {h[0], h[1]};
    const u32 b0 = tid % 16 * 16;
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const u32 word[4] = {v[q].x, v[q].y, v[q].z, v[q].w};
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        if (b0 + 8 * q + 2 * k < c) low += word[k] & 0xFFFFu;
        if (b0 + 8 * q + 2 * k + 1 < c) low += word[k] >> 16;
      }
    }
  }
  low = wave_incl_sum(low);
  const u32 have = (u32)__popcll(mine.mask), incl = wave_incl_sum(have), lanes_before = incl - have;
  if (lane == kWave - 1) { L.low[wave] = low; L.wave_cnt[wave] = incl; }
  const u32 wave_n = (u32)__builtin_amdgcn_readlane((int)incl, kWave - 1);
  L.key[tid] = kEmptyKey;
#pragma unroll
  for (u32 w = 0; w < kSmallWaves / 2; ++w) (&L.cnt[0][0])[w * kSmallThreads + tid] = 0;
  if (tid == 0) { L.full = 0; L.look.clear(); }
  if (LOOKUP && c == 0 && tid == 0) { note_tight(t, a.create, tight); a.often.heavy_next->count = 0; }
  small_list(L.list[wave], mine, lanes_before, 0);
  __syncthreads();
  u32 cnt, start, wave_before;
  {
    const u32 of_lane = lane < kSmallWaves ? L.wave_cnt[lane] : 0u;
    const u32 upto = wave_incl_sum(of_lane);
    cnt = (u32)__builtin_amdgcn_readlane((int)upto, kWave - 1);
    wave_before = (u32)__builtin_amdgcn_readlane((int)(upto - of_lane), wave);
    start = (u32)__builtin_amdgcn_readlane((int)wave_incl_sum(lane < kSmallWaves ? L.low[lane] : 0u), kWave - 1);
  }
  if (tid == 0) {
    a.bucket_start[c] = start;
    if (c + 1 == gridDim.x) a.bucket_start[c + 1] = n;
    if (cnt == 0) {
      a.count[c] = 0;
      if (LOOKUP) a.often.med_span[c] = make_uint2(0u, 0u);
    }
    if (small_too_long(cnt, n)) small_report(a);
  }
  if (cnt == 0) return;

  // every key finds or takes a slot and is counted
  const u64 lt = lanemask_lt();
  u32 slot0[K];         // of the wave's first kSmallPiece occurrences
  for (u32 p0 = 0; p0 < wave_n; p0 += kSmallPiece) {
    if (p0) small_list(L.list[wave], mine, lanes_before, p0);
    u32 i[K];
    u64 key[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const bool on = p0 + k * kWave + lane < wave_n;
      i[k] = on ? L.list[wave][k * kWave + lane] : 0;
      key[k] = on ? a.keys[i[k]] : 0;
    }
#pragma unroll
    for (int k = 0; k < K; ++k) {
      if (p0 + k * kWave >= wave_n) continue;                // (the same for the whole wave)
      bool on = p0 + k * kWave + lane < wave_n;
      // (the reserved key marks free slots here)
      if (on && key[k] == kEmptyKey) { L.full = 1; on = false; }
      const SameKey same = same_key(key[k], on);
      const bool led = same.lanes >> lane & 1u, first = led && (int)lane == same.first;
      u32 s = 0;
      if (on && (!led || first)) {
        s = small_take(L, key[k], a.log2_nat);
        if (s == kSmallSlots) { L.full = 1; s = 0; }
        else atomicAdd(&L.cnt[wave][s / 2], (first ? (u32)__popcll(same.lanes) : 1u) << (s % 2 * 16));
      }
      const u32 theirs = wave_lane(s, same.first);
      if (p0 == 0) slot0[k] = led ? theirs : s;
    }
  }
  __syncthreads();
  const bool slow = L.full != 0;
  u32 u_count;
  if (slow) {
    __syncthreads();      // (L.full read by all)
    for (u32 p0 = 0; p0 < wave_n; p0 += kSmallPiece) {
      small_list(L.list[wave], mine, lanes_before, p0);
      for (u32 e = p0 + lane; e < min(wave_n, p0 + kSmallPiece); e += kWave) {
        const u32 i = L.list[wave][e - p0], j = start + wave_before + e;
        a.dealt[j] = a.keys[i];
        a.bags[j] = i;
      }
    }
    __syncthreads();
    group_slow<kSmallThreads>(a.dealt, start, start + cnt, a.uniq, a.seg_off, a.bags, a.upos, a.count, a.slow, a.ctx, L.slow);
    __syncthreads();
    u_count = a.count[c] & ~kSlowBucket;
    // (more than an eighth of the occurrences in such buckets: whichever block adds the last of them sees it)
    if (tid == 0 && (u64)__hip_atomic_load(&a.ctx->n_slow, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) * 8 > n) small_report(a);
  } else {
    // per slot: the key's number in the bucket, its group's start, and the occurrences in earlier waves
    u32 here = 0;
    uint16_t* mine16 = reinterpret_cast<uint16_t*>(&L.cnt[0][0]) + tid;
#pragma unroll
    for (u32 w = 0; w < kSmallWaves; ++w) {
      const u32 v = mine16[w * kSmallSlots];
      mine16[w * kSmallSlots] = (uint16_t)here;
      here += v;
    }
    u32 total;
    const u32 before = block_excl_sum<kSmallThreads>(here ? 1u << 20 | here : 0u, L.scratch, &total);
    static_assert(kSmallMax < 1u << 20 && kSmallSlots < 1u << 12, "packed into one word");
    if (here) {
      const u32 num = before >> 20, place = before & 0xFFFFFu;
      L.place[tid] = place;
      L.num[tid] = (uint16_t)num;
      L.ukey[num] = L.key[tid];
      L.uoff[num] = place;
      a.uniq[start + num] = L.key[tid];
      a.seg_off[start + num] = start + place;
    }
    u_count = total >> 20;
    if (tid == 0) {
      L.uoff[u_count] = cnt;
      a.seg_off[start + u_count] = start + cnt;
      a.count[c] = u_count;
      atomicAdd(&a.ctx->uniq_shard[c % kCountShards], u_count);
    }
    __syncthreads();
  }

  if (look) {
    const bool create_here = a.create.how != kCreateNone;      // (kCreateIfRoom takes the kernels apart)
    u32 missing = 0;
    for (u32 k0 = tid & ~3u; k0 < u_count; k0 += kSmallThreads) {
      const u32 k = k0 + tid % kLookupLanes, u = start + k;
      const bool on = k < u_count;
      u64 my_key = kEmptyKey;
      u32 len = 0;
      if (on) {
        my_key = slow ? a.uniq[u] : L.ukey[k];
        len = slow ? a.seg_off[u + 1] - a.seg_off[u] : L.uoff[k + 1] - L.uoff[k];
      }
      bool mine_new;
      const u32 row = lookup_key(t, my_key, create_here, min(a.create.new_cap, kSmallNewCap), L.look, &mine_new);
      if (!on) continue;
      a.rows[u] = row;
      if (!slow) L.ukey[k] = row;
      if (tight && mine_new) a.create.fresh[u] = a.create.stamp;
      if (row == kNoRow) ++missing;
      list_key(a.often, med_first(start), u, my_key, len, L.look);
    }
    if (missing) atomicAdd(&L.look.missing, missing);
    __syncthreads();
  }

  // per occurrence: its key's number and row, its place in the grouped order
  if (slow) {
    // (bags holds the occurrences in the grouped order; their keys' numbers follow from the groups' starts)
    for (u32 u = start + wave; u < start + u_count; u += kSmallWaves) {
      const u32 row = look ? a.rows[u] : kNoRow;
      for (u32 j = a.seg_off[u] + lane; j < a.seg_off[u + 1]; j += kWave) {
        if (a.own_bags) continue;
        a.places[a.bags[j]] = make_uint4(row, j, u, 0);
        a.bags[j] = 0;
      }
    }
  } else {
    for (u32 p0 = 0; p0 < wave_n; p0 += kSmallPiece) {
      if (wave_n > kSmallPiece) small_list(L.list[wave], mine, lanes_before, p0);
      u32 i[K], s[K];
#pragma unroll
      for (int k = 0; k < K; ++k) {
        const bool on = p0 + k * kWave + lane < wave_n;
        i[k] = on ? L.list[wave][k * kWave + lane] : 0;
        s[k] = !on ? 0 : p0 ? small_find(L, a.keys[i[k]], a.log2_nat) : slot0[k];
      }
#pragma unroll
      for (int k = 0; k < K; ++k) {
        if (p0 + k * kWave >= wave_n) continue;              // (the same for the whole wave)
        const bool on = p0 + k * kWave + lane < wave_n;
        const u32 half = s[k] % 2 * 16;
        u32 rank = 0;
        if (ORDERED) {
          const SameKey same = same_key(s[k], on);
          const bool led = same.lanes >> lane & 1u, first = led && (int)lane == same.first;
          if (on && (!led || first))
            rank = atomicAdd(&L.cnt[wave][s[k] / 2], (first ? (u32)__popcll(same.lanes) : 1u) << half) >> half & 0xFFFFu;
          const u32 theirs = wave_lane(rank, same.first);
          if (led) rank = theirs + (u32)__popcll(same.lanes & lt);
        } else {
          const u64 same = match_mask<(int)kSmallSlotBits>(s[k], on);
          const u32 before = (u32)__popcll(same & lt);
          if (on && before == 0) rank = atomicAdd(&L.cnt[wave][s[k] / 2], (u32)__popcll(same) << half) >> half & 0xFFFFu;
          rank = __shfl(rank, same ? __ffsll((unsigned long long)same) - 1 : 0, kWave) + before;
        }
        if (on) {
          const u32 num = L.num[s[k]], j = start + L.place[s[k]] + rank;
          a.bags[j] = a.own_bags ? i[k] : 0;
          if (!a.own_bags) a.places[i[k]] = make_uint4((u32)L.ukey[num], j, start + num, 0);
        }
      }
    }
  }
  if (look) {
    __syncthreads();
    end_lookup<kSmallThreads>(t, a.often, a.create, med_first(start), L.look);
  }
}

// A lookup of its own (hps_prepare): the rows into the occurrences' words.
__global__ void __launch_bounds__(256)
small_rows(const TableState* st, const u32* __restrict__ rows, u32 n, uint4* __restrict__ places) {
  if (load_error(st) != 0) return;
  for (u32 i = blockIdx.x * 256 + threadIdx.x; i < n; i += gridDim.x * 256) places[i].x = rows[places[i].z];
}
// hps_last_unique: the ranks of the occurrences' keys.
__global__ void __launch_bounds__(256)
small_ranks(const uint4* __restrict__ places, const u32* __restrict__ rank, u32 n, u32* __restrict__ out) {
  for (u32 i = blockIdx.x * 256 + threadIdx.x; i < n; i += gridDim.x * 256) out[i] = rank[places[i].z];
}

}  // namespace hps
