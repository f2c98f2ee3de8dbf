// Key dedup, bucket form, part 2: every bucket's occurrences are grouped by key inside one workgroup.
//
// After partition.hpp the keys and bags of a natural bucket (a few hundred to a few thousand occurrences) are
// contiguous, in occurrence order.  group_bucket enters the keys into a hash table in LDS and
// counts, so that for bucket c, which starts at position s,
//   uniq[s .. s+u)       its distinct keys, in no particular order (count[c] = u)
//   seg_off[s .. s+u]    where each key's group starts in bags, and the bucket's end
//   bags[s ..]           bags of the occurrences, grouped by key, occurrence order inside a group
//   upos[s ..]           per position as dealt out (partition.hpp: code): the key's number in the bucket
// Distinct keys are thus numbered by position, with gaps between the buckets: nothing has to be
// counted across buckets.  A heavy key's bucket is one group as it stands; its number is its start.
//
// Ascending unique keys and ranks (hps_last_unique) are worked out when they are asked for:
// where the buckets are in key order, order_uniques sorts each bucket's distinct keys (and the
// heavy keys that lie among them), emit_uniques adds up the buckets before it.  Of buckets by hash,
// gather_uniques collects the distinct keys, the plain form's radix passes sort them, and take_ranks
// notes every key's rank for emit_uniques.
//
// Which keys are heavy is a hint (partition.hpp).  Hot keys of click logs persist from batch to batch, so the hint is
// nearly always right; when it is not (a new hot key, keys bunched in a small part of their range: the next dedups then go
// by borders or by hash) some bucket exceeds what fits LDS and its workgroup orders it through global memory
// instead: slower, same result.
#pragma once

#include "common.hpp"
#include "sort.hpp"
#include "partition.hpp"

namespace hps {

constexpr int kGroupItems = 8;             // occurrences per thread: buckets of up to 8 * threads in LDS
constexpr u32 kSlowBucket = 0x80000000u;   // count[c]: the bucket was ordered the slow way (upos has 32-bit entries)
constexpr u32 kHeavyShare = 16384;         // heavy: more than n / kHeavyShare occurrences (and a bucket's eighth, hps.hip)

// ---- the slow way: a bucket too large for LDS ----------------------------------------
template <int THREADS>
struct SlowLds {
  u32 hist[kRadix];
  u32 bin[kRadix];
  u32 wave_cnt[THREADS / kWave][kRadix];
  u32 scratch[THREADS / kWave + 1];
  u32 flag;
};

// One stable pass of the pairs in [a, b) from (ksrc, psrc) to (kdst, pdst) by the
// digit at `shift`.  Returns false, having moved nothing, if all digits are equal.
template <int THREADS>
__device__ bool slow_radix_pass(const u64* ksrc, const u64* psrc, u64* kdst, u64* pdst, u32 a,
                                u32 b, int shift, SlowLds<THREADS>& L) {
  const u32 tid = threadIdx.x, wave = tid / kWave;
  const u64 lt = lanemask_lt();
  for (u32 d = tid; d < (u32)kRadix; d += THREADS) L.hist[d] = 0;
  for (int w = tid; w < THREADS / kWave * kRadix; w += THREADS) (&L.wave_cnt[0][0])[w] = 0;
  if (tid == 0) L.flag = 0;
  __syncthreads();
  for (u32 j = a + tid; j < b; j += THREADS) atomicAdd(&L.hist[key_digit(ksrc[j], shift)], 1u);
  __syncthreads();
  if (tid < (u32)kRadix && L.hist[tid] == b - a) L.flag = 1;
  u32 total;
  const u32 ex = block_excl_sum<THREADS>(tid < (u32)kRadix ? L.hist[tid] : 0, L.scratch, &total);
  if (L.flag) return false;        // written before the scan's barriers
  if (tid < (u32)kRadix) L.bin[tid] = a + ex;
  __syncthreads();
  for (u32 base = a; base < b; base += THREADS) {
    const u32 j = base + tid;
    const bool valid = j < b;
    const u64 key = valid ? ksrc[j] : 0;
    const u64 pay = valid ? psrc[j] : 0;
    const u32 d = key_digit(key, shift);
    u32 before, same;
    match_digit(d, valid, lt, &before, &same);
    const bool leader = valid && before == 0;
    if (leader) L.wave_cnt[wave][d] = same;
    __syncthreads();
    u32 dest = 0;
    if (valid) {
      dest = L.bin[d] + before;
      for (u32 w = 0; w < wave; ++w) dest += L.wave_cnt[w][d];
    }
    __syncthreads();
    if (leader) {
      atomicAdd(&L.bin[d], same);
      L.wave_cnt[wave][d] = 0;
    }
    if (valid) { kdst[dest] = key; pdst[dest] = pay; }
    __syncthreads();
  }
  return true;
}
static_assert(kRadix <= 256, "a digit per thread of the smallest block");

// Orders the pairs in [a, b) of (keys, pay) by full key, equal keys keeping their order.  The passes go
// back and forth between them and a second pair of arrays; afterwards keys / pay are the pair that holds the result.
template <int THREADS>
__device__ void slow_sort(u64*& keys, u64*& pay, u64* keys2, u64* pay2, u32 a, u32 b, SlowLds<THREADS>& L) {
  for (int shift = 0; shift < 64; shift += kRadixBits) {
    if (slow_radix_pass<THREADS>(keys, pay, keys2, pay2, a, b, shift, L)) {
      u64* x = keys; keys = keys2; keys2 = x;
      x = pay; pay = pay2; pay2 = x;
    }
    __syncthreads();
  }
}

// Scratch of the slow way beside the dealt-out keys, which nothing reads after it.
struct SlowScratch {
  u64 *pay, *keys2, *pay2;
};

template <int THREADS>
__device__ void group_slow(u64* keys, u32 start, u32 end, u64* __restrict__ uniq,
                           u32* __restrict__ seg_off, u32* __restrict__ bags, u32* __restrict__ upos,
                           u32* __restrict__ count, const SlowScratch& S, PullCtx* __restrict__ ctx, SlowLds<THREADS>& L) {
  const u32 tid = threadIdx.x;
  for (u32 p = start + tid; p < end; p += THREADS) S.pay[p] = (u64)bags[p] | ((u64)p << 32);
  __syncthreads();
  u64 *sk = keys, *sp = S.pay;
  slow_sort<THREADS>(sk, sp, S.keys2, S.pay2, start, end, L);
  if (tid == 0) {
    // For the host's choice of the next dedups' form: how much went this way, and how much
    // of that because ONE key fills the bucket (then the sorted bucket's middle element is
    // that key: count it) -- a key that turned frequent without warning, which the next
    // hint will list, and not keys that do not suit the buckets.
    const u64 mid_key = sk[start + (end - start) / 2];
    u32 lo = start, hi = end;
    while (lo < hi) { const u32 m = lo + (hi - lo) / 2; if (sk[m] < mid_key) lo = m + 1; else hi = m; }
    const u32 first = lo;
    hi = end;
    while (lo < hi) { const u32 m = lo + (hi - lo) / 2; if (sk[m] <= mid_key) lo = m + 1; else hi = m; }
    atomicAdd(&ctx->n_slow, end - start);
    if ((lo - first) * 2 >= end - start) atomicAdd(&ctx->n_slow_one_key, end - start);
  }
  u32 heads_before = 0;
  for (u32 base = start; base < end; base += THREADS) {
    const u32 j = base + tid;
    const bool valid = j < end;
    const u64 key = valid ? sk[j] : 0;
    const bool head = valid && (j == start || key != sk[j - 1]);
    u32 heads;
    const u32 before = block_excl_sum<THREADS>(head ? 1u : 0u, L.scratch, &heads);
    if (valid) {
      const u32 r = heads_before + before + (head ? 1u : 0u) - 1;
      const u64 pay = sp[j];
      if (head) { uniq[start + r] = key; seg_off[start + r] = j; }
      bags[j] = (u32)pay;
      upos[(u32)(pay >> 32)] = r;
    }
    heads_before += heads;
  }
  if (tid == 0) {
    seg_off[start + heads_before] = end;
    count[blockIdx.x] = heads_before | kSlowBucket;
    atomicAdd(&ctx->uniq_shard[blockIdx.x % kCountShards], heads_before);
  }
}

// ---- the usual way --------------------------------------------------------------------
constexpr u32 kMaxProbes = 512;            // a key that has looked at so many slots takes the slow way
template <int THREADS>
struct GroupLds {
  static constexpr u32 kCap = THREADS * kGroupItems;      // occurrences
  static constexpr u32 kSlots = kCap / 4 * 3;             // hash slots: distinct keys
  union {
    struct {
      u64 key[kSlots];       // kEmptyKey: free
      u32 cnt[kSlots];       // occurrences of the key; then number in the bucket << 16 | group's start
    };
    u32 bag[kCap];           // the bags, grouped, on their way out (when key[] is no longer needed)
    SlowLds<THREADS> slow;
  };
  u32 scratch[THREADS / kWave + 1];
  u32 full;          // the bucket goes the slow way after all
};

// One natural bucket per block: bucket_start[blockIdx.x] ...  keys / bags: as dealt out; bags are
// regrouped in place, keys may be overwritten.  ORDERED: how occurrences are ranked (sort.hpp: digit_rank).
template <int THREADS, bool ORDERED>
__global__ void __launch_bounds__(THREADS, 8)
group_bucket(u64* keys, const u32* __restrict__ bucket_start, u64* __restrict__ uniq,
             u32* __restrict__ seg_off, u32* __restrict__ bags, u32* __restrict__ upos, u32* __restrict__ count,
             SlowScratch S, PullCtx* __restrict__ ctx, TableState* __restrict__ st) {
  typedef GroupLds<THREADS> Lds;
  constexpr u32 kSlots = Lds::kSlots;
  constexpr int kPer = kSlots / THREADS;                  // slots a thread scans
  constexpr int kWaves = THREADS / kWave;
  __shared__ Lds L;
  const u32 tid = threadIdx.x, wave = tid / kWave, lane = tid & (kWave - 1);
  const u32 start = bucket_start[blockIdx.x], end = bucket_start[blockIdx.x + 1];
  const u32 cnt = end - start;
  if (cnt == 0) {
    if (tid == 0) count[blockIdx.x] = 0;
    return;
  }
  if (cnt > Lds::kCap) {
    for (u32 p = start + tid; p < end; p += THREADS) if (keys[p] == kEmptyKey) raise_error(st, kErrReserved);
    group_slow<THREADS>(keys, start, end, uniq, seg_off, bags, upos, count, S, ctx, L.slow);
    return;
  }
  // a wave owns `items` runs of 64 consecutive occurrences: element wave_first + r * 64 + lane
  const u32 items = (cnt + THREADS - 1) / THREADS;
  const u32 wave_first = wave * kWave * items;
  u32 slot[kGroupItems];
  {
    u64 key[kGroupItems];
#pragma unroll
    for (int r = 0; r < kGroupItems; ++r)
      key[r] = (u32)r < items ? keys[start + min(wave_first + r * kWave + lane, cnt - 1)] : 0;
    for (u32 s = tid; s < kSlots; s += THREADS) { L.key[s] = kEmptyKey; L.cnt[s] = 0; }
    if (tid == 0) L.full = 0;
    __syncthreads();
    // every key finds or takes a slot; all of a thread's keys take a step before the next step
    u32 open = 0;
#pragma unroll
    for (int r = 0; r < kGroupItems; ++r) {
      slot[r] = __umulhi(key_hash(key[r]), kSlots);
      if (wave_first + r * kWave + lane < cnt && (u32)r < items) {
        // (the reserved key marks free slots here: the slow way takes it as the key it is)
        if (key[r] == kEmptyKey) { raise_error(st, kErrReserved); L.full = 1; }
        else open |= 1u << r;
      }
    }
    for (u32 step = 0; open; ++step) {
      u64 seen[kGroupItems];
#pragma unroll
      for (int r = 0; r < kGroupItems; ++r) if (open >> r & 1u) seen[r] = L.key[slot[r]];
#pragma unroll
      for (int r = 0; r < kGroupItems; ++r)
        if ((open >> r & 1u) && seen[r] == kEmptyKey) {
          seen[r] = atomicCAS((unsigned long long*)&L.key[slot[r]], (unsigned long long)kEmptyKey,
                              (unsigned long long)key[r]);
          if (seen[r] == kEmptyKey) seen[r] = key[r];
        }
#pragma unroll
      for (int r = 0; r < kGroupItems; ++r) {
        if (!(open >> r & 1u)) continue;
        if (seen[r] == key[r]) open &= ~(1u << r);
        else slot[r] = slot[r] + 1 == kSlots ? 0 : slot[r] + 1;
      }
      if (step >= kMaxProbes) { L.full = 1; break; }     // (about) more distinct keys than slots
    }
  }
  __syncthreads();
  if (L.full) {
    __syncthreads();
    group_slow<THREADS>(keys, start, end, uniq, seg_off, bags, upos, count, S, ctx, L.slow);
    return;
  }
  // ranks among the occurrences of the same key: the waves take turns
  u32 rank[kGroupItems];
  const u64 lt = lanemask_lt();
  for (int w = 0; w < kWaves; ++w) {
    if (wave == (u32)w) {
#pragma unroll
      for (int r = 0; r < kGroupItems; ++r)
        if ((u32)r < items)
          rank[r] = digit_rank<ORDERED, 13>(&L.cnt[slot[r]], slot[r], wave_first + r * kWave + lane < cnt, lt);
    }
    __syncthreads();
  }
  // per slot: the key's number in the bucket (occupied slots before it) and its group's start
  u32 c[kPer], sum = 0, total;
#pragma unroll
  for (int q = 0; q < kPer; ++q) {
    c[q] = L.cnt[kPer * tid + q];
    sum += c[q] ? c[q] | 0x10000u : 0u;
  }
  u32 at = block_excl_sum<THREADS>(sum, L.scratch, &total);
#pragma unroll
  for (int q = 0; q < kPer; ++q) {
    if (!c[q]) continue;
    L.cnt[kPer * tid + q] = at;
    uniq[start + (at >> 16)] = L.key[kPer * tid + q];
    seg_off[start + (at >> 16)] = start + (at & 0xFFFFu);
    at += c[q] | 0x10000u;
  }
  if (tid == 0) {
    seg_off[start + (total >> 16)] = end;
    count[blockIdx.x] = total >> 16;
    atomicAdd(&ctx->uniq_shard[blockIdx.x % kCountShards], total >> 16);
  }
  u32 bag[kGroupItems];
#pragma unroll
  for (int r = 0; r < kGroupItems; ++r)
    bag[r] = (u32)r < items ? bags[start + min(wave_first + r * kWave + lane, cnt - 1)] : 0;
  __syncthreads();
  // (16-bit entries, packed from the bucket's first 32-bit word on)
  uint16_t* up = reinterpret_cast<uint16_t*>(upos + start);
#pragma unroll
  for (int r = 0; r < kGroupItems; ++r) {
    const u32 e = wave_first + r * kWave + lane;
    if (e < cnt && (u32)r < items) {
      const u32 v = L.cnt[slot[r]];
      up[e] = (uint16_t)(v >> 16);
      rank[r] += v & 0xFFFFu;                  // now the place in the grouped order
    }
  }
  __syncthreads();      // bag[] shares its memory with key[] and cnt[]
#pragma unroll
  for (int r = 0; r < kGroupItems; ++r)
    if (wave_first + r * kWave + lane < cnt && (u32)r < items) L.bag[rank[r]] = bag[r];
  __syncthreads();
  for (u32 j = tid; j < cnt; j += THREADS) bags[start + j] = L.bag[j];
}

// The number in its bucket of the key at position start + e (of a bucket with this count word).
__device__ __forceinline__ u32 upos_at(const u32* upos, u32 start, u32 e, u32 count_word) {
  return count_word & kSlowBucket ? upos[start + e] : (u32)reinterpret_cast<const uint16_t*>(upos + start)[e];
}

// ---- ascending unique keys and ranks, on request ----------------------------------------
constexpr int kOrderThreads = 1024;
// order_uniques by the threads of the buckets' workgroups: threads of its own, keys it holds in LDS
constexpr int order_threads(int group) { return group == 256 ? 512 : 1024; }
constexpr u32 order_cap(int group) { return 8 * order_threads(group); }
constexpr u32 order_max_heavy(int group) { return group == 256 ? 1023 : kMaxHeavy; }
static_assert(GroupLds<256>::kSlots + order_max_heavy(256) <= order_cap(256) &&
                  GroupLds<1024>::kSlots + order_max_heavy(1024) <= order_cap(1024), "a bucket's distinct keys and all heavy keys");

// Bucket c: local_rank[u] = rank of key number u among the bucket's distinct keys and the heavy keys
// that lie in the bucket's part of the key range; bucket_total[c] = how many those are.
//
// The keys are dealt into kOrderCells cells in key order (by their place between the smallest and the
// largest of them), and a key's rank is its cell's start plus the smaller keys of the cell: hashed
// keys share a cell with one or two others.  Where a cell holds many (keys bunched inside the bucket),
// a bitonic network sorts them.  9.8 M occurrences, 2.8 M distinct keys: the whole of hps_last_unique
// takes 175 us; with the network throughout, 485.  Small buckets (GROUP: threads of their workgroups) are ordered by
// half the threads, so that three blocks fit a CU and all are under way at once: 0.3 M occurrences, the call 40 us with blocks
// of 1024 for 8192 keys, 25 with these.
constexpr u32 kOrderCellMax = 32;
template <int GROUP>
__global__ void __launch_bounds__(order_threads(GROUP))
order_uniques(const u64* __restrict__ uniq, const u32* __restrict__ bucket_start, const u32* __restrict__ count,
              u32 n_nat, const u64* __restrict__ border, const PullCtx* __restrict__ ctx,
              u32* __restrict__ local_rank, u32* __restrict__ bucket_total) {
  constexpr int kThreads = order_threads(GROUP), kPer = order_cap(GROUP) / kThreads, kWaves = kThreads / kWave;
  constexpr u32 kOrderCells = (GROUP == 256 ? 2 : 4) * kThreads;
  __shared__ u64 key[order_cap(GROUP)];
  __shared__ u32 num[order_cap(GROUP)];
  __shared__ u32 cell[kOrderCells + 1];
  __shared__ u64 s_lo[kWaves], s_hi[kWaves];
  __shared__ u32 scratch[kWaves + 1];
  __shared__ u32 s_n, s_crowded;
  const u32 tid = threadIdx.x, c = blockIdx.x;
  const u32 start = bucket_start[c], word = count[c], u = word & ~kSlowBucket;
  const bool slow = (word & kSlowBucket) != 0;       // already in order, and maybe too many for LDS
  const u32 n_heavy = ctx->n_heavy;
  const KeyRange range = ctx->range;
  if (tid == 0) { s_n = slow ? 0 : u; s_crowded = 0; }
  if (!slow) for (u32 i = tid; i < u; i += kThreads) { key[i] = uniq[start + i]; num[i] = start + i; }
  __syncthreads();
  for (u32 h = tid; h < n_heavy; h += kThreads) {
    const u32 at = bucket_start[n_nat + h];
    if (bucket_start[n_nat + h + 1] == at) continue;
    const u64 k = uniq[at];
    if (!in_bucket(k, c, range, border, n_nat)) continue;
    const u32 i = atomicAdd(&s_n, 1u);
    key[i] = k;
    num[i] = at;
  }
  for (u32 i = tid; i <= kOrderCells; i += kThreads) cell[i] = 0;
  __syncthreads();
  const u32 n = s_n;
  // this thread's keys, and the ends of all of them
  u64 mine[kPer];
  u32 mine_num[kPer], place[kPer];
  u64 lo = ~0ull, hi = 0;
#pragma unroll
  for (int q = 0; q < kPer; ++q) {
    const u32 i = q * kThreads + tid;
    mine[q] = i < n ? key[i] : 0;
    mine_num[q] = i < n ? num[i] : 0;
    if (i < n) { lo = min(lo, mine[q]); hi = max(hi, mine[q]); }
  }
#pragma unroll
  for (int d = 1; d < kWave; d <<= 1) {
    lo = min(lo, (u64)__shfl_xor((unsigned long long)lo, d, kWave));
    hi = max(hi, (u64)__shfl_xor((unsigned long long)hi, d, kWave));
  }
  if (lane_id() == 0) { s_lo[tid / kWave] = lo; s_hi[tid / kWave] = hi; }
  __syncthreads();
  sampled_ends<kThreads>(s_lo, s_hi, &lo, &hi);
  KeyRange r;
  r.lo = lo; r.span = hi - lo; r.base = 0;
  r.pre = r.span >> 32 ? 32 - __clzll((long long)r.span) : 0;
  r.direct = r.span < kOrderCells;
  r.mult = r.direct ? 0u : (u32)(((u64)kOrderCells << 32) / ((r.span >> r.pre) + 1));
#pragma unroll
  for (int q = 0; q < kPer; ++q)
    if (q * kThreads + tid < n) {
      place[q] = atomicAdd(&cell[bucket_of(mine[q], r)], 1u);
      if (place[q] >= kOrderCellMax) s_crowded = 1;
    }
  __syncthreads();
  if (!s_crowded) {
    constexpr int kCells = kOrderCells / kThreads;
    u32 v[kCells], sum = 0, total;
#pragma unroll
    for (int q = 0; q < kCells; ++q) { v[q] = cell[kCells * tid + q]; sum += v[q]; }
    u32 at = block_excl_sum<kThreads>(sum, scratch, &total);
#pragma unroll
    for (int q = 0; q < kCells; ++q) { cell[kCells * tid + q] = at; at += v[q]; }
    if (tid == 0) cell[kOrderCells] = total;
    __syncthreads();
#pragma unroll
    for (int q = 0; q < kPer; ++q)
      if (q * kThreads + tid < n) key[cell[bucket_of(mine[q], r)] + place[q]] = mine[q];
    __syncthreads();
#pragma unroll
    for (int q = 0; q < kPer; ++q)
      if (q * kThreads + tid < n) {
        const u32 k = bucket_of(mine[q], r), end = cell[k + 1];
        u32 rank = cell[k];
        for (u32 i = rank; i < end; ++i) rank += key[i] < mine[q] ? 1u : 0u;
        place[q] = rank;
      }
    __syncthreads();
    if (!slow) {
#pragma unroll
      for (int q = 0; q < kPer; ++q)
        if (q * kThreads + tid < n) local_rank[mine_num[q]] = place[q];
    } else {          // the merge below wants the heavy keys in order
#pragma unroll
      for (int q = 0; q < kPer; ++q)
        if (q * kThreads + tid < n) { key[place[q]] = mine[q]; num[place[q]] = mine_num[q]; }
      __syncthreads();
    }
  } else {
    u32 size = 2;
    while (size < n) size <<= 1;
    // (the reserved key is never among them: it goes the slow way and is in no list of heavy keys)
    for (u32 i = n + tid; i < size; i += kThreads) { key[i] = ~0ull; num[i] = ~0u; }
    for (u32 k = 2; k <= size; k <<= 1) {
      for (u32 j = k >> 1; j > 0; j >>= 1) {
        __syncthreads();
        for (u32 i = tid; i < size; i += kThreads) {
          const u32 partner = i ^ j;
          if (partner > i && (key[i] > key[partner]) == ((i & k) == 0)) {
            const u64 x = key[i]; key[i] = key[partner]; key[partner] = x;
            const u32 y = num[i]; num[i] = num[partner]; num[partner] = y;
          }
        }
      }
    }
    __syncthreads();
    if (!slow) for (u32 i = tid; i < n; i += kThreads) local_rank[num[i]] = i;
  }
  if (slow) {
    // two ordered lists: the bucket's own keys (global memory) and the heavy ones among them (LDS)
    for (u32 i = tid; i < u; i += kThreads) {
      const u64 k = uniq[start + i];
      u32 a = 0, b = n;
      while (a < b) { const u32 m = (a + b) / 2; if (key[m] < k) a = m + 1; else b = m; }
      local_rank[start + i] = i + a;
    }
    for (u32 i = tid; i < n; i += kThreads) {
      const u64 k = key[i];
      u32 a = 0, b = u;
      while (a < b) { const u32 m = (a + b) / 2; if (uniq[start + m] < k) a = m + 1; else b = m; }
      local_rank[num[i]] = i + a;
    }
  }
  if (tid == 0) bucket_total[c] = n + (slow ? u : 0);
}

// Buckets by hash: all distinct keys side by side, with the positions they are numbered by; *n_out = how many.  The block
// behind the natural buckets' takes the heavy keys.
__global__ void __launch_bounds__(kOrderThreads)
gather_uniques(const u64* __restrict__ uniq, const u32* __restrict__ bucket_start, const u32* __restrict__ count,
               u32 n_nat, const PullCtx* __restrict__ ctx, u64* __restrict__ keys_out, u32* __restrict__ pos_out, u32* __restrict__ n_out) {
  __shared__ u32 scratch[kOrderThreads / kWave + 1];
  const u32 tid = threadIdx.x, c = blockIdx.x;
  u32 mine = 0, base;
  for (u32 i = tid; i < c; i += kOrderThreads) mine += count[i] & ~kSlowBucket;
  (void)block_excl_sum<kOrderThreads>(mine, scratch, &base);
  if (c < n_nat) {
    const u32 start = bucket_start[c], u = count[c] & ~kSlowBucket;
    for (u32 i = tid; i < u; i += kOrderThreads) { keys_out[base + i] = uniq[start + i]; pos_out[base + i] = start + i; }
    return;
  }
  const u32 n_heavy = ctx->n_heavy;
  for (u32 h0 = 0; h0 < n_heavy; h0 += kOrderThreads) {
    const u32 h = h0 + tid;
    const u32 at = h < n_heavy ? bucket_start[n_nat + h] : 0;
    const bool on = h < n_heavy && bucket_start[n_nat + h + 1] != at;
    u32 all;
    const u32 before = block_excl_sum<kOrderThreads>(on ? 1u : 0u, scratch, &all);
    if (on) { keys_out[base + before] = uniq[at]; pos_out[base + before] = at; }
    base += all;
  }
  if (tid == 0) *n_out = base;
}

// From the sorted distinct keys (payload: position in the upper half): the keys, and every key's rank by its position.
__global__ void __launch_bounds__(kOrderThreads)
take_ranks(const u64* __restrict__ keys, const u64* __restrict__ pay, const u32* __restrict__ n_dev, const PullCtx* __restrict__ sort_ctx,
           TableState* __restrict__ st, u64* __restrict__ uniq_out, u32* __restrict__ local_rank) {
  if (sort_ctx->sort_error) {      // (never expected: a wait of the passes gave up)
    if (threadIdx.x == 0) raise_error(st, kErrInternal);
    return;
  }
  const u32 n = *n_dev;
  for (u32 j = blockIdx.x * kOrderThreads + threadIdx.x; j < n; j += gridDim.x * kOrderThreads) {
    local_rank[(u32)(pay[j] >> 32)] = j;
    if (uniq_out) uniq_out[j] = keys[j];
  }
}

// uniq_out (may be null): the keys in ascending order; rank_by_pos / rank_by_heavy (null: not
// wanted): every position's and heavy bucket's rank, for spread().  bucket_total == null: local_rank holds the
// final ranks already (buckets by hash).
__global__ void __launch_bounds__(kOrderThreads)
emit_uniques(const u64* __restrict__ uniq, const u32* __restrict__ bucket_start, const u32* __restrict__ count,
             const u32* __restrict__ upos, u32 n_nat, const u64* __restrict__ border, const PullCtx* __restrict__ ctx,
             const u32* __restrict__ local_rank, const u32* __restrict__ bucket_total, u64* __restrict__ uniq_out,
             u32* __restrict__ rank_by_pos, u32* __restrict__ rank_by_heavy) {
  __shared__ u32 scratch[kOrderThreads / kWave + 1];
  const u32 tid = threadIdx.x, c = blockIdx.x;
  const u32 start = bucket_start[c], end = bucket_start[c + 1], word = count[c], u = word & ~kSlowBucket;
  u32 mine = 0, base = 0;
  if (bucket_total) {
    for (u32 i = tid; i < c; i += kOrderThreads) mine += bucket_total[i];
    (void)block_excl_sum<kOrderThreads>(mine, scratch, &base);
  }
  if (uniq_out)
    for (u32 i = tid; i < u; i += kOrderThreads) uniq_out[base + local_rank[start + i]] = uniq[start + i];
  if (rank_by_pos)
    for (u32 e = tid; e < end - start; e += kOrderThreads)
      rank_by_pos[start + e] = base + local_rank[start + upos_at(upos, start, e, word)];
  const u32 n_heavy = ctx->n_heavy;
  const KeyRange range = ctx->range;
  for (u32 h = tid; h < n_heavy; h += kOrderThreads) {
    const u32 at = bucket_start[n_nat + h];
    if (bucket_start[n_nat + h + 1] == at) continue;
    const u64 k = uniq[at];
    if (bucket_total ? !in_bucket(k, c, range, border, n_nat) : h % n_nat != c) continue;
    const u32 rank = base + local_rank[at];
    if (uniq_out) uniq_out[rank] = k;
    if (rank_by_heavy) rank_by_heavy[h] = rank;
  }
}

}  // namespace hps
