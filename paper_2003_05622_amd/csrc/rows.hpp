// The entry points that move whole rows: get and insert (by key), dump (by slot).
//
// What bounds them is the number of random lines they ask for: per key one bucket, the row's
// line(s) and the accumulator's, 128 bytes each; the other side (the caller's arrays) streams.  So a
// wave takes 64 keys at a time, one per lane, finds them four lanes per bucket as the pull's
// lookup does, and then moves the 64 rows with all lanes as one flat run of 16-byte words,
// kRowInFlight words in flight per lane: whole lines on both sides and no idle lanes for any row
// width.  Measured (four lanes copying a row four bytes at a time before, in brackets):
//   get, 2.05 M keys, dim 32: 114 us (439);
//   insert with values, 1.3 M new keys, dim 16: 149 us (247 in two kernels that each probed), which is
//   what two random partial-line writes per key (row, accumulator) cost at 22 G/s;
//   dump of 0.16 M changed rows out of 6 M slots, dim 32: 38 us (302, one thread per row).
#pragma once

#include "common.hpp"
#include "table.hpp"

namespace hps {

constexpr int kRowThreads = 256;
constexpr int kRowMaxBlocks = 1 << 20;     // a wave takes one or a few batches of 64 keys
constexpr int kRowInFlight = 8;

__device__ __forceinline__ bool aligned16(const void* p) { return ((uintptr_t)p & 15u) == 0; }

// The caller's arrays may be aligned to four bytes only.
__device__ __forceinline__ float4 load_caller4(const float* p, bool aligned) {
  if (aligned) return *reinterpret_cast<const float4*>(p);
  return make_float4(p[0], p[1], p[2], p[3]);
}
// What goes out is not read again here: stored past the L2, it leaves the cache to the table's lines (get of
// 2.05 M keys, dim 32, many of them several times: 166 -> 114 us; of 1.6 M bfloat16 rows, dim 64: 252 -> 194).
__device__ __forceinline__ void store_caller4(float* p, bool aligned, float4 v) {
  typedef float Words4 __attribute__((ext_vector_type(4)));
  if (aligned) {
    const Words4 x = {v.x, v.y, v.z, v.w};
    __builtin_nontemporal_store(x, reinterpret_cast<Words4*>(p));
    return;
  }
  p[0] = v.x; p[1] = v.y; p[2] = v.z; p[3] = v.w;
}

// Goes through the `words` 16-byte words of each of the 64 keys of a wave, flat: word e of the
// run is word e % words of key e / words.  Lane l starts at word l and advances by 64 words.
struct FlatWalk {
  u32 key, col;         // where this lane stands
  u32 d_key, d_col;     // what 64 words further means
  __device__ __forceinline__ FlatWalk(u32 words) {
    key = lane_id() / words; col = lane_id() % words;
    d_key = kWave / words; d_col = kWave % words;
  }
  __device__ __forceinline__ void next(u32 words) {
    key += d_key; col += d_col;
    if (col >= words) { col -= words; ++key; }
  }
};

// Calls load(row, key, col) and store(value, row, key, col) for every word of the rows of the
// wave's 64 keys, kRowInFlight loads before their stores; my_row: lane l's row number of key l
// (kSkipRow: nothing; kNoRow: nothing either, or with ZERO a store of V()).
constexpr u32 kSkipRow = kNoRow - 1;       // (above any row number: hps.hip, kMaxSlots)
template <bool ZERO, typename V, typename LOAD, typename STORE>
__device__ __forceinline__ void move_rows(u32 my_row, u32 words, LOAD load, STORE store) {
  FlatWalk at(words);
  for (u32 i0 = 0; i0 < words; i0 += kRowInFlight) {       // 64 * words words, 64 per step
    V v[kRowInFlight];
    u32 row[kRowInFlight], key[kRowInFlight], col[kRowInFlight];
#pragma unroll
    for (int q = 0; q < kRowInFlight; ++q) {
      row[q] = i0 + q < words ? (u32)__shfl((int)my_row, (int)at.key, kWave) : kSkipRow;
      key[q] = at.key; col[q] = at.col;
      v[q] = V();
      if (row[q] < kSkipRow) v[q] = load(row[q], key[q], col[q]);
      at.next(words);
    }
#pragma unroll
    for (int q = 0; q < kRowInFlight; ++q)
      if (row[q] < kSkipRow || (ZERO && row[q] == kNoRow)) store(v[q], row[q], key[q], col[q]);
  }
}

// rows by key, nothing created; found_out[u] tells whether the table holds the key.  w_out / acc_out
// of a key it does not hold are left unwritten, or with ZERO set to zero (while the sticky status
// is set, all of them: then nothing is looked up).
template <bool BF16, bool ZERO>
__global__ void __launch_bounds__(kRowThreads)
get_rows(TableView t, const u64* __restrict__ keys, u64 n_keys, float* __restrict__ w_out,
         float* __restrict__ acc_out, uint8_t* __restrict__ found_out) {
  const bool failed = load_error(t.st) != 0;
  if (failed && !ZERO) return;
  const u32 lane = lane_id(), sub = lane % kLookupLanes;
  const u64 n_waves = (u64)gridDim.x * (kRowThreads / kWave);
  const bool aligned = aligned16(w_out) && aligned16(acc_out);
  for (u64 first = ((u64)blockIdx.x * (kRowThreads / kWave) + threadIdx.x / kWave) * kWave; first < n_keys;
       first += n_waves * kWave) {
    const u64 u = first + lane;
    u64 key = u < n_keys && !failed ? keys[u] : kEmptyKey, line;
    u32 row, free_at;
    search_keys<kLookupLanes>(t, &key, &line, &row, &free_at, sub);
    if (u < n_keys) found_out[u] = row != kNoRow;
    else row = kSkipRow;
    float* w_first = w_out + first * t.dim;
    if (t.acc_len == 1) {
      if (row < kSkipRow) acc_out[u] = acc_value(*acc_row(t, row));
      else if (ZERO && row == kNoRow) acc_out[u] = 0.f;
    }
    move_rows<ZERO, StoredW4<BF16>>(
        row, t.dim >> 2, [&](u32 r, u32, u32 col) { return load_stored_w4<BF16>(t, r, col); },
        [&](const StoredW4<BF16>& v, u32, u32 k, u32 col) {
          store_caller4(w_first + k * t.dim + 4 * col, aligned, v.value());
        });
    if (t.acc_len != 1) {
      float* acc_first = acc_out + first * t.acc_len;
      move_rows<ZERO, StoredW4<false>>(
          row, t.acc_len >> 2,
          [&](u32 r, u32, u32 col) {
            StoredW4<false> s;
            s.raw = reinterpret_cast<const float4*>(acc_row(t, r))[col];
            return s;
          },
          [&](const StoredW4<false>& s, u32, u32 k, u32 col) {
            float4 v = s.raw;
            v.x = acc_value(v.x); v.y = acc_value(v.y); v.z = acc_value(v.z); v.w = acc_value(v.w);
            store_caller4(acc_first + k * t.acc_len + 4 * col, aligned, v);
          });
    }
  }
}

// Raises the sticky error if the reserved key is among keys[0 .. n): the kernels after it
// then change nothing.
__global__ void __launch_bounds__(kRowThreads)
check_keys(const u64* __restrict__ keys, u64 n, TableState* st) {
  bool bad = false;
  for (u64 i = (u64)blockIdx.x * kRowThreads + threadIdx.x; i < n; i += (u64)gridDim.x * kRowThreads)
    bad = bad || keys[i] == kEmptyKey;
  if (bad) raise_error(st, kErrReserved);
}

// Bulk insert.  VALUES = false: absent keys get their initial row, present keys stay.  VALUES:
// rows are created or overwritten from w_in / acc_in (null: init_acc).  If the table has room
// even if every key were new, absent keys are created here; else they are only counted
// (miss_shard), for insert_missing to create all of them or none.
template <bool BF16, bool VALUES>
__global__ void __launch_bounds__(kRowThreads)
insert_rows(TableView t, const u64* __restrict__ keys, u64 n_keys, const float* __restrict__ w_in,
            const float* __restrict__ acc_in) {
  if (load_error(t.st) != 0) return;
  __shared__ u32 s_made, s_missing;
  if (threadIdx.x == 0) s_made = s_missing = 0;
  __syncthreads();
  // (the size does not change while this kernel runs: every thread decides the same)
  const bool create_here = t.st->size + n_keys <= t.capacity;
  const u32 lane = lane_id(), sub = lane % kLookupLanes, lane0 = lane & ~3u;
  const u64 n_waves = (u64)gridDim.x * (kRowThreads / kWave);
  const bool aligned = aligned16(w_in) && aligned16(acc_in);
  u32 made = 0, missing = 0;
  for (u64 first = ((u64)blockIdx.x * (kRowThreads / kWave) + threadIdx.x / kWave) * kWave; first < n_keys;
       first += n_waves * kWave) {
    const u64 u = first + lane;
    u64 key = u < n_keys ? keys[u] : kEmptyKey, line;
    u32 row, free_at;
    const u32 absent = search_keys<kLookupLanes>(t, &key, &line, &row, &free_at, sub);
    u32 write = VALUES ? row : kNoRow;          // the row this lane's key wants written
    if (!create_here) {
      if (absent >> sub & 1u) ++missing;
    } else if (__any(absent != 0)) {
      // all first attempts in flight together, then whatever is left of each
      line += free_at >> 3;
      u64 seen[kLookupLanes];
#pragma unroll
      for (int k = 0; k < kLookupLanes; ++k) {
        const u64 kk = quad_lane(key, k), kl = quad_lane(line, k);
        const u32 slot = quad_lane(free_at, k) & 7u;
        seen[k] = 0;
        if ((absent >> k & 1u) && sub == slot >> 1)
          seen[k] = atomicCAS((unsigned long long*)&t.keys[kl * kSlotsPerLine + slot],
                              (unsigned long long)kEmptyKey, (unsigned long long)kk);
      }
#pragma unroll
      for (int k = 0; k < kLookupLanes; ++k) {
        const u64 kk = quad_lane(key, k), kl = quad_lane(line, k);
        const u32 slot = quad_lane(free_at, k) & 7u;
        if (!(absent >> k & 1u)) continue;
        const u64 got = __shfl(seen[k], (int)(lane0 + (slot >> 1)), kWave);
        bool created;
        const u32 r = claim_after4<false>(t, kk, sub, kl, slot, got, &created);
        if (r == kNoRow) {
          raise_error(t.st, kErrInternal);            // (cannot happen: the table has room)
          continue;
        }
        if (sub == (u32)k) {
          if (created) ++made;
          if (created || VALUES) write = r;
        }
      }
    }
    if (VALUES) {
      const float* w_first = w_in + first * t.dim;
      move_rows<false, float4>(
          write, t.dim >> 2,
          [&](u32, u32 k, u32 col) { return load_caller4(w_first + k * t.dim + 4 * col, aligned); },
          [&](float4 v, u32 r, u32, u32 col) { store_w4_as<BF16>(t, r, col, v); });
    } else if (__any(write != kNoRow)) {
      // initial rows: one word of one row per lane and turn
      const u64 base = mix64(key ^ t.init_seed);
      FlatWalk at(t.dim >> 2);
      for (u32 i = 0; i < t.dim >> 2; ++i) {
        const u32 r = (u32)__shfl((int)write, (int)at.key, kWave);
        const u64 b = __shfl((unsigned long long)base, (int)at.key, kWave);
        if (r != kNoRow) store_w4_as<BF16>(t, r, at.col, init_weight4(b, at.col, t.init_range));
        at.next(t.dim >> 2);
      }
    }
    const bool given = VALUES && acc_in != nullptr;
    if (t.acc_len == 1) {
      if (write != kNoRow) *acc_row(t, write) = given ? acc_value(acc_in[u]) : t.init_acc;
    } else {
      const float* acc_first = acc_in + first * t.acc_len;
      move_rows<false, float4>(
          write, t.acc_len >> 2,
          [&](u32, u32 k, u32 col) {
            return given ? load_caller4(acc_first + k * t.acc_len + 4 * col, aligned)
                         : make_float4(t.init_acc, t.init_acc, t.init_acc, t.init_acc);
          },
          [&](float4 v, u32 r, u32, u32 col) {
            v.x = acc_value(v.x); v.y = acc_value(v.y); v.z = acc_value(v.z); v.w = acc_value(v.w);
            reinterpret_cast<float4*>(acc_row(t, r))[col] = v;
          });
    }
  }
  if (made) atomicAdd(&s_made, made);
  if (missing) atomicAdd(&s_missing, missing);
  __syncthreads();
  if (threadIdx.x == 0) {
    if (s_made) atomicAdd(&t.st->made_shard[blockIdx.x % kCountShards], s_made);
    if (s_missing) atomicAdd(&t.st->miss_shard[blockIdx.x % kCountShards], s_missing);
  }
}

// dump: every occupied slot (DIRTY: every occupied slot whose row is marked as updated; the mark
// of a row that is written out is cleared), order unspecified.  A block looks at kDumpSlots * ROUNDS
// slots at a time, lists the rows to go out in LDS, takes places for them from one counter and
// moves them with all lanes.  The counter goes on from dump to dump: `counted` is where it stood.
//
// What bounds it is the read of every slot's key or mark, and the one counter, whose additions the memory
// side takes one after the other: kDumpRounds = 4 keeps them few.  Where the accumulators lie in an array
// of their own, one per row, the marks are read first, and keys only of marked slots (an empty slot's
// accumulator may hold anything).  0.16 M changed rows out of 6 M slots, dim 32: 85 us with one round
// a block and keys first, 38 now.
constexpr int kDumpItems = 4;
constexpr int kDumpSlots = kRowThreads * kDumpItems;
constexpr int kDumpMaxBlocks = 4096;
constexpr int kDumpRounds = 4;
constexpr u64 kDumpSmall = 1u << 20;      // fewer slots: one round a block, so that all CUs have a block
template <bool DIRTY, int ROUNDS>
__global__ void __launch_bounds__(kRowThreads)
dump_rows(TableView t, u64* __restrict__ keys_out, float* __restrict__ w_out,
          float* __restrict__ acc_out, u64 max_rows, unsigned long long* __restrict__ counter, u64 counted) {
  __shared__ u32 scratch[kRowThreads / kWave + 1];
  __shared__ unsigned long long s_base;
  __shared__ u32 s_slot[kDumpSlots * ROUNDS];
  const u64 n_slots = t.n_lines * kSlotsPerLine;          // a multiple of 16
  const u64 n_rounds = (n_slots + kDumpSlots * ROUNDS - 1) / (kDumpSlots * ROUNDS);
  const bool aligned = aligned16(w_out) && aligned16(acc_out);
  const u32 words = t.dim >> 2, acc_words = t.acc_len >> 2;
  const bool marks_first = DIRTY && t.acc_pitch == sizeof(float);
  for (u64 round = blockIdx.x; round < n_rounds; round += gridDim.x) {
    const u64 first = round * (kDumpSlots * ROUNDS) + threadIdx.x * kDumpItems;
    u32 out = 0;                                          // bit: the slot goes out
    if (marks_first) {
      float4 m[ROUNDS];
#pragma unroll
      for (int k = 0; k < ROUNDS; ++k) {
        const u64 s0 = first + k * kDumpSlots;
        m[k] = s0 < n_slots ? *reinterpret_cast<const float4*>(t.acc + s0 * sizeof(float)) : make_float4(0.f, 0.f, 0.f, 0.f);
      }
#pragma unroll
      for (int k = 0; k < ROUNDS; ++k)
        out |= ((acc_is_marked(m[k].x) ? 1u : 0u) | (acc_is_marked(m[k].y) ? 2u : 0u) | (acc_is_marked(m[k].z) ? 4u : 0u) |
                (acc_is_marked(m[k].w) ? 8u : 0u)) << (kDumpItems * k);
      u64 key[ROUNDS * kDumpItems];
#pragma unroll
      for (int q = 0; q < ROUNDS * kDumpItems; ++q)
        key[q] = out >> q & 1u ? t.keys[first + q / kDumpItems * kDumpSlots + q % kDumpItems] : kEmptyKey;
#pragma unroll
      for (int q = 0; q < ROUNDS * kDumpItems; ++q)
        if (key[q] == kEmptyKey) out &= ~(1u << q);
    } else {
#pragma unroll
      for (int k = 0; k < ROUNDS; ++k) {
        const u64 s0 = first + k * kDumpSlots;
        if (s0 >= n_slots) continue;
        const ulonglong2 a = reinterpret_cast<const ulonglong2*>(t.keys + s0)[0];
        const ulonglong2 b = reinterpret_cast<const ulonglong2*>(t.keys + s0)[1];
        out |= ((a.x != kEmptyKey ? 1u : 0u) | (a.y != kEmptyKey ? 2u : 0u) | (b.x != kEmptyKey ? 4u : 0u) |
                (b.y != kEmptyKey ? 8u : 0u)) << (kDumpItems * k);
      }
      if (DIRTY) {
        float mark[ROUNDS * kDumpItems];
#pragma unroll
        for (int q = 0; q < ROUNDS * kDumpItems; ++q)
          mark[q] = out >> q & 1u ? *acc_row(t, first + q / kDumpItems * kDumpSlots + q % kDumpItems) : 0.f;
#pragma unroll
        for (int q = 0; q < ROUNDS * kDumpItems; ++q)
          if (!acc_is_marked(mark[q])) out &= ~(1u << q);
      }
    }
    u32 total;
    u32 at = block_excl_sum<kRowThreads>((u32)__popc(out), scratch, &total);
    for (u32 left = out; left; left &= left - 1) {
      const u32 q = __ffs(left) - 1;
      s_slot[at++] = (u32)(first + q / kDumpItems * kDumpSlots + q % kDumpItems);
    }
    if (threadIdx.x == 0 && total) s_base = atomicAdd(counter, (unsigned long long)total) - counted;
    __syncthreads();
    if (total) {
      const u64 base = s_base;
      const u32 count = base >= max_rows ? 0u : (u32)min((u64)total, max_rows - base);
      for (u32 i = threadIdx.x; i < count; i += kRowThreads) keys_out[base + i] = t.keys[s_slot[i]];
      if (t.acc_len == 1)
        for (u32 i = threadIdx.x; i < count; i += kRowThreads) {
          float* a = acc_row(t, s_slot[i]);
          const float v = acc_value(*a);
          acc_out[base + i] = v;
          if (DIRTY) *a = v;
        }
      float* w_first = w_out + base * t.dim;
#pragma unroll 4
      for (u32 e = threadIdx.x; e < count * words; e += kRowThreads)
        store_caller4(w_first + 4 * e, aligned, load_w4(t, s_slot[e / words], e % words));
      if (t.acc_len != 1) {
        float* acc_first = acc_out + base * t.acc_len;
        for (u32 e = threadIdx.x; e < count * acc_words; e += kRowThreads) {
          float4* a = reinterpret_cast<float4*>(acc_row(t, s_slot[e / acc_words])) + e % acc_words;
          float4 v = *a;
          if (DIRTY && e % acc_words == 0) a->x = acc_value(v.x);
          v.x = acc_value(v.x);
          store_caller4(acc_first + 4 * e, aligned, v);
        }
      }
    }
    __syncthreads();
  }
}

}  // namespace hps
