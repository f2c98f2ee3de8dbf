// Row gather + per-bag pooling: pooled[b, :] = sum over the bag's occurrences of the
// row of that occurrence's key (inv_len == null), or their mean (inv_len != null: it
// also receives 1 / (bag length) per bag, which the push needs to hand every occurrence
// its share of the bag's gradient).  A group of LPR lanes owns one bag at a time;
// each lane carries COLS float4 columns (lane*4 + k*LPR*4; COLS = 1 up to dim 256).
// Eight occurrences are in flight at a time.  Wide rows (dim 64, keys that repeat: the caches serve nearly all of them) are bound by
// the instructions per row, so a row's number and place are worked out by one lane of the group and handed to the others by moves; narrow
// ones by the lines they ask for (9.8 M occurrences, dim 16: 170 us, 58 G rows/s) and by the round trips of a turn, which
// overlap.  8.4 M occurrences, dim 64: 215 us with every lane loading every number, 208 now; 40 K, dim 100: 8.9 and 7.6.
// The kernel also ends the pull (table.hpp: end_pull).
#pragma once

#include "common.hpp"
#include "table.hpp"

namespace hps {

constexpr int kPoolThreads = 256;
constexpr int kPoolMaxBlocks = 1024;   // the groups loop over the bags (1536 to 3072 blocks measured no faster)
constexpr int kPoolInFlight = 8;
// Pooled rows are stored past the L2, which is left to the table's rows, where they are more than it holds for the kernel that reads
// them next; never in small mini-batches, whose rows fit beside them.  (us a step of pull, a kernel that reads the pooled rows, push,
// stored past the L2 and into it; that kernel a matrix product: 256 KB 53.4 and 52.5, 2 MB 63 and 61, 4 MB 67.6 and 64.9, 4.8 MB 94.1 and 92.3,
// 8 MB 73.8 and 72.9, 16 MB 87.0 and 88.1, 33 MB 90.8 and 92.1, 102 MB 371 and 374, 262 MB 869 and 879; a product by element: 5 MB 44.6 and 43.4,
// 10 MB 67.8 and 68.6, 33 MB 86.7 and 87.4, 102 MB 368 and 373, 262 MB 886 and 893; small form, 15 MB: 50.8 and 49.0, a matrix product 58.2 and 56.8.)
constexpr u64 kPoolPastL2 = 8u << 20;

// A bag's occurrences: 0 <= lo <= hi <= n whatever the offsets array holds, so that the kernel reads nothing outside row_of[0, n)
// and no sum of a place and a few more overflows (n < 2^30).
struct BagRange {
  i32 lo, hi;
};
__host__ __device__ __forceinline__ BagRange load_bag(const i32* __restrict__ offsets, u32 b, u32 n_bags, u32 n) {
  BagRange r = {0, 0};
  if (b < n_bags) {
    const i32 lo = offsets[b], hi = offsets[b + 1], most = (i32)n;
    r.lo = lo < 0 ? 0 : lo > most ? most : lo;
    r.hi = hi < r.lo ? r.lo : hi > most ? most : hi;
  }
  return r;
}

// A group's bags are b, b + n_groups, ...; `bag` and `next` the first two's occurrences.
template <int LPR, int COLS, bool BF16, bool SMALL>
__device__ __forceinline__ void pool_bags_as(const TableView& t, const i32* __restrict__ offsets, u32 b, BagRange bag, BagRange next,
                                             u32 n_bags, u32 n, const u32* __restrict__ row_of,
                                             float* __restrict__ pooled, float* __restrict__ inv_len,
                                             const uint4* __restrict__ places, u32* __restrict__ bags, bool past_l2) {
  const u32 sub = threadIdx.x % LPR;
  const u32 dim4 = t.dim >> 2;
  const u32 n_groups = gridDim.x * (kPoolThreads / LPR);
  float4 acc[COLS];
#pragma unroll
  for (int c = 0; c < COLS; ++c) acc[c] = make_float4(0.f, 0.f, 0.f, 0.f);
  // the rows of the next eight occurrences; each lane looks up its share of them
  GroupOffsets<LPR> rows;
  u32 at[GroupOffsets<LPR>::kOwn];      // SMALL: positions in the grouped order
  auto load_rows = [&](i32 i0, i32 hi) {
#pragma unroll
    for (int q = 0; q < GroupOffsets<LPR>::kOwn; ++q) {
      const u32 j = q * LPR + sub;
      const bool on = j < (u32)kPoolInFlight && i0 + (i32)j < hi;
      u32 r = kNoRow;
      if (SMALL) {
        const uint2 p = on ? *reinterpret_cast<const uint2*>(places + i0 + j) : make_uint2(kNoRow, kNoRow);
        r = p.x;
        at[q] = p.y;
      } else if (on) {
        r = row_of[i0 + j];
      }
      rows.own[q] = r == kNoRow ? kNowhere : (u64)r * t.w_pitch;
    }
  };
  i32 i0 = bag.lo;
  load_rows(i0, bag.hi);
  // Eight rows a turn, of one bag.  The row numbers of the next turn, whichever bag that is in, and the bounds of the bag after
  // it are requested behind the rows of this one, so that a turn is one round trip and not three.
  while (b < n_bags) {
    // the rows as stored (all loads first: nothing between them that needs their data) ...
    StoredW4<BF16> raw[kPoolInFlight][COLS];
#pragma unroll
    for (int k = 0; k < kPoolInFlight; ++k) {
      u64 offset;
      const bool on = rows.get(k, &offset);
#pragma unroll
      for (int c = 0; c < COLS; ++c) {
        const u32 col = sub + c * LPR;
        if (on && col < dim4) raw[k][c].raw = reinterpret_cast<const decltype(raw[k][c].raw)*>(t.w + offset)[col];
      }
    }
    if (SMALL) {
#pragma unroll
      for (int q = 0; q < GroupOffsets<LPR>::kOwn; ++q)
        if (at[q] != kNoRow) bags[at[q]] = b;
    }
    const bool last = i0 + kPoolInFlight >= bag.hi;
    i0 = last ? next.lo : i0 + kPoolInFlight;
    load_rows(i0, last ? next.hi : bag.hi);
    BagRange after = next;
    if (last) after = load_bag(offsets, b + 2 * n_groups, n_bags, n);
    // ... then as float32 (all-zero bits are 0.0 in both formats)
    float4 v[kPoolInFlight][COLS];
#pragma unroll
    for (int k = 0; k < kPoolInFlight; ++k)
#pragma unroll
      for (int c = 0; c < COLS; ++c) v[k][c] = raw[k][c].value();
    // the (up to) eight rows as a balanced tree, then onto the running sum: a fixed shape,
    // and a smaller rounding error than adding one row after the other
#pragma unroll
    for (int c = 0; c < COLS; ++c) {
#pragma unroll
      for (int w = 1; w < kPoolInFlight; w <<= 1) {
#pragma unroll
        for (int k = 0; k + w < kPoolInFlight; k += 2 * w) {
          v[k][c].x += v[k + w][c].x; v[k][c].y += v[k + w][c].y;
          v[k][c].z += v[k + w][c].z; v[k][c].w += v[k + w][c].w;
        }
      }
      acc[c].x += v[0][c].x; acc[c].y += v[0][c].y; acc[c].z += v[0][c].z; acc[c].w += v[0][c].w;
    }
    if (last) {
      if (inv_len) {
        const float len = (float)max(bag.hi - bag.lo, 1);
        if (sub == 0) inv_len[b] = 1.0f / len;
#pragma unroll
        for (int c = 0; c < COLS; ++c) { acc[c].x /= len; acc[c].y /= len; acc[c].z /= len; acc[c].w /= len; }
      }
      float4* out = reinterpret_cast<float4*>(pooled + (u64)b * t.dim);
#pragma unroll
      for (int c = 0; c < COLS; ++c) {
        const u32 col = sub + c * LPR;
        typedef float Words4 __attribute__((ext_vector_type(4)));
        const Words4 x = {acc[c].x, acc[c].y, acc[c].z, acc[c].w};
        if (col < dim4) {
          if (past_l2) {
            // (an instruction of its own on either side: the compiler would make one store of the two, and an ordinary one)
            asm volatile("s_nop 0");
            __builtin_nontemporal_store(x, reinterpret_cast<Words4*>(out + col));
            asm volatile("s_nop 0");
          } else {
            *reinterpret_cast<Words4*>(out + col) = x;
          }
        }
        acc[c] = make_float4(0.f, 0.f, 0.f, 0.f);
      }
      b += n_groups;
      bag = next;
      next = after;
    }
  }
}

// row_of[i]: the row of occurrence i's key.  SMALL (small.hpp): that is in places[i], with its position in the order grouped
// by key, for which its bag is put down.
template <int LPR, int COLS, bool SMALL>
__global__ void __launch_bounds__(kPoolThreads)
pool_bags(TableView t, const i32* __restrict__ offsets, u32 n_bags, u32 n, const u32* __restrict__ row_of,
          float* __restrict__ pooled, float* __restrict__ inv_len, const uint4* __restrict__ places, u32* __restrict__ bags,
          PullEnd end) {
  const u32 b = (blockIdx.x * kPoolThreads + threadIdx.x) / LPR, n_groups = gridDim.x * (kPoolThreads / LPR);
  const BagRange bag = load_bag(offsets, b, n_bags, n), next = load_bag(offsets, b + n_groups, n_bags, n);
  if (!end_pull(t, end)) return;
  const bool past_l2 = !SMALL && (u64)n_bags * t.dim * sizeof(float) > kPoolPastL2;
  if (t.bf16) pool_bags_as<LPR, COLS, true, SMALL>(t, offsets, b, bag, next, n_bags, n, row_of, pooled, inv_len, places, bags, past_l2);
  else pool_bags_as<LPR, COLS, false, SMALL>(t, offsets, b, bag, next, n_bags, n, row_of, pooled, inv_len, places, bags, past_l2);
}

// Plain form of the dedup: row_of[i] = rows[inverse[i]].
__global__ void __launch_bounds__(kPoolThreads)
rows_by_rank(const TableState* st, const i32* __restrict__ inverse, const u32* __restrict__ rows, u32 n,
             u32* __restrict__ row_of) {
  if (load_error(st) != 0) return;      // (the dedup may have failed: its ranks are not to be trusted)
  for (u32 i = blockIdx.x * kPoolThreads + threadIdx.x; i < n; i += gridDim.x * kPoolThreads) row_of[i] = rows[inverse[i]];
}

// Measurement aid, not part of the path: reads random rows of LPR * 16 bytes of an array the
// way the pooling kernel reads table rows (LPR lanes x 16 bytes per row, eight rows in flight
// per lane group, same block size and grid) and nothing else, so that a benchmark can time
// the rate at which this GPU returns such rows.  Every lane group takes per_group rows
// (a multiple of 8) at pseudo-random places; the sums go to sink[group * LPR + lane] only
// to keep the loads alive.
template <int LPR>
__global__ void __launch_bounds__(kPoolThreads)
random_row_probe(const float4* __restrict__ rows, u64 n_rows, u32 per_group, float* __restrict__ sink) {
  const u32 group = (blockIdx.x * kPoolThreads + threadIdx.x) / LPR, sub = threadIdx.x % LPR;
  u64 state = mix64((u64)group + 1);
  float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
  for (u32 i = 0; i < per_group; i += kPoolInFlight) {
    float4 v[kPoolInFlight];
#pragma unroll
    for (int k = 0; k < kPoolInFlight; ++k) {
      state = state * 6364136223846793005ull + 1442695040888963407ull;
      v[k] = rows[__umul64hi(state, n_rows) * LPR + sub];
    }
#pragma unroll
    for (int k = 0; k < kPoolInFlight; ++k) { acc.x += v[k].x; acc.y += v[k].y; acc.z += v[k].z; acc.w += v[k].w; }
  }
  sink[(u64)group * LPR + sub] = acc.x + acc.y + acc.z + acc.w;
}

}  // namespace hps
