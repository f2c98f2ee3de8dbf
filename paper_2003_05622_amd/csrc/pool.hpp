// Row gather + per-bag pooling: pooled[b, :] = sum over the bag's occurrences of the
// row of that occurrence's key (inv_len == null), or their mean (inv_len != null: it
// also receives 1 / (bag length) per bag, which the push needs to hand every occurrence
// its share of the bag's gradient).  A group of LPR lanes owns one bag at a time;
// each lane carries COLS float4 columns (lane*4 + k*LPR*4; COLS = 1 up to dim 256).
// Eight occurrences are in flight at a time: their row numbers, then their rows.
// The kernel also ends the pull (table.hpp: end_pull).
#pragma once

#include "common.hpp"
#include "table.hpp"

namespace hps {

constexpr int kPoolThreads = 256;
constexpr int kPoolMaxBlocks = 1024;   // the groups loop over the bags (1536 to 3072 blocks measured no faster)
constexpr int kPoolInFlight = 8;

template <int LPR, int COLS, bool BF16, bool SMALL>
__device__ __forceinline__ void pool_bags_as(const TableView& t, const i32* __restrict__ offsets,
                                             u32 n_bags, u32 n, const u32* __restrict__ row_of,
                                             float* __restrict__ pooled, float* __restrict__ inv_len,
                                             const uint4* __restrict__ places, u32* __restrict__ bags) {
  const u32 sub = threadIdx.x % LPR;
  const u32 dim4 = t.dim >> 2;
  const u32 n_groups = gridDim.x * (kPoolThreads / LPR);
  for (u32 b = (blockIdx.x * kPoolThreads + threadIdx.x) / LPR; b < n_bags; b += n_groups) {
    float4 acc[COLS];
#pragma unroll
    for (int c = 0; c < COLS; ++c) acc[c] = make_float4(0.f, 0.f, 0.f, 0.f);
    // clamped, so that no offsets array can make the kernel read outside row_of[0, n)
    const i32 lo = max(offsets[b], 0), hi = min(offsets[b + 1], (i32)n);
    for (i32 i0 = lo; i0 < hi; i0 += kPoolInFlight) {
      u32 r[kPoolInFlight];
#pragma unroll
      for (int k = 0; k < kPoolInFlight; ++k) {
        if (SMALL) {
          const uint2 p = i0 + k < hi ? *reinterpret_cast<const uint2*>(places + i0 + k) : make_uint2(kNoRow, 0u);
          r[k] = p.x;
          // (the lanes of the group share the stores)
          if (i0 + k < hi && (u32)k % LPR == sub) bags[p.y] = b;
        } else {
          r[k] = i0 + k < hi ? row_of[i0 + k] : kNoRow;
        }
      }
      // the rows as stored (all loads first: nothing between them that needs their data) ...
      StoredW4<BF16> raw[kPoolInFlight][COLS];
#pragma unroll
      for (int k = 0; k < kPoolInFlight; ++k) {
#pragma unroll
        for (int c = 0; c < COLS; ++c) {
          const u32 col = sub + c * LPR;
          raw[k][c] = (r[k] != kNoRow && col < dim4) ? load_stored_w4<BF16>(t, r[k], col) : StoredW4<BF16>();
        }
      }
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
    }
    if (inv_len) {
      const float len = (float)max(hi - lo, 1);
      if (sub == 0) inv_len[b] = 1.0f / len;
#pragma unroll
      for (int c = 0; c < COLS; ++c) { acc[c].x /= len; acc[c].y /= len; acc[c].z /= len; acc[c].w /= len; }
    }
    float4* out = reinterpret_cast<float4*>(pooled + (u64)b * t.dim);
#pragma unroll
    for (int c = 0; c < COLS; ++c) {
      const u32 col = sub + c * LPR;
      if (col < dim4) out[col] = acc[c];
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
  if (!end_pull(t, end)) return;
  if (t.bf16) pool_bags_as<LPR, COLS, true, SMALL>(t, offsets, n_bags, n, row_of, pooled, inv_len, places, bags);
  else pool_bags_as<LPR, COLS, false, SMALL>(t, offsets, n_bags, n, row_of, pooled, inv_len, places, bags);
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
