// Gradient reduce-by-key fused with the Adagrad row update.
//
// The dedup left the occurrences grouped by distinct key: seg_off[u] .. seg_off[u+1]
// are the positions of key u, and bags[j] is the bag of the occurrence at
// position j.  The gradient of a sum-pooled bag reaches every occurrence
// unchanged, so the gradient of key u is the sum of grads[bags[j]] over its
// positions.  Keys are handled by how often they occur; the pull's lookup already
// sorted the frequent ones into work lists (table.hpp, OftenLists):
//
//   short   a span of distinct keys, or a part of one, per block, a group of LPR lanes per key with
//           at most kShortSeg occurrences: reduced and updated on the spot;
//   medium  one wave per listed key: its lane groups stride over the positions, then add up;
//   chunks  one block per listed chunk of a very frequent key: tree-reduced partial sum; the
//           block that finishes a key's last chunk adds up the partials in chunk order (tree) and
//           updates the row.
//
// What bounds it is the lines asked for: a gradient row per occurrence, and of every distinct key the
// row and the accumulator, read and written (9.8 M occurrences of 2.8 M keys, dim 16: 412 us; at 54 G
// lines read and 22 G lines read and written back a second they take 440, less what L2 holds).  The
// blocks of the one launch take the roles in this order; the chunks first (4.2 M occurrences, dim 64,
// bfloat16 rows: 247 us instead of 216) or the medium keys first (221) were slower, and so was
// forcing eight waves per SIMD (spills: 449 instead of 412 us).
// Every sum has a fixed shape, so results do not depend on scheduling.
#pragma once

#include "common.hpp"
#include "table.hpp"

namespace hps {

constexpr int kPushThreads = 256;
constexpr u32 kPushMediumBlocks = 512, kPushMaxMediumBlocks = 2048;      // waves loop; about two waves a span
// (one block per chunk, as many as the mini-batch could have, up to this: with 512 the skewed
// workload, most of whose occurrences are chunks of very frequent keys, ran its push at two
// waves per SIMD, 0.55 ms instead of 0.32; blocks without a chunk return at once)
constexpr int kPushChunkBlocks = 4096;
// Few spans are shared out over several blocks each, up to kPushMaxParts and kPushSplitBlocks in all, until a
// lane group has about four keys: wide rows leave a block eight lane groups or fewer, which would take
// the keys of a whole span one after the other (40 K occurrences, dim 100: 59 -> 28 us; where the
// spans fill the GPU anyway, more blocks only put off the medium keys and the chunks: 4.2 M occurrences in
// 1024 spans, dim 64, bfloat16 rows, 216 us with one block a span and 273 with two).
constexpr u32 kPushSplitBlocks = 1024;
constexpr int kPushMaxParts = 8;         // blocks that share a span
constexpr int kPushInFlight = 8;  // gradient rows a lane group has in flight
constexpr int kStepRowwise = 0;      // Adagrad, one accumulator per row
constexpr int kStepElementwise = 1;  // Adagrad, one accumulator per element
constexpr int kStepAdd = 2;          // Section 4.1 accumulate: the summed values are added

struct PushArgs {
  UniqueSpans spans;
  const u32* seg_off;
  const u32* bags;
  const u32* rows;
  const float* grads;
  const float* inv_len;   // != null (mean pooling): per bag, the share of its gradient an occurrence gets
  const PullCtx* ctx;
  const u32* med_list;        // unique indices
  const uint2* med_span;      // per block of the lookup: its part of the list
  const uint4* chunk_items;   // (unique index, chunk number, number of the chunked key, its first chunk item)
  u32* arrived;               // per chunked key: chunks summed so far
  u32 chunk_blocks, medium_blocks;      // roles of push_main's blocks: chunks, medium, short
  u32 chunk;                  // occurrences per chunk
  u32 parts;                  // short: blocks that share one span
  float* partials;      // [chunk item][dim]
  float lr, eps;
  int kind;   // what a touched row takes: kStepRowwise, kStepElementwise or kStepAdd
};

// One step on row r with the row's summed gradient (or summed values) held as
// float4 columns spread over the LPR lanes of a group.  Marks the row as updated.
template <int LPR, int COLS>
__device__ __forceinline__ void adagrad_row(const TableView& t, u32 r, const float4* g, u32 sub,
                                            float lr, float eps, int kind) {
  const u32 dim4 = t.dim >> 2;
  if (kind == kStepAdd) {
#pragma unroll
    for (int c = 0; c < COLS; ++c) {
      const u32 col = sub + c * LPR;
      if (col < dim4) {
        float4 v = load_w4(t, r, col);
        v.x += g[c].x; v.y += g[c].y; v.z += g[c].z; v.w += g[c].w;
        store_w4(t, r, col, v);
      }
    }
    if (sub == 0) {
      float* G = acc_row(t, r);
      *G = acc_marked(*G);
    }
  } else if (kind == kStepRowwise) {
    float ss = 0.f;
#pragma unroll
    for (int c = 0; c < COLS; ++c)
      if (sub + c * LPR < dim4) ss += g[c].x * g[c].x + g[c].y * g[c].y + g[c].z * g[c].z + g[c].w * g[c].w;
#pragma unroll
    for (int d = LPR / 2; d > 0; d >>= 1) ss += __shfl_xor(ss, d, kWave);
    float* G = acc_row(t, r);
    const float Gn = acc_value(*G) + ss / (float)t.dim;
    const float scale = lr / (sqrtf(Gn) + eps);
#pragma unroll
    for (int c = 0; c < COLS; ++c) {
      const u32 col = sub + c * LPR;
      if (col < dim4) {
        float4 v = load_w4(t, r, col);
        v.x -= scale * g[c].x; v.y -= scale * g[c].y; v.z -= scale * g[c].z; v.w -= scale * g[c].w;
        store_w4(t, r, col, v);
      }
    }
    if (sub == 0) *G = acc_marked(Gn);
  } else {
    float4* G = reinterpret_cast<float4*>(acc_row(t, r));
#pragma unroll
    for (int c = 0; c < COLS; ++c) {
      const u32 col = sub + c * LPR;
      if (col < dim4) {
        float4 a = G[col], v = load_w4(t, r, col);
        a.x = acc_value(a.x) + g[c].x * g[c].x; a.y += g[c].y * g[c].y; a.z += g[c].z * g[c].z; a.w += g[c].w * g[c].w;
        v.x -= lr * g[c].x / (sqrtf(a.x) + eps);
        v.y -= lr * g[c].y / (sqrtf(a.y) + eps);
        v.z -= lr * g[c].z / (sqrtf(a.z) + eps);
        v.w -= lr * g[c].w / (sqrtf(a.w) + eps);
        if (col == 0) a.x = acc_marked(a.x);
        G[col] = a;
        store_w4(t, r, col, v);
      }
    }
  }
}

// Adds the bag gradients of positions lo, lo+stride, ... < hi, kPushInFlight positions
// in flight at a time; each batch is summed as a balanced tree, then added.
template <int LPR, int COLS>
__device__ __forceinline__ void add_positions(float4* g, const PushArgs& a, u32 lo, u32 hi,
                                              u32 stride, u32 dim, u32 sub) {
  const u32 dim4 = dim >> 2;
  typedef GroupOffsets<LPR> Offsets;
  for (u32 j0 = lo; j0 < hi; j0 += kPushInFlight * stride) {
    // (Each lane looks up its share of the bags.  Requesting the next ones behind the rows, as the pooling does, costs two waves per SIMD
    // and more: 4.2 M occurrences, dim 64, bfloat16 rows, 218 -> 417 us.)
    Offsets rows;
    float own_share[Offsets::kOwn];
#pragma unroll
    for (int q = 0; q < Offsets::kOwn; ++q) {
      const u32 k = q * LPR + sub, j = j0 + k * stride;
      const bool on = k < (u32)kPushInFlight && j < hi;
      const u32 bag = on ? a.bags[j] : 0u;
      rows.own[q] = on ? (u64)bag * (dim * sizeof(float)) : kNowhere;
      own_share[q] = a.inv_len && on ? a.inv_len[bag] : 1.0f;
    }
    float4 v[kPushInFlight][COLS];
#pragma unroll
    for (int k = 0; k < kPushInFlight; ++k) {
      u64 offset;
      const bool on = rows.get(k, &offset);
      const float4* row = reinterpret_cast<const float4*>(reinterpret_cast<const char*>(a.grads) + offset);
#pragma unroll
      for (int c = 0; c < COLS; ++c) {
        const u32 col = sub + c * LPR;
        v[k][c] = (on && col < dim4) ? row[col] : make_float4(0.f, 0.f, 0.f, 0.f);
      }
    }
    if (a.inv_len) {
#pragma unroll
      for (int k = 0; k < kPushInFlight; ++k) {
        const float share = __uint_as_float(group_lane<LPR>(__float_as_uint(own_share[k / LPR < Offsets::kOwn ? k / LPR : 0]), k % LPR));
#pragma unroll
        for (int c = 0; c < COLS; ++c) {
          v[k][c].x *= share; v[k][c].y *= share; v[k][c].z *= share; v[k][c].w *= share;
        }
      }
    }
#pragma unroll
    for (int c = 0; c < COLS; ++c) {
#pragma unroll
      for (int w = 1; w < kPushInFlight; w <<= 1) {
#pragma unroll
        for (int k = 0; k + w < kPushInFlight; k += 2 * w) {
          v[k][c].x += v[k + w][c].x; v[k][c].y += v[k + w][c].y;
          v[k][c].z += v[k + w][c].z; v[k][c].w += v[k + w][c].w;
        }
      }
      g[c].x += v[0][c].x; g[c].y += v[0][c].y; g[c].z += v[0][c].z; g[c].w += v[0][c].w;
    }
  }
}

template <int LPR, int COLS>
__device__ __forceinline__ void push_short_role(const TableView& t, const PushArgs& a, u32 block) {
  const u32 sub = threadIdx.x % LPR;
  const bool heavies = block < heavy_blocks(a.spans);
  const u32 rest = block - heavy_blocks(a.spans), span = rest / a.parts, h0 = block * kHeavyGroup;
  const u32 part = heavies ? 0 : rest % a.parts, parts = heavies ? 1 : a.parts;
  u32 first = 0, count;
  if (heavies) count = a.ctx->n_heavy > h0 ? min(kHeavyGroup, a.ctx->n_heavy - h0) : 0u;
  else unique_span(a.spans, a.ctx, span, &first, &count);
  for (u32 k = part * (kPushThreads / LPR) + threadIdx.x / LPR; k < count; k += parts * (kPushThreads / LPR)) {
    u32 u = first + k;
    if (heavies) {
      u = a.spans.bucket_start[a.spans.n_spans + h0 + k];
      if (a.spans.bucket_start[a.spans.n_spans + h0 + k + 1] == u) continue;
    }
    const u32 lo = a.seg_off[u], hi = a.seg_off[u + 1], r = a.rows[u];
    if (hi - lo > kShortSeg || r == kNoRow) continue;      // on one of the lists, or nowhere
    float4 g[COLS];
#pragma unroll
    for (int c = 0; c < COLS; ++c) g[c] = make_float4(0.f, 0.f, 0.f, 0.f);
    add_positions<LPR, COLS>(g, a, lo, hi, 1, t.dim, sub);
    adagrad_row<LPR, COLS>(t, r, g, sub, a.lr, a.eps, a.kind);
  }
}

template <int LPR, int COLS>
__device__ __forceinline__ void push_medium_role(const TableView& t, const PushArgs& a, u32 block) {
  constexpr u32 kGroups = kWave / LPR;
  constexpr u32 kWavesPerBlock = kPushThreads / kWave;
  const u32 group = lane_id() / LPR, sub = lane_id() % LPR;
  // The waves go through the parts of the list, a part at a time by `sharers` waves: a span's by a few, a group of heavy keys'
  // (up to 64, of hundreds of occurrences each) by as many as it has entries.
  const u32 n_heavy = heavy_blocks(a.spans), n_waves = a.medium_blocks * kWavesPerBlock;
  const u32 heavy_work = n_heavy * kHeavyGroup, sharers = max(1u, n_waves / max(1u, a.spans.n_spans));
  const u32 work = heavy_work + a.spans.n_spans * sharers;
  u32 at = block * kWavesPerBlock + threadIdx.x / kWave, m = 0, step = 1;
  uint2 part = make_uint2(0u, 0u);
  bool fresh = true;
  while (true) {
    if (fresh) {
      if (at >= work) break;
      if (at < heavy_work) {
        part = a.med_span[at / kHeavyGroup];
        m = at % kHeavyGroup;
        step = kHeavyGroup;
      } else {
        part = a.med_span[n_heavy + (at - heavy_work) / sharers];
        m = (at - heavy_work) % sharers;
        step = sharers;
      }
      at += n_waves;
      fresh = false;
    }
    if (m >= part.y) { fresh = true; continue; }
    const u32 u = a.med_list[part.x + m];
    m += step;
    float4 g[COLS];
#pragma unroll
    for (int c = 0; c < COLS; ++c) g[c] = make_float4(0.f, 0.f, 0.f, 0.f);
    add_positions<LPR, COLS>(g, a, a.seg_off[u] + group, a.seg_off[u + 1], kGroups, t.dim, sub);
#pragma unroll
    for (int c = 0; c < COLS; ++c) {
#pragma unroll
      for (int d = LPR; d < kWave; d <<= 1) {
        g[c].x += __shfl_xor(g[c].x, d, kWave);
        g[c].y += __shfl_xor(g[c].y, d, kWave);
        g[c].z += __shfl_xor(g[c].z, d, kWave);
        g[c].w += __shfl_xor(g[c].w, d, kWave);
      }
    }
    const u32 r = a.rows[u];
    if (group == 0 && r != kNoRow) adagrad_row<LPR, COLS>(t, r, g, sub, a.lr, a.eps, a.kind);
  }
}

// Sums, over the kPushThreads/LPR groups of the block, the float4 columns each
// group holds; the result is valid in group 0.  `lds` holds kPushThreads float4.
template <int LPR, int COLS>
__device__ __forceinline__ void block_tree_sum(float4* g, float4* lds, u32 dim4) {
  constexpr int kGroups = kPushThreads / LPR;
  const u32 group = threadIdx.x / LPR, sub = threadIdx.x % LPR;
#pragma unroll
  for (int c = 0; c < COLS; ++c) {
    if ((u32)(c * LPR) >= dim4) break;       // block-uniform: no columns left
    const bool has = sub + c * LPR < dim4;
    for (int s = kGroups / 2; s > 0; s >>= 1) {
      __syncthreads();
      if (has && group >= (u32)s && group < (u32)(2 * s)) lds[(group - s) * LPR + sub] = g[c];
      __syncthreads();
      if (has && group < (u32)s) {
        const float4 v = lds[group * LPR + sub];
        g[c].x += v.x; g[c].y += v.y; g[c].z += v.z; g[c].w += v.w;
      }
    }
  }
}

// Partial rows go from one block to another inside the launch: written through to memory and read
// from there (agent-scope accesses), and counted in only once the writes are acknowledged.
// A release fence instead would write back the whole L2 of the XCD, once per chunk.
__device__ __forceinline__ void store_partial(u64* p, float4 v) {
  __hip_atomic_store(p, (u64)__float_as_uint(v.x) | (u64)__float_as_uint(v.y) << 32, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  __hip_atomic_store(p + 1, (u64)__float_as_uint(v.z) | (u64)__float_as_uint(v.w) << 32, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ float4 load_partial(const u64* p) {
  const u64 a = __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  const u64 b = __hip_atomic_load(p + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return make_float4(__uint_as_float((u32)a), __uint_as_float((u32)(a >> 32)), __uint_as_float((u32)b), __uint_as_float((u32)(b >> 32)));
}

template <int LPR, int COLS>
__device__ __forceinline__ void push_chunks_role(const TableView& t, const PushArgs& a, u32 block,
                                                 u32 n_blocks, float4* lds, u32* s_last) {
  constexpr int kGroups = kPushThreads / LPR;
  const u32 kChunk = a.chunk;
  static_assert(LPR <= kWave, "group 0 lies in one wave");
  const u32 n_items = a.ctx->n_chunk_items;
  const u32 group = threadIdx.x / LPR, sub = threadIdx.x % LPR, dim4 = t.dim >> 2;
  for (u32 item = block; item < n_items; item += n_blocks) {
    const uint4 it = a.chunk_items[item];
    const u32 begin = a.seg_off[it.x], end = a.seg_off[it.x + 1];
    const u32 n_chunks = (end - begin + kChunk - 1) / kChunk;
    const u32 lo = begin + it.y * kChunk, hi = min(lo + kChunk, end);
    float4 g[COLS];
#pragma unroll
    for (int c = 0; c < COLS; ++c) g[c] = make_float4(0.f, 0.f, 0.f, 0.f);
    add_positions<LPR, COLS>(g, a, lo + group, hi, kGroups, t.dim, sub);
    block_tree_sum<LPR, COLS>(g, lds, dim4);
    if (n_chunks > 1) {
      if (group == 0) {
        u64* out = reinterpret_cast<u64*>(a.partials + (u64)item * t.dim);
#pragma unroll
        for (int c = 0; c < COLS; ++c)
          if (sub + c * LPR < dim4) store_partial(out + 2 * (sub + c * LPR), g[c]);
      }
      if (threadIdx.x < kWave) {
        // (the wave that holds group 0: its stores are done before its count)
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        if (threadIdx.x == 0)
          *s_last = __hip_atomic_fetch_add(&a.arrived[it.z], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1 == n_chunks;
      }
      __syncthreads();
      const bool last = *s_last != 0;
      __syncthreads();      // (s_last is written again for the next item)
      if (!last) continue;
#pragma unroll
      for (int c = 0; c < COLS; ++c) g[c] = make_float4(0.f, 0.f, 0.f, 0.f);
      // (eight partial rows requested at a time, added in chunk order: a key that fills thousands of
      // chunks would otherwise wait for every row in turn)
      for (u32 c0 = group; c0 < n_chunks; c0 += kPushInFlight * kGroups) {
        float4 v[kPushInFlight][COLS];
#pragma unroll
        for (int k = 0; k < kPushInFlight; ++k) {
          const u32 c = c0 + k * kGroups;
          const u64* row = reinterpret_cast<const u64*>(a.partials + (u64)(it.w + (c < n_chunks ? c : c0)) * t.dim);
#pragma unroll
          for (int q = 0; q < COLS; ++q) {
            const u32 col = sub + q * LPR;
            v[k][q] = (c < n_chunks && col < dim4) ? load_partial(row + 2 * col) : make_float4(0.f, 0.f, 0.f, 0.f);
          }
        }
#pragma unroll
        for (int k = 0; k < kPushInFlight; ++k)
#pragma unroll
          for (int q = 0; q < COLS; ++q) {
            g[q].x += v[k][q].x; g[q].y += v[k][q].y; g[q].z += v[k][q].z; g[q].w += v[k][q].w;
          }
      }
      block_tree_sum<LPR, COLS>(g, lds, dim4);
    }
    const u32 r = a.rows[it.x];
    if (group == 0 && r != kNoRow) adagrad_row<LPR, COLS>(t, r, g, sub, a.lr, a.eps, a.kind);
  }
}

template <int LPR, int COLS>
__global__ void __launch_bounds__(kPushThreads) push_main(TableView t, PushArgs a) {
  __shared__ float4 lds[kPushThreads];
  __shared__ u32 s_last;
  if (a.kind == kStepAdd && blockIdx.x == 0 && threadIdx.x < kWave) commit_absent_wave(t.st);
  if (load_error(t.st) != 0) return;
  const u32 b = blockIdx.x;
  const u32 n_short = heavy_blocks(a.spans) + a.spans.n_spans * a.parts;
  if (b < n_short) {
    push_short_role<LPR, COLS>(t, a, b);
  } else if (b < n_short + a.medium_blocks) {
    push_medium_role<LPR, COLS>(t, a, b - n_short);
  } else {
    push_chunks_role<LPR, COLS>(t, a, b - n_short - a.medium_blocks, a.chunk_blocks, lds, &s_last);
  }
}

}  // namespace hps
