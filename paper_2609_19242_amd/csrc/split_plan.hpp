// How the dK/dV walks of a backward are cut into chunks (SplitArgs in
// common.hpp): the decision, and where the chunks' partial sums lie.  Host code.
#pragma once

#include "bdlm_attn.h"

#include <algorithm>
#include <cmath>
#include <cstddef>

#include "common.hpp"

namespace bdlm {

inline size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

inline MaskRule host_rule(const bdlm_problem* p, const int* prefix) {
  return MaskRule{(int)p->block_size, p->clean_intra, (int)p->window, (int)(p->L / p->block_size), (int)p->L, prefix};
}

// The row statistics' part of the backward workspace.
inline size_t stats_bytes(const bdlm_problem* p, int32_t n_q, const bdlm_range* q_ranges) {
  if (!p || !q_ranges || n_q < 1 || n_q > kMaxQ || p->batch < 1 || p->heads < 1 || p->head_dim < 1) return 0;
  size_t tot = 0;
  for (int i = 0; i < n_q; ++i) {
    const size_t rows = (size_t)p->batch * (size_t)(q_ranges[i].len > 0 ? q_ranges[i].len : 0);
    tot += 2 * align256(rows * p->heads * sizeof(float));  // LSE * log2(e), then D = rowsum(dO * O)
  }
  return tot;
}

inline float resolved_scale(const bdlm_problem* p) {
  return p->scale > 0.f ? p->scale : 1.0f / std::sqrt((float)p->head_dim);
}

// Does the scheduled dK/dV kernel run this call?
inline bool scheduled_dkdv(const bdlm_problem* p, int n_q, const bdlm_range* q_ranges) {
  int n_q_rows = 0;  // query ranges with rows (empty ones add no work to dK/dV)
  for (int i = 0; i < n_q; ++i) n_q_rows += q_ranges[i].len > 0 ? 1 : 0;
  return dkdv_uses_scheduled_kernel(p->dtype == BDLM_BF16, p->hilo, n_q_rows, resolved_scale(p));
}

inline int key_tile_rows(const bdlm_problem* p) { return p->dtype == BDLM_F32 ? kRowsF32 : kBwdKeysBf16; }

// Steps of the walk of the keys [first, last] of a stream (an upper bound with
// a clean-context table, which lies in device memory: it may let every
// corrupted query see a clean key.  The decision to cut takes the bound too, so
// a drafter's clean walks look all alike and are cut less than they could be).
inline int64_t walk_steps(const bdlm_problem* p, int n_q, const bdlm_range* q_ranges, int stream, int64_t first,
                          int64_t last) {
  const bool f32 = p->dtype == BDLM_F32;
  // a step: 16 rows of one head (fp32), 32 rows of two heads, or 64 rows of one head (odd groups)
  const int64_t group = p->heads / p->kv_heads, per_block = f32 || group % 2 ? group : group / 2;
  const int step = f32 ? kRowsF32 : group % 2 ? 64 : 32;
  const MaskRule rule = host_rule(p, nullptr);
  int64_t n = 0;
  for (int i = 0; i < n_q; ++i) {
    const bdlm_range& qr = q_ranges[i];
    int lo, hi, lo1, hi1;
    query_interval(qr.stream, stream, (int)first, rule, lo, hi);
    query_interval(qr.stream, stream, (int)last, rule, lo1, hi1);
    if (p->clean_prefix && stream == BDLM_CLEAN && qr.stream == BDLM_CORRUPTED) {
      lo = 0;
      hi1 = kBig;
    }
    const int64_t u0 = std::max<int64_t>(lo - qr.pos0, 0), u1 = std::min<int64_t>(hi1 - qr.pos0, qr.len);
    if (u1 > u0) n += ((u1 + step - 1) / step - u0 / step) * per_block;
  }
  return n;
}

// A key tile's walk covers the queries that see it: every query for the first
// clean keys, one block for corrupted keys.  With few (batch, KV head, tile)
// workgroups the longest walk, not the card, sets the kernel's time.  Walks
// longer than the average load per CU are then cut into chunks of that length
// (fp32: a quarter of it, as its workgroups are lighter), at least min_unit
// steps, below which a workgroup's fixed cost and its partial sums outweigh the
// balance (half as many where every chunk has a CU to itself: 4/2 heads, 256,
// 512 and 768 tokens, 8 -> 4 steps: 26.8 -> 21.6, 27.7 -> 24.3 and 29.3 -> 28.0
// us; 1,024 tokens no longer fit and lose, 31.5 -> 40.4).
// Measured: 2,040 tokens, 32/8 heads: dK/dV 375 -> 207 us, and 12 us for the
// sums (half the average per chunk: 210 and 17); 8K, 32/4 heads, adaptive
// two-term products: 5.5 -> 3.4 ms (half the average: 3.7); 512 tokens, 4/2
// heads: 55 -> 24 us with the sums.  Calls whose longest walk is within
// kCutSteps (or a third) of the average stay whole, as cutting costs about that
// much (3,000 tokens, 16/16 heads: 94 steps, 75 on average: 180 us cut, 167
// whole; 6,000 tokens, 32/8 heads: 750 and 580: 1,157 and 1,216 us).  So does
// a rank's share of a sharded context whose few queries see most keys: many
// walks, all about as long (kMaxChunkBytes: rank 0 of 16 at 41,392 tokens, 24/8
// heads: 178 us whole, 216 cut at the average; rank 0 of 8 at 11,920, 32/4
// heads: 79 us in chunks of 44 steps, 100 in chunks of 22).
//
// The plan takes the problem and its queries only, and the workspace holds it
// for any key ranges that do not overlap, so that a key range's dK and dV do
// not depend on which other key ranges are in the call: chunk k's partial sums
// of a key lie at the key's position in region k of its stream, the positions
// that a walk of more than k chunks may cover whichever row its tile starts at.
struct SplitPlan {
  int64_t unit = 0;       // steps per chunk (0: walks stay whole)
  int64_t rows = 0;       // rows of partial sums per (batch, KV head)
  size_t counts_bytes = 0, bytes = 0;  // of the workspace: counts, counts + partials
  int32_t at[2][kMaxChunks] = {};      // SplitArgs::at
};
constexpr int kCus = 256;
constexpr int kMaxSplitTiles = 16 * kCus;  // with more (tile, batch, KV head) workgroups per stream the CUs get about
                                           // the average load anyway
constexpr size_t kMaxChunkBytes = (size_t)256 << 20;
constexpr int kCutSteps = 25, kMinUnitF32 = 8, kMinUnitBf16 = 8, kMinUnitBf16Idle = 4;

inline SplitPlan split_plan(const bdlm_problem* p, int n_q, const bdlm_range* q_ranges) {
  SplitPlan pl;
  const bool f32 = p->dtype == BDLM_F32;
  if (!f32 && !scheduled_dkdv(p, n_q, q_ranges)) return pl;
  const int tile = key_tile_rows(p);
  const int64_t pairs = (int64_t)p->kv_heads * p->batch, tiles = (p->L + tile - 1) / tile;
  if (tiles * pairs > kMaxSplitTiles) return pl;
  // The allocation-free backward cuts the same calls the same way, so its scratch sets the limit.
  const size_t stats = stats_bytes(p, n_q, q_ranges);
  if (stats >= BDLM_NOALLOC_SCRATCH_BYTES) return pl;
  const size_t room = BDLM_NOALLOC_SCRATCH_BYTES - stats;

  int32_t walk[2][kMaxSplitTiles];
  int64_t total = 0, longest_of[2] = {0, 0};
  for (int s = 0; s < 2; ++s)
    for (int64_t t = 0; t < tiles; ++t) {
      const int64_t n = walk_steps(p, n_q, q_ranges, s, t * tile, std::min<int64_t>((t + 1) * tile, p->L) - 1);
      walk[s][t] = (int32_t)n;
      longest_of[s] = std::max(longest_of[s], n);
      total += n * pairs;
    }
  const int64_t longest = std::max(longest_of[0], longest_of[1]);

  const int64_t average =
      total / (f32 ? kCus : kCus * dkdv_wgs_per_cu(p->head_dim, p->hilo, p->heads / p->kv_heads));
  int64_t unit = f32 ? std::max<int64_t>(kMinUnitF32, average / 4) : std::max<int64_t>(kMinUnitBf16, average);
  if (!f32 && average < kMinUnitBf16) {
    // a nearly idle card: shorter chunks as long as every workgroup has a CU to itself
    const int64_t u = std::max<int64_t>(kMinUnitBf16Idle, average);
    int64_t wgs = 0;
    for (int s = 0; s < 2; ++s) wgs += tiles * std::max<int64_t>((longest_of[s] + u - 1) / u, 1);
    if (wgs * pairs <= kCus) unit = u;
  }
  const int64_t margin = f32 ? 0 : std::min<int64_t>(kCutSteps, average / 3);
  if (longest <= average + margin) return pl;
  const size_t row_bytes = (size_t)2 * p->head_dim * (f32 ? sizeof(double) : sizeof(float));
  // Longer chunks where the (tile, chunk) pairs, counted along the slowest fall
  // from a stream's longest walk, come to more than kMaxChunkBytes of partial sums.
  for (; longest > unit; unit *= 2) {
    int64_t chunks = 0;
    for (int s = 0; s < 2; ++s) {
      if (longest_of[s] <= unit) continue;
      int64_t fall = tiles > 1 ? longest_of[s] : 0;
      for (int64_t t = 1; t < tiles; ++t) fall = std::min<int64_t>(fall, (longest_of[s] - walk[s][t]) / t);
      chunks += (2 * tiles * (longest_of[s] + unit) - fall * tiles * (tiles - 1) + 2 * unit - 1) / (2 * unit);
    }
    if ((size_t)(chunks * pairs) * (tile * row_bytes + sizeof(int32_t)) <= kMaxChunkBytes) break;
  }
  if (longest <= unit) return pl;

  // Per tile of a stream an upper bound of the walk of any tile that starts in
  // it: that of the rows it may cover (window walks, which such a bound would
  // lengthen a lot, by quarters of a tile).
  const int grid = p->window > 0 ? tile / 4 : tile;
  int32_t reach[2][kMaxSplitTiles];
  int64_t reach_max = 0;
  for (int s = 0; s < 2; ++s)
    for (int64_t t = 0; t < tiles; ++t) {
      int64_t m = 0;
      for (int64_t k0 = t * tile; k0 < std::min<int64_t>((t + 1) * tile, p->L); k0 += grid)
        m = std::max(m, walk_steps(p, n_q, q_ranges, s, k0, std::min<int64_t>(k0 + grid + tile - 1, p->L) - 1));
      reach[s][t] = (int32_t)m;
      reach_max = std::max(reach_max, m);
    }
  pl.counts_bytes = align256((size_t)((2 * tiles + kMaxK) * pairs) * sizeof(int32_t));
  // longer chunks where the partial sums do not fit
  for (; longest > unit; unit += (unit + 3) / 4) {
    if (reach_max > unit * kMaxChunks) continue;
    int64_t rows = 0;
    for (int s = 0; s < 2; ++s)
      for (int64_t k = 0; k < kMaxChunks; ++k) {
        int64_t a = -1, b = 0;
        for (int64_t t = 0; t < tiles; ++t)
          if (reach[s][t] > std::max<int64_t>(k, 1) * unit) {  // (walks of one chunk leave no partial sums)
            if (a < 0) a = t * tile;
            b = std::min<int64_t>((t + 2) * tile, p->L);
          }
        if (a < 0) break;
        pl.at[s][k] = (int32_t)(rows - a);
        rows += b - a;
      }
    pl.bytes = pl.counts_bytes + (size_t)(rows * pairs) * row_bytes;
    if (pl.bytes <= room) {
      pl.unit = unit;
      pl.rows = rows;
      return pl;
    }
  }
  return SplitPlan{};
}

// The chunks of a call's key ranges under a plan (unit 0: whole walks).
// Ranges that overlap stay whole: they would share partial sums.
inline SplitArgs split_args(const bdlm_problem* p, int n_q, const bdlm_range* q_ranges, int n_k,
                            const bdlm_range* k_ranges, const SplitPlan& pl) {
  SplitArgs s{};
  bool cut = pl.unit > 0;
  for (int i = 0; i < n_k; ++i)
    for (int j = 0; j < i; ++j) {
      const bdlm_range &a = k_ranges[i], &b = k_ranges[j];
      if (a.stream == b.stream && a.pos0 < b.pos0 + b.len && b.pos0 < a.pos0 + a.len && a.len > 0 && b.len > 0)
        cut = false;
    }
  s.unit = cut ? (int32_t)pl.unit : 1;
  s.rows_per_pair = cut ? (int32_t)pl.rows : 0;
  const int tile = key_tile_rows(p);
  int64_t wgs = 0, chunked = 0;
  for (int j = 0; j < n_k; ++j) {
    const bdlm_range& kr = k_ranges[j];
    const int64_t nt = (kr.len + tile - 1) / tile;
    int64_t walk = 0;
    if (cut)
      for (int64_t t = 0; t < nt; ++t)
        walk = std::max(walk, walk_steps(p, n_q, q_ranges, kr.stream, kr.pos0 + t * tile,
                                         kr.pos0 + std::min<int64_t>((t + 1) * tile, kr.len) - 1));
    const int64_t ch = cut ? std::max<int64_t>((walk + pl.unit - 1) / pl.unit, 1) : 1;
    s.chunks[j] = (int32_t)ch;
    wgs += nt * ch;
    if (ch > 1) chunked += nt;
  }
  s.wgs_per_pair = (int32_t)wgs;
  s.tiles_per_pair = (int32_t)chunked;
  for (int k = 0; cut && k < kMaxChunks; ++k) {
    s.at[0][k] = pl.at[0][k];
    s.at[1][k] = pl.at[1][k];
  }
  return s;
}

}  // namespace bdlm
