// Key-major work items shared by the dK/dV kernels: key tiles whose walks may
// be cut into chunks (SplitArgs in common.hpp), and the sums over the chunks.
#pragma once

#include "common.hpp"

namespace bdlm {

// The key tile of a workgroup of the dK/dV kernel: tiles of a (batch, KV head)
// pair in visiting order (heaviest range first), the first chunks of all tiles
// of a range, then the second ones, and so on: the workgroups that run side by
// side then read the same query rows (the walks of the scheduled kernel start
// at the last query row whatever the tile).
struct KeyTileItem {
  int b, kvh, r, t, chunk;
  int tile;  // index among the tiles of the chunked ranges of all pairs (of the tile's count)
};
__device__ inline bool key_tile_item(const AttnArgs& a, int wg, KeyTileItem& it) {
  int bk, rank;
  if (!xcd_pair_item(wg, a.kv_heads * a.batch, a.split.wgs_per_pair, true, bk, rank)) return false;
  it.b = bk / a.kv_heads;
  it.kvh = bk - it.b * a.kv_heads;
  it.r = a.order[0];
  it.tile = bk * a.split.tiles_per_pair;
  for (int n = 0; n < a.n_k; ++n) {
    const int r = a.order[n], ch = a.split.chunks[r], nw = a.kr[r].ntiles * ch;
    it.r = r;
    if (rank < nw) break;
    rank -= nw;
    if (ch > 1) it.tile += a.kr[r].ntiles;
  }
  const int nt = imax(a.kr[it.r].ntiles, 1);
  it.chunk = rank / nt;
  it.t = rank - it.chunk * nt;
  it.tile += it.t;
  return true;
}

// First row of the partial sums of a chunk of key tile t (of ROWS rows) of range r.
template <int ROWS>
__device__ inline int64_t partial_row(const AttnArgs& a, int b, int kvh, int r, int t, int chunk) {
  const KRangeArg& kr = a.kr[r];
  return (int64_t)(b * a.kv_heads + kvh) * a.split.rows_per_pair + kr.pos0 + t * ROWS + a.split.at[kr.stream][chunk];
}

// A tile of the chunked ranges, for the kernel that adds up its chunks: tile
// `n` of all pairs' chunked tiles.
struct SumItem {
  int b, kvh, r, t;
};
__device__ inline void sum_item(const AttnArgs& a, int n, SumItem& it) {
  const int bk = n / a.split.tiles_per_pair;
  int tile = n - bk * a.split.tiles_per_pair;
  it.b = bk / a.kv_heads;
  it.kvh = bk - it.b * a.kv_heads;
  it.r = a.order[0];
  for (int k = 0; k < a.n_k; ++k) {
    const int r = a.order[k];
    it.r = r;
    if (a.split.chunks[r] <= 1) continue;
    if (tile < a.kr[r].ntiles) break;
    tile -= a.kr[r].ntiles;
  }
  it.t = tile;
}

}  // namespace bdlm
