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
  int64_t slot;  // index of the tile's chunk 0 in the partials (chunked ranges)
};
__device__ inline bool key_tile_item(const AttnArgs& a, int wg, KeyTileItem& it) {
  int bk, rank;
  if (!xcd_pair_item(wg, a.kv_heads * a.batch, a.split.wgs_per_pair, true, bk, rank)) return false;
  it.b = bk / a.kv_heads;
  it.kvh = bk - it.b * a.kv_heads;
  it.r = a.order[0];
  int64_t base = 0;
  for (int n = 0; n < a.n_k; ++n) {
    const int r = a.order[n], ch = a.split.chunks[r], nw = a.kr[r].ntiles * ch;
    it.r = r;
    if (rank < nw) break;
    rank -= nw;
    if (ch > 1) base += slots_before(a.kr[r].ntiles, a.split.walk[r], a.split.fall[r], a.split.unit);
  }
  const int ch = a.split.chunks[it.r];
  const int nt = imax(a.kr[it.r].ntiles, 1);
  it.chunk = rank / nt;
  it.t = rank - it.chunk * nt;
  it.slot = 0;
  if (ch > 1)
    it.slot = (int64_t)bk * a.split.slots_per_pair + base +
              slots_before(it.t, a.split.walk[it.r], a.split.fall[it.r], a.split.unit);
  return true;
}

// A tile of the chunked ranges, for the kernel that adds up its chunks: tile
// `n` of all pairs' chunked tiles.
struct SumItem {
  int b, kvh, r, t;
  int64_t slot;
};
__device__ inline void sum_item(const AttnArgs& a, int n, SumItem& it) {
  const int bk = n / a.split.tiles_per_pair;
  int tile = n - bk * a.split.tiles_per_pair;
  it.b = bk / a.kv_heads;
  it.kvh = bk - it.b * a.kv_heads;
  it.r = a.order[0];
  it.slot = (int64_t)bk * a.split.slots_per_pair;
  for (int k = 0; k < a.n_k; ++k) {
    const int r = a.order[k], ch = a.split.chunks[r];
    it.r = r;
    if (ch <= 1) continue;
    if (tile < a.kr[r].ntiles) break;
    tile -= a.kr[r].ntiles;
    it.slot += slots_before(a.kr[r].ntiles, a.split.walk[r], a.split.fall[r], a.split.unit);
  }
  it.t = tile;
  it.slot += slots_before(tile, a.split.walk[it.r], a.split.fall[it.r], a.split.unit);
}

}  // namespace bdlm
