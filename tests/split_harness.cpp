// Host harness for the cut dK/dV walks (split_plan.hpp).  Reads calls from
// stdin: "batch L block heads kv_heads head_dim fp32 intra hilo window",
// a clean-context table "n entries...", then query and key ranges "n (stream
// pos0 len)...".  Per call prints "unit rows_per_pair tiles_per_pair
// counts_bytes bytes stats wgs_per_cu", then per key range "chunks ntiles" and per tile
// its walk as the kernels count it and the first partial row of each chunk at
// work (two or more).
#include <cstdio>
#include <vector>

#include "split_plan.hpp"

using namespace bdlm;

static bool read_ranges(std::vector<bdlm_range>& out) {
  int n;
  if (std::scanf("%d", &n) != 1) return false;
  for (int i = 0; i < n; ++i) {
    bdlm_range r{};
    long long pos0, len;
    if (std::scanf("%d %lld %lld", &r.stream, &pos0, &len) != 3) return false;
    r.pos0 = pos0;
    r.len = len;
    out.push_back(r);
  }
  return true;
}

int main() {
  long long batch, L, M, window;
  int heads, kv, dim, f32, intra, hilo, n_table;
  while (std::scanf("%lld %lld %lld %d %d %d %d %d %d %lld %d", &batch, &L, &M, &heads, &kv, &dim, &f32, &intra, &hilo,
                    &window, &n_table) == 11) {
    std::vector<int> table((size_t)n_table);
    for (int& x : table)
      if (std::scanf("%d", &x) != 1) return 1;
    std::vector<bdlm_range> q, k;
    if (!read_ranges(q) || !read_ranges(k)) return 1;
    bdlm_problem p{};
    p.batch = batch;
    p.L = L;
    p.block_size = M;
    p.heads = heads;
    p.kv_heads = kv;
    p.head_dim = dim;
    p.dtype = f32 ? BDLM_F32 : BDLM_BF16;
    p.clean_intra = intra;
    p.hilo = hilo;
    p.window = window;
    p.clean_prefix = n_table ? table.data() : nullptr;
    const SplitPlan pl = split_plan(&p, (int)q.size(), q.data());
    const SplitArgs a = split_args(&p, (int)q.size(), q.data(), (int)k.size(), k.data(), pl);
    std::printf("%lld %d %d %zu %zu %zu %d\n", (long long)pl.unit, a.rows_per_pair, a.tiles_per_pair, pl.counts_bytes,
                pl.bytes, stats_bytes(&p, (int)q.size(), q.data()), dkdv_wgs_per_cu(dim, hilo, heads / kv));
    const MaskRule rule = host_rule(&p, p.clean_prefix);
    const int tile = key_tile_rows(&p), group = heads / kv;
    const int bm = f32 ? kRowsF32 : group % 2 ? 64 : 32, per = f32 || group % 2 ? group : group / 2;
    for (size_t j = 0; j < k.size(); ++j) {
      const int nt = (int)((k[j].len + tile - 1) / tile);
      std::printf("%d %d", a.chunks[j], nt);
      for (int t = 0; t < nt; ++t) {
        const int first = (int)k[j].pos0 + t * tile, last = first + imin(tile, (int)k[j].len - t * tile) - 1;
        int steps = 0;
        for (const bdlm_range& r : q) {
          int lo, hi, lo1, hi1;
          query_interval(r.stream, k[j].stream, first, rule, lo, hi);
          query_interval(r.stream, k[j].stream, last, rule, lo1, hi1);
          const int u0 = imax(lo - (int)r.pos0, 0), u1 = imin(hi1 - (int)r.pos0, (int)r.len);
          if (u1 > u0) steps += ((u1 + bm - 1) / bm - u0 / bm) * per;
        }
        const int n = a.chunks[j] > 1 ? chunks_of(steps, a.unit, a.chunks[j]) : 1;
        std::printf(" | %d %d", steps, n);
        for (int c = 0; n > 1 && c < n; ++c) std::printf(" %d", first + a.at[k[j].stream][c]);
      }
      std::printf("\n");
    }
  }
  return 0;
}
