// Internal definitions shared by the BDLM attention kernels and the C ABI layer.
//
// The mask of BDLM training (arXiv 2609.19242, Sec. 3.2 and App. A step 1) is
// expressed as intervals: for a query row at position pq of stream qs, the
// visible keys of stream ks form one interval of positions [lo, hi), and for a
// key row at position pk the queries that see it form one interval too.  Both
// ends are non-decreasing in the position, which is what makes tile
// classification a closed form: over a tile of query rows [pq0, pq1] the union
// of the visible key intervals is [lo(pq0), hi(pq1)) and their intersection is
// [lo(pq1), hi(pq0)).  Key tiles inside the intersection are fully visible
// (no mask test), tiles outside the union are skipped, and only the few in
// between evaluate the mask per element.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace bdlm {

enum : int { kClean = 0, kCorrupted = 1 };
enum : int { kIntraCausal = 0, kIntraBlock = 1 };

constexpr int kMaxQ = 4;
// Products that take their P or dS operand as two bf16 terms (the hilo mask of
// the problem; the values of the BDLM_HILO_* bits of the C ABI).
constexpr int kHiloPv = 1;    // forward P V
constexpr int kHiloDkDv = 2;  // backward P^T dO and dS^T Q (dK/dV kernel)
constexpr int kHiloDq = 4;    // backward dS K (dQ kernel)
constexpr int kHiloAdaptive = 8;  // the second term only on tiles where some probability reaches kHiloTau
constexpr float kHiloTau = 1.0f / 64;
constexpr int kMaxK = 32;
constexpr int kMaxParts = 32;
constexpr int kBig = 0x3fffffff;  // "to the end of the stream" (positions stay below 2^30)

__host__ __device__ inline int imax(int a, int b) { return a > b ? a : b; }
__host__ __device__ inline int imin(int a, int b) { return a < b ? a : b; }

// The mask's parameters.  block_size M and the clean-to-clean reading come
// from Sec. 3.2.  Two optional generalisations keep every visible set an
// interval with non-decreasing ends:
//  * window W > 0 (sliding-window layers, App. "Savings Breakdowns"): a query
//    sees only the last W positions of its clean context, i.e. clean keys in
//    [e - W, e) where e is the end of the context it would see without the
//    window (q + 1, the end of q's block, or the start of q's corrupted block);
//  * prefix (DFlash2 drafter attention, eq:dflash2-block-attention): the clean
//    context of corrupted block b ends at prefix[b] (the block's anchor a_b)
//    instead of at M b.  The table holds nblk = L / M entries, non-decreasing
//    and in [0, L]; entries are clamped into [0, L] when read, so a table that
//    breaks the contract changes the mask but never addresses out of bounds.
struct MaskRule {
  int M, intra, window, nblk, L;
  const int* prefix;  // device (kernels) or host (host code) table, or null
};

// End of the clean context of corrupted block b.
__host__ __device__ inline int clean_end_of_block(const MaskRule& r, int b) {
  if (!r.prefix) return b * r.M;
  const int v = r.prefix[imin(imax(b, 0), r.nblk - 1)];
  return imin(imax(v, 0), r.L);
}

// First corrupted block whose clean context ends after position x (nblk if none).
__host__ __device__ inline int first_block_ending_after(const MaskRule& r, int x) {
  if (!r.prefix) return imin(x / r.M + 1, r.nblk);
  int lo = 0, hi = r.nblk;  // invariant: the answer lies in [lo, hi]
  while (lo < hi) {
    const int mid = (lo + hi) >> 1;
    if (clean_end_of_block(r, mid) > x) hi = mid;
    else lo = mid + 1;
  }
  return lo;
}

// Visible key positions [lo, hi) for a query of stream qs at position pq,
// over keys of stream ks.  Empty when hi <= lo.
__host__ __device__ inline void key_interval(int qs, int pq, int ks, const MaskRule& r, int& lo, int& hi) {
  const int M = r.M, bq = pq / M;
  if (qs == kClean) {
    lo = 0;
    hi = (ks == kClean) ? (r.intra == kIntraBlock ? (bq + 1) * M : pq + 1) : 0;
  } else if (ks == kCorrupted) {  // own corrupted block, bidirectional
    lo = bq * M;
    hi = lo + M;
  } else {  // clean context of the block: the clean prefix of the earlier blocks
    lo = 0;
    hi = clean_end_of_block(r, bq);
  }
  if (ks == kClean && r.window > 0) lo = imax(lo, hi - r.window);
}

// Query positions [lo, hi) of stream qs that see a key of stream ks at
// position pk (the same rules read from the key side).
__host__ __device__ inline void query_interval(int qs, int ks, int pk, const MaskRule& r, int& lo, int& hi) {
  const int M = r.M, bk = pk / M, W = r.window;
  if (qs == kClean) {
    if (ks == kClean) {
      lo = (r.intra == kIntraBlock) ? bk * M : pk;
      // with a window: e(q) <= pk + W, e(q) = q + 1 or the end of q's block
      hi = W <= 0 ? kBig : (r.intra == kIntraBlock ? M * ((pk + W) / M) : pk + W);
    } else {
      lo = kBig;
      hi = kBig;
    }
  } else if (ks == kCorrupted) {
    lo = bk * M;
    hi = lo + M;
  } else {
    // blocks whose clean context [e - W, e) holds pk: e > pk and e <= pk + W
    lo = first_block_ending_after(r, pk) * M;
    hi = W <= 0 ? kBig : first_block_ending_after(r, pk + W) * M;
  }
}


// One query range as the kernels see it.  Pointers are to element 0 of the
// range for batch element 0; row i of batch b is at row (b * bstride + i).
struct QRangeArg {
  int32_t stream;
  int32_t pos0;
  int32_t len;
  int32_t ntiles;     // tiles of this range at the kernel's tile height
  int64_t bstride;    // rows between batch elements
  int32_t tile0;      // first tile of this range in the flattened tile list
  int32_t pad;
  const void* q;
  void* o;
  float* lse;
  const void* dO;
  void* dq;
  float* l2;          // LSE * log2(e), +inf where LSE = -inf, [batch][heads][len]
  float* delta;       // D = rowsum(dO * O), [batch][heads][len]
};

struct KRangeArg {
  int32_t stream;
  int32_t pos0;
  int32_t len;
  int32_t ntiles;
  int64_t bstride;
  int32_t tile0;
  int32_t pad;
  const void* k;
  const void* v;
  void* dk;
  void* dv;
};

// Long dK/dV walks cut into chunks (split_plan.hpp): key range r's tiles are
// walked by up to chunks[r] workgroups, ceil(walk / unit) of them at work, each
// of which leaves its partial sums in `partials`; a second kernel adds them up
// in chunk order.  chunks[r] = 1: one workgroup per tile, which writes the
// gradients itself.
constexpr int kMaxChunks = 64;
struct SplitArgs {
  int32_t wgs_per_pair;    // workgroups per (batch, KV head): sum over ranges of tiles x chunks
  int32_t tiles_per_pair;  // tiles of the chunked ranges per (batch, KV head)
  int32_t unit;            // walk steps per chunk aimed at
  int32_t rows_per_pair;   // rows of partial sums (dK and dV of one key and chunk) per (batch, KV head)
  int32_t* counts;         // chunks at work, per tile of the chunked ranges
  void* partials;
  int32_t chunks[kMaxK];
  int32_t at[2][kMaxChunks];  // chunk k's row of the key at position 0 of a stream (as if it had one)
};

// Workgroups that share a walk of n steps: about `unit` steps each, at most max_chunks.
__host__ __device__ inline int chunks_of(int n, int unit, int max_chunks) {
  return imin(imax((n + unit - 1) / unit, 1), max_chunks);
}

struct AttnArgs {
  int32_t n_q, n_k;
  int32_t batch, heads, kv_heads, group;
  int32_t M, intra;
  int32_t window;      // clean keys per query at most (0: no limit)
  int32_t nblk;        // blocks per stream, L / M
  int32_t L;
  int32_t stats_form;  // bwd workspace per query row: 0 = (LSE log2(e), D), 1 = (-LSE / scale, -D)
  const int* prefix;   // clean context end per corrupted block (device), or null
  float scale;        // softmax scale
  float scale_log2;   // scale * log2(e): scores are kept in the base-2 domain
  int32_t total_tiles;   // flattened tiles (query tiles for fwd, key tiles for bwd)
  int32_t interleave;    // fwd: query ranges have equal tile counts, visit them round-robin
  int32_t out_f32;       // O, dQ, dK, dV are fp32 (else the input dtype)
  int32_t hilo;          // kHilo* bits: products whose P or dS operand is bf16 hi + lo
  float hilo_tau;        // those products take the second term only on tiles where some P reaches this (0: all tiles)
  int32_t order[kMaxK];  // bwd: visiting order of key ranges (heaviest first)
  QRangeArg qr[kMaxQ];
  KRangeArg kr[kMaxK];
  SplitArgs split;       // dK/dV kernels
};

struct MergeArgs {
  int32_t n_parts;
  int32_t heads;
  int64_t rows;
  int64_t batch;
  int64_t pstride, ostride;  // rows between batch elements in the parts and in the output (>= rows)
  const void* o_parts[kMaxParts];
  const float* lse_parts[kMaxParts];
  void* o;
  float* lse;
};

__host__ __device__ inline MaskRule rule_of(const AttnArgs& a) {
  return MaskRule{a.M, a.intra, a.window, a.nblk, a.L, a.prefix};
}

// Workgroups are dispatched round-robin over the 8 XCDs of an MI355X, each
// with its own L2.  Work item of hardware workgroup wg when every one of nbk
// (batch, KV head) pairs has T items, numbered heaviest first: the XCDs form
// g = gcd(nbk, 8) groups of 8 / g, each serving nbk / g pairs, and a group's
// items are dealt to its XCDs in turn, so that a pair's K/V (or Q/dO) meets in
// as few L2s as the balance allows and every XCD gets its share of heavy and
// light items.  (Contiguous spans of items per XCD, right for nbk a multiple
// of 8, gave one XCD all the heavy items of a pair and another all the light
// ones otherwise: at 8K, 4 KV heads, the heavy half of a causal triangle is
// three quarters of the work.)  The launch has workgroups_for() workgroups;
// false: this one has no item.
// interleave: a group's pairs advance side by side instead of one after the
// other.  The key-major kernels do, so that the heaviest tiles of all pairs
// start first (one pair after the other left the second pair's heaviest tiles
// to start late and end last: 7-8% of the kernel at batch 2 and 4, 4K keys);
// the query-major ones keep pairs in sequence (side by side they put the K/V
// of several heads in one XCD's L2 at once and were slower).
__host__ __device__ inline bool xcd_pair_item(int wg, int nbk, int T, bool interleave, int& pair, int& rank) {
  const int lg = (nbk & 7) == 0 ? 3 : (nbk & 3) == 0 ? 2 : (nbk & 1) == 0 ? 1 : 0;  // log2 g
  const int lm = 3 - lg, xcd = wg & 7;
  const int grp = xcd >> lm, m = nbk >> lg;
  const int item = ((wg >> 3) << lm) + (xcd & ((1 << lm) - 1));
  if (item >= m * T) return false;
  if (interleave) {
    rank = item / m;
    pair = grp * m + item - rank * m;
  } else {
    pair = item / T;
    rank = item - pair * T;
    pair += grp * m;
  }
  return true;
}
inline int workgroups_for(int items) { return (items + 7) & ~7; }

// Launchers (defined in the .hip files).  All return hipSuccess or the launch error.
// Query tile of the bf16 forward: rows per workgroup, teams (fwd_bf16.hip).
struct QTile {
  int rows, teams;
};
hipError_t launch_fwd_bf16(const AttnArgs& a, int head_dim, QTile q, hipStream_t s);
hipError_t launch_fwd_f32(const AttnArgs& a, int head_dim, hipStream_t s);
hipError_t launch_merge(const MergeArgs& a, int head_dim, int part_dtype, int out_dtype, hipStream_t s);
hipError_t launch_bwd_bf16(const AttnArgs& a, int head_dim, hipStream_t s);
hipError_t launch_bwd_dkdv(const AttnArgs& a, int head_dim, hipStream_t s);
hipError_t launch_bwd_dkdv_sum(const AttnArgs& a, int head_dim, hipStream_t s);
hipError_t launch_bwd_dq_bf16(const AttnArgs& a, int head_dim, int rows, hipStream_t s);
hipError_t launch_bwd_dq_f32(const AttnArgs& a, int head_dim, hipStream_t s);
hipError_t launch_bwd_dkv_f32(const AttnArgs& a, int head_dim, hipStream_t s);
hipError_t launch_bwd_sum_f32(const AttnArgs& a, int head_dim, hipStream_t s);

// The walk of a key tile of the scheduled dK/dV kernel over its visible query
// rows, by step index.  The rows come as up to two query ranges; range r is
// seen by the tile's keys in the 32-row blocks [a_r, b_r) (a_r = b_r = 0 when
// empty).  Step i is (range q, block s, head pair hp): blocks from the top
// down, at each block every range active there (range 0 first), each with its
// npairs head pairs in order.  The block axis splits at the four range ends
// into at most three segments with a fixed set of active ranges: segment k
// covers blocks [p_{k+1}, p_k) with cnt_k active ranges (the first q0_k), so
// step i follows from its segment in closed form.
struct WalkPlan {
  int p0, p1, p2, p3;  // range ends, descending
  int st1, st2, nsteps;  // first steps of segments 1 and 2; steps in all
  int cnt0, cnt1, cnt2, q00, q01, q02, npairs;
};
__host__ __device__ inline WalkPlan walk_plan(int a0, int b0, int a1, int b1, int npairs) {
  WalkPlan w;
  int p0 = b0, p1 = a0, p2 = b1, p3 = a1;
  auto cx = [](int& x, int& y) {
    const int hi = imax(x, y), lo = imin(x, y);
    x = hi;
    y = lo;
  };
  cx(p0, p1);
  cx(p2, p3);
  cx(p0, p2);
  cx(p1, p3);
  cx(p1, p2);
  auto act = [](int a, int b, int blk) { return a <= blk && blk < b ? 1 : 0; };
  w.p0 = p0;
  w.p1 = p1;
  w.p2 = p2;
  w.p3 = p3;
  w.cnt0 = act(a0, b0, p1) + act(a1, b1, p1);
  w.cnt1 = act(a0, b0, p2) + act(a1, b1, p2);
  w.cnt2 = act(a0, b0, p3) + act(a1, b1, p3);
  w.q00 = act(a0, b0, p1) ? 0 : 1;
  w.q01 = act(a0, b0, p2) ? 0 : 1;
  w.q02 = act(a0, b0, p3) ? 0 : 1;
  w.npairs = npairs;
  w.st1 = (p0 - p1) * w.cnt0 * npairs;
  w.st2 = w.st1 + (p1 - p2) * w.cnt1 * npairs;
  w.nsteps = w.st2 + (p2 - p3) * w.cnt2 * npairs;
  return w;
}
struct WalkStep {
  int q, s, hp;
  bool live;  // i < nsteps (q, s, hp are meaningless otherwise)
};
__host__ __device__ inline WalkStep walk_step(const WalkPlan& w, int i) {
  const bool k1 = i >= w.st1, k2 = i >= w.st2;
  // (selects between differences: selects between fields become loads through
  // a selected address, which keeps the plan in memory)
  const int p01 = w.p1 - w.p0, p12 = w.p2 - w.p1, c01 = w.cnt1 - w.cnt0, c12 = w.cnt2 - w.cnt1;
  const int q01 = w.q01 - w.q00, q12 = w.q02 - w.q01, s12 = w.st2 - w.st1;
  const int top = w.p0 + (k1 ? p01 : 0) + (k2 ? p12 : 0) - 1;
  const int cnt = w.cnt0 + (k1 ? c01 : 0) + (k2 ? c12 : 0);
  const int q0 = w.q00 + (k1 ? q01 : 0) + (k2 ? q12 : 0);
  const int off = i - (k1 ? w.st1 : 0) - (k2 ? s12 : 0);
  const int per = imax(cnt * w.npairs, 1);
  const int sr = off / per, rem = off - sr * per;
  const int ridx = rem >= w.npairs ? 1 : 0;
  WalkStep st;
  st.live = i >= 0 && i < w.nsteps;
  st.hp = rem - ridx * w.npairs;
  st.q = cnt == 2 ? ridx : q0;
  st.s = top - sr;
  return st;
}

// The dK/dV kernel of bwd_dkdv.hip (single-term or adaptive two-term dK/dV
// products, at most two query ranges with rows) starts its score and dP
// accumulators at -LSE/scale and -D, so the backward workspace holds those
// (stats form 1); the general kernel of bwd_bf16.hip and the fp32 kernel read
// LSE log2(e) and D (form 0).  The general kernel also takes scales so small
// that LSE/scale could pass the fp32 range.
constexpr float kMinScheduledScale = 0x1p-96f;
inline bool dkdv_uses_scheduled_kernel(int dtype_bf16, int hilo, int n_q, float scale) {
  const bool terms_ok = !(hilo & kHiloDkDv) || (hilo & kHiloAdaptive);
  return dtype_bf16 && terms_ok && n_q <= 2 && scale >= kMinScheduledScale;
}

// Workgroups of that kernel that a CU holds: two where a wave has at most 256
// registers, at head_dim 64 but for the two-term form on odd groups (280).
// Planned as two, that form's walks were cut too short: adaptive, head_dim 64,
// 24/8 heads, 2K / 4K / 8K tokens 162 / 423 / 1,275 -> 152 / 407 / 1,179 us;
// 16/16 heads, 1K / 4K 49 / 245 -> 43 / 225 (6/2 heads, 3K: 97 -> 110).
inline int dkdv_wgs_per_cu(int head_dim, int hilo, int group) {
  return head_dim == 64 && !((hilo & kHiloDkDv) && group % 2) ? 2 : 1;
}

// Tile heights the launchers use (the C ABI fills ntiles/tile0 with them).
// The bf16 forward and dQ kernels take 256 query rows per workgroup (8 waves,
// one workgroup per CU) when some row of the call can see many keys, and 128
// (4 waves, two workgroups per CU) when none can see more than the kernel's
// short-walk limit: on short walks one workgroup's start-up and barriers
// overlap the other's products, which outweighs copying every K/V tile for
// half as many rows; on long walks the extra copies cost more.
constexpr int kQRowsLongBf16 = 256;
constexpr int kQRowsShortBf16 = 128;
constexpr int64_t kFwdShortWalk = 16384;  // keys a row may see for the 128-row forward
constexpr int64_t kDqShortWalk = 8192;    // ... and for the 128-row dQ kernel
constexpr int64_t kTeamWgs = 256;         // 128-row tiles of a call at most for two teams (forward)
// (the single-term forward at head_dim 64 always takes 128 rows: its 4-wave
// workgroups run at three waves per SIMD; 64K, 16/8 heads 19.7 -> 16.9 ms)
inline bool fwd_short_always(int head_dim, int hilo) { return head_dim == 64 && !(hilo & kHiloPv); }
constexpr int kRowsF32 = 16;       // fp32 path: query rows, or key rows, per workgroup
constexpr int kBwdKeysBf16 = 128;  // key rows per backward workgroup (4 waves x 32)

}  // namespace bdlm
