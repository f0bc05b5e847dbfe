// BDLM attention backward for fp32 inputs, gfx950.
//
// Exact gradients from the saved O and LSE (arXiv 2609.19242 App. C; the
// query gradient eq:correctness-query-gradient and the key/value gradients
// summed over every query row, eq:correctness-clean-gradient):
//   P = exp(scale q.k - LSE),  dP = dO.v,  dS = P (dP - D),  D = dO.O,
//   dQ = scale sum_k dS k,  dK = scale sum_q dS q,  dV = sum_q P dO.
// Inputs and outputs are fp32; scores, exponentials and sums are carried in
// fp64 on the fp64 matrix cores (f64tile.hpp).  Two deterministic passes, no
// atomics:
//  * dQ, query-major like the forward: a workgroup owns 16 query rows of one
//    head (Q and dO as fp64 operands in LDS), its four waves share out the
//    visible 16-key tiles; it also forms D and leaves it in the workspace.
//  * dK/dV, key-major: a workgroup owns 16 keys of one KV head (K and V as
//    fp64 operands in LDS), its four waves share out the visible (16-query
//    tile, head of the group) units.  The early keys are seen by every query
//    while late ones by few, so on small problems a few workgroups would run
//    long after the rest; given workspace, long walks are cut into chunks of
//    about equal work whose fp64 partial sums a second kernel adds up in
//    chunk order.
// Measured against one thread per query row (dQ) or key row (dK, dV), both
// kernels together: L = 256, 2/2 heads, d 64: 10.7 ms -> 44 us; L = 1125, 8/2
// heads, d 128: 621 -> 0.55 ms.
// Registers at head_dim 128: dK and dV keep 128 of a lane's 256 VGPRs, and where
// the guarded path meets the plain one 39 are spilled (128 bytes of scratch per
// lane), with 63 SGPRs (50 at head_dim 64, which spills no VGPR).
#include "f64tile.hpp"
#include "ktiles.hpp"
#include "qtiles.hpp"

namespace bdlm {

namespace {

constexpr int kWaves = 4;

template <int D>
__global__ __launch_bounds__(kWaves * 64) __attribute__((amdgpu_waves_per_eu(2, 2))) void bwd_dq_f32_kernel(
    const AttnArgs a) {
  constexpr int NC = D / 16, OPS = 16 * D;
  // Q and dO as fp64 row operands during the walk, the waves' dQ^T sums after it
  __shared__ __attribute__((aligned(16))) double lds[kWaves * 16 * kRedRow<D>];
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int i = lane & 15, g = lane >> 4;

  QTileItem it;
  if (!q_tile_item(a, workgroup_id(), it)) return;
  const QRangeArg& qr = a.qr[it.r];
  const int kvh = it.h / a.group;
  const int64_t H = a.heads, HKV = a.kv_heads;
  const int row0 = it.t * 16, nvalid = imin(16, qr.len - row0);
  const int64_t qoff = (((int64_t)it.b * qr.bstride + row0) * H + it.h) * D;
  stage_row_operands<D>(lds, (const float*)qr.q + qoff, H * D, nvalid, tid, kWaves * 64);
  stage_row_operands<D>(lds + OPS, (const float*)qr.dO + qoff, H * D, nvalid, tid, kWaves * 64);

  // D = dO.O of this lane's query; the four lanes of a column share the row.
  const int qi = imin(i, nvalid - 1);
  double dl = 0.0;
  {
    const float* op = (const float*)qr.o + qoff + (int64_t)qi * H * D;
    const float* dp = (const float*)qr.dO + qoff + (int64_t)qi * H * D;
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      const fl4 x = *(const fl4*)(op + 16 * c + 4 * g), y = *(const fl4*)(dp + 16 * c + 4 * g);
#pragma unroll
      for (int e = 0; e < 4; ++e) dl = __builtin_fma((double)x[e], (double)y[e], dl);
    }
    dl = col_sum(dl);
  }
  const int64_t hrow = (int64_t)it.b * H + it.h;
  const float lse = qr.lse[hrow * qr.bstride + row0 + qi];
  if (w == 0 && g == 0 && i < nvalid) qr.delta[hrow * qr.len + row0 + i] = (float)dl;
  const bool dead = lse == -INFINITY;  // the row sees no key
  const double lse2 = (double)lse * kLog2eD;
  const double c = (double)a.scale * kLog2eD;
  const int pq = qr.pos0 + row0 + qi;
  const int pq0 = qr.pos0 + row0, pq1 = qr.pos0 + row0 + nvalid - 1;
  const bool any_dead = __builtin_amdgcn_ballot_w64(dead) != 0;
  __syncthreads();

  AccTiles<D> acc;
  acc.zero();
  int j = -1, t = 0, t1 = 0, f0 = 0, f1 = 0, skip = w;
  auto advance = [&]() __attribute__((always_inline)) -> bool {
    t += kWaves;
    while (t >= t1) {
      if (j >= 0) skip = t - t1;
      if (++j >= a.n_k) return false;
      key_tile_span(a, j, qr.stream, pq0, pq1, 16, t, t1, f0, f1);
      t += skip;
    }
    return true;
  };
  t = t1 = -kWaves;
  while (advance()) {
    const KRangeArg& kr = a.kr[j];
    const int64_t koff = (((int64_t)it.b * kr.bstride + t * 16) * HKV + kvh) * D;
    const int krows = imin(16, kr.len - t * 16);
    const RowTile kt = row_tile<D>(kr.k, koff, krows, HKV * D);
    fl4 kx[NC], vx[NC];
    ColOps<D> kc;
    load_rows<D>(kx, kt, i, g);
    load_rows<D>(vx, row_tile<D>(kr.v, koff, krows, HKV * D), i, g);
    kc.load(kt, i, g);
    const bool full = t >= f0 && t < f1 && !any_dead;
    int lo = 0, wid = 0;
    if (!full) lane_key_interval(a, j, qr.stream, pq, lo, wid);
    if (dead) wid = 0;
    const int kbase = kr.pos0 + t * 16 - lo;
    auto seen = [&](int row) { return full || (unsigned)(kbase + row) < (unsigned)wid; };

    const f64x4 s = row_product<D>(kx, lds, lane);
    const f64x4 dp = row_product<D>(vx, lds + OPS, lane);
    f64x4 ds;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const bool see = seen(4 * r + g);
      const double p = exp2_f64(see ? __builtin_fma(s[r], c, -lse2) : kHidden);
      ds[r] = p * (see ? dp[r] - dl : 0.0);
    }
    // as in the forward: hidden keys must not spread an infinity or NaN of K
    if (full || !kc.non_finite()) col_product<D>(acc, kc, ds);
    else col_product_guarded<D>(acc, kt, ds, seen, i, g);
  }

  __syncthreads();  // every wave has left the walk: Q and dO are no longer read
  acc_to_lds<D>(acc, lds + w * 16 * kRedRow<D>, i, g);
  __syncthreads();
  constexpr int EPT = 16 * D / (kWaves * 64);
  const int q = tid / (D / EPT), d0 = (tid % (D / EPT)) * EPT;
  if (q < nvalid) {
    float* out = (float*)qr.dq + qoff + (int64_t)q * H * D + d0;
#pragma unroll
    for (int e4 = 0; e4 < EPT / 4; ++e4) {
      fl4 o;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        double x = 0.0;
#pragma unroll
        for (int k = 0; k < kWaves; ++k) x += lds[(k * 16 + q) * kRedRow<D> + d0 + 4 * e4 + e];
        o[e] = (float)(x * (double)a.scale);
      }
      *(fl4*)(out + 4 * e4) = o;
    }
  }
}

template <int D>
__global__ __launch_bounds__(kWaves * 64) __attribute__((amdgpu_waves_per_eu(2, 2))) void bwd_dkv_f32_kernel(
    const AttnArgs a) {
  constexpr int NC = D / 16, OPS = 16 * D;
  // K and V as fp64 row operands during the walk, the waves' sums after it
  __shared__ __attribute__((aligned(16))) double lds[kWaves * 16 * kRedRow<D>];
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int i = lane & 15, g = lane >> 4;
  KeyTileItem it;
  if (!key_tile_item(a, workgroup_id(), it)) return;
  const KRangeArg& kr = a.kr[it.r];
  const int64_t H = a.heads, HKV = a.kv_heads;
  const int row0 = it.t * 16, nvalid = imin(16, kr.len - row0);
  const int ki = imin(i, nvalid - 1), pk = kr.pos0 + row0 + ki;

  // Units of the walk: (query range, 16-query tile, head of the group), from
  // the end of the first two ranges down, side by side (walk_plan), then the
  // other ranges.  The visible queries of every key tile extend to the end of
  // a range, so the same chunk of all tiles, which run together, reads the
  // same rows, from L2.
  const int kp0 = kr.pos0 + row0, kp1 = kr.pos0 + row0 + nvalid - 1;
  // Tiles [t0, t1) of query range q that some key of this tile sees, and the
  // rows [i0, i1) of the range that every one of them sees.
  struct Span {
    int t0, t1, i0, i1;
  };
  auto span = [&](int q) __attribute__((always_inline)) -> Span {
    Span s{0, 0, 0, 0};
    if (q >= a.n_q) return s;
    const QRangeArg& qr = a.qr[q];
    int lo0, hi0, lo1, hi1;
    query_interval(qr.stream, kr.stream, kp0, rule_of(a), lo0, hi0);
    query_interval(qr.stream, kr.stream, kp1, rule_of(a), lo1, hi1);
    const int u0 = imax(lo0 - qr.pos0, 0), u1 = imin(hi1 - qr.pos0, qr.len);
    if (u1 > u0) {
      s.t0 = u0 / 16;
      s.t1 = (u1 + 15) / 16;
      s.i0 = imax(lo1 - qr.pos0, 0);
      s.i1 = imin(hi0 - qr.pos0, qr.len);
    }
    return s;
  };
  const Span s0 = span(0), s1 = span(1);
  const WalkPlan wp = walk_plan(s0.t0, s0.t1, s1.t0, s1.t1, a.group);
  int units = wp.nsteps;
  for (int q = 2; q < a.n_q; ++q) {
    const Span s = span(q);
    units += (s.t1 - s.t0) * a.group;
  }
  const int nch = a.split.chunks[it.r] > 1 ? chunks_of(units, a.split.unit, a.split.chunks[it.r]) : 1;
  if (it.chunk == 0 && tid == 0 && a.split.chunks[it.r] > 1) a.split.counts[it.tile] = nch;
  if (it.chunk >= nch) return;
  const int n0 = it.chunk * a.split.unit, n1 = it.chunk + 1 < nch ? n0 + a.split.unit : units;

  const int64_t koff = (((int64_t)it.b * kr.bstride + row0) * HKV + it.kvh) * D;
  stage_row_operands<D>(lds, (const float*)kr.k + koff, HKV * D, nvalid, tid, kWaves * 64);
  stage_row_operands<D>(lds + OPS, (const float*)kr.v + koff, HKV * D, nvalid, tid, kWaves * 64);
  __syncthreads();

  const double c = (double)a.scale * kLog2eD;
  AccTiles<D> dk, dv;
  dk.zero();
  dv.zero();
  for (int n = n0 + w; n < n1; n += kWaves) {
    int q, t, hq;
    Span sp;
    if (n < wp.nsteps) {
      const WalkStep ws = walk_step(wp, n);
      q = ws.q;
      t = ws.s;
      hq = ws.hp;
      sp = q ? s1 : s0;
    } else {
      int m = n - wp.nsteps, size = 0;
      q = 1;
      do {
        m -= size;
        sp = span(++q);
        size = (sp.t1 - sp.t0) * a.group;
      } while (m >= size);
      t = sp.t0 + m / a.group;
      hq = m % a.group;
    }
    const QRangeArg& qr = a.qr[q];
    const int h = it.kvh * a.group + hq;
    int qlo, qhi;  // the queries of the range that see this lane's key
    query_interval(qr.stream, kr.stream, pk, rule_of(a), qlo, qhi);
    qlo = imax(qlo, qr.pos0);
    const int qw = imax(imin(qhi, qr.pos0 + qr.len) - qlo, 0);
    const int64_t hrow = (int64_t)it.b * H + h;
    const int64_t qoff = (((int64_t)it.b * qr.bstride + t * 16) * H + h) * D;
    const int qrows = imin(16, qr.len - t * 16);
    const RowTile qt = row_tile<D>(qr.q, qoff, qrows, H * D), ot = row_tile<D>(qr.dO, qoff, qrows, H * D);
    fl4 qx[NC], ox[NC];
    ColOps<D> cx;
    load_rows<D>(qx, qt, i, g);
    float lse[4], dl[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int row = imin(t * 16 + 4 * r + g, qr.len - 1);
      lse[r] = qr.lse[hrow * qr.bstride + row];
      dl[r] = qr.delta[hrow * qr.len + row];
    }
    const f64x4 s = row_product<D>(qx, lds, lane);
    load_rows<D>(ox, ot, i, g);
    cx.load(ot, i, g);
    const f64x4 dp = row_product<D>(ox, lds + OPS, lane);
    bool dead = false;
#pragma unroll
    for (int r = 0; r < 4; ++r) dead |= lse[r] == -INFINITY;
    const bool full = t * 16 >= sp.i0 && t * 16 + 16 <= sp.i1 && __builtin_amdgcn_ballot_w64(dead) == 0;
    const int qbase = qr.pos0 + t * 16 - qlo;
    auto seen_row = [&](int row) { return full || (unsigned)(qbase + row) < (unsigned)qw; };
    f64x4 p, ds;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const bool see = seen_row(4 * r + g) && lse[r] != -INFINITY;
      p[r] = exp2_f64(see ? __builtin_fma(s[r], c, -(double)lse[r] * kLog2eD) : kHidden);
      ds[r] = p[r] * (see ? dp[r] - (double)dl[r] : 0.0);
    }
    // guarded form: a row that sees no key hides from every column
    auto seen = [&](int row) {
      const float z = qr.lse[hrow * qr.bstride + imin(t * 16 + row, qr.len - 1)];
      return seen_row(row) && z != -INFINITY;
    };
    if (full || !cx.non_finite()) {
      col_product<D>(dv, cx, p);
    } else {
      col_product_guarded<D>(dv, ot, p, seen, i, g);
    }
    cx.load(qt, i, g);
    if (full || !cx.non_finite()) {
      col_product<D>(dk, cx, ds);
    } else {
      col_product_guarded<D>(dk, qt, ds, seen, i, g);
    }
  }

  // Sum the waves through LDS, dV then dK; one chunk writes the gradients,
  // several write fp64 partials [dV, dK][key][d].
  constexpr int EPT = 16 * D / (kWaves * 64);
  const int k = tid / (D / EPT), d0 = (tid % (D / EPT)) * EPT;
#pragma unroll
  for (int which = 0; which < 2; ++which) {
    __syncthreads();
    acc_to_lds<D>(which == 0 ? dv : dk, lds + w * 16 * kRedRow<D>, i, g);
    __syncthreads();
    double x[EPT];
#pragma unroll
    for (int e = 0; e < EPT; ++e) {
      x[e] = 0.0;
#pragma unroll
      for (int u = 0; u < kWaves; ++u) x[e] += lds[(u * 16 + k) * kRedRow<D> + d0 + e];
    }
    if (nch > 1) {
      double* dst = (double*)a.split.partials + partial_row<16>(a, it.b, it.kvh, it.r, it.t, it.chunk) * (2 * D) +
                    (which * nvalid + k) * D + d0;
      if (k < nvalid) {
#pragma unroll
        for (int e = 0; e < EPT; e += 2) *(f64x2*)(dst + e) = f64x2{x[e], x[e + 1]};
      }
    } else if (k < nvalid) {
      float* dst = (float*)(which == 0 ? kr.dv : kr.dk) + koff + (int64_t)k * HKV * D + d0;
      const double sc = which == 0 ? 1.0 : (double)a.scale;
#pragma unroll
      for (int e4 = 0; e4 < EPT / 4; ++e4) {
        fl4 o;
#pragma unroll
        for (int e = 0; e < 4; ++e) o[e] = (float)(x[4 * e4 + e] * sc);
        *(fl4*)(dst + 4 * e4) = o;
      }
    }
  }
}

// dK, dV of the chunked key tiles: the sum of the chunks' partials in chunk
// order.  One workgroup per tile (grid: every tile of the chunked ranges).
template <int D>
__global__ __launch_bounds__(256) void bwd_sum_f32_kernel(const AttnArgs a) {
  constexpr int OPS = 16 * D, EPT = OPS / 256;
  SumItem it;
  sum_item(a, blockIdx.x, it);
  const KRangeArg& kr = a.kr[it.r];
  const int nch = a.split.counts[blockIdx.x];
  if (nch <= 1) return;
  const int nvalid = imin(16, kr.len - it.t * 16);
  const int k = threadIdx.x / (D / EPT), d0 = (threadIdx.x % (D / EPT)) * EPT;
  if (k >= nvalid) return;
  const int64_t off = (((int64_t)it.b * kr.bstride + it.t * 16 + k) * a.kv_heads + it.kvh) * D + d0;
#pragma unroll
  for (int which = 0; which < 2; ++which) {
    double x[EPT] = {};
    for (int ch = 0; ch < nch; ++ch) {
      const double* src = (const double*)a.split.partials +
                          partial_row<16>(a, it.b, it.kvh, it.r, it.t, ch) * (2 * D) + (which * nvalid + k) * D + d0;
#pragma unroll
      for (int e = 0; e < EPT; ++e) x[e] += src[e];
    }
    float* dst = (float*)(which == 0 ? kr.dv : kr.dk) + off;
    const double sc = which == 0 ? 1.0 : (double)a.scale;
#pragma unroll
    for (int e4 = 0; e4 < EPT / 4; ++e4) {
      fl4 o;
#pragma unroll
      for (int e = 0; e < 4; ++e) o[e] = (float)(x[4 * e4 + e] * sc);
      *(fl4*)(dst + 4 * e4) = o;
    }
  }
}

}  // namespace

// a.total_tiles and a.qr's tiles describe 16-row query tiles.
hipError_t launch_bwd_dq_f32(const AttnArgs& a, int head_dim, hipStream_t s) {
  const int n = workgroups_for(a.total_tiles * a.heads * a.batch);
  if (n == 0) return hipSuccess;
  if (head_dim == 128) hipLaunchKernelGGL((bwd_dq_f32_kernel<128>), grid_of(n), dim3(kWaves * 64), 0, s, a);
  else hipLaunchKernelGGL((bwd_dq_f32_kernel<64>), grid_of(n), dim3(kWaves * 64), 0, s, a);
  return hipGetLastError();
}

// a.kr's tiles describe 16-row key tiles; a.split is filled.
hipError_t launch_bwd_dkv_f32(const AttnArgs& a, int head_dim, hipStream_t s) {
  const int n = workgroups_for(a.split.wgs_per_pair * a.kv_heads * a.batch);
  if (n == 0) return hipSuccess;
  if (head_dim == 128) hipLaunchKernelGGL((bwd_dkv_f32_kernel<128>), grid_of(n), dim3(kWaves * 64), 0, s, a);
  else hipLaunchKernelGGL((bwd_dkv_f32_kernel<64>), grid_of(n), dim3(kWaves * 64), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_bwd_sum_f32(const AttnArgs& a, int head_dim, hipStream_t s) {
  const int n = a.split.tiles_per_pair * a.kv_heads * a.batch;
  if (n == 0) return hipSuccess;
  if (head_dim == 128) hipLaunchKernelGGL((bwd_sum_f32_kernel<128>), dim3(n), dim3(256), 0, s, a);
  else hipLaunchKernelGGL((bwd_sum_f32_kernel<64>), dim3(n), dim3(256), 0, s, a);
  return hipGetLastError();
}

}  // namespace bdlm
