// BDLM attention forward for fp32 inputs (fp32 in, fp32 out), gfx950.
//
// Scores, exponentials and sums are carried in fp64, so that the only rounding
// left is the final cast; the two products run on the fp64 matrix cores
// (f64tile.hpp).  A workgroup of four waves owns 16 query rows of one head and
// walks the 16-key tiles that any of them sees (the mask rules of common.hpp;
// arXiv 2609.19242 Sec. 3.2), the tiles dealt out to the waves in turn.  Each
// wave keeps its own online softmax (running max, row sums, O^T accumulators),
// and the four are merged through LDS at the end.  Dealing keys, not query
// rows, to the waves keeps a short problem's walk a quarter as long: fp32
// problems are small, and 16 rows per workgroup are what gives the chip enough
// of them.  K and V go straight from global memory (L2) into registers as
// float4 operands: a wave needs 16 KB per 64 matrix products of 64 cycles
// each, well below what the L1 delivers, so nothing is staged.
// Bound by the fp64 matrix rate, on small problems by the walk's latency.
// Measured against one thread per row with a serial fp64 chain per key:
// L = 256, 2/2 heads, d 64: 402 -> 17 us; L = 1125, 8/2 heads, d 128: 6.1 ms
// -> 0.15 ms (35 TFLOP/s).  (At head_dim 128 six VGPRs are spilled.)
// Output: normalised O and natural-log LSE; a row that sees no key gets O = 0
// and LSE = -inf.
#include "f64tile.hpp"
#include "qtiles.hpp"

namespace bdlm {

namespace {

constexpr int kWaves = 4;
// The running max of a row moves only when a score exceeds it by this much (in
// powers of two): p and the sums stay far below the fp64 range, and their
// relative precision does not depend on the reference.
constexpr double kRescale = 256.0;

template <int D>
__global__ __launch_bounds__(kWaves * 64) __attribute__((amdgpu_waves_per_eu(2, 2))) void fwd_f32_kernel(
    const AttnArgs a) {
  constexpr int NC = D / 16;
  // Q as fp64 row operands during the walk, the waves' O^T sums after it
  __shared__ __attribute__((aligned(16))) double lds[kWaves * 16 * kRedRow<D>];
  __shared__ double red_m[kWaves][16], red_l[kWaves][16];
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
  __syncthreads();

  const int pq = qr.pos0 + row0 + imin(i, nvalid - 1);  // this lane's query (a column of S^T)
  const int pq0 = qr.pos0 + row0, pq1 = qr.pos0 + row0 + nvalid - 1;
  const double c = (double)a.scale * kLog2eD;

  AccTiles<D> acc;
  acc.zero();
  double m = -INFINITY, l = 0.0;
  fl4 kx[NC];

  // This wave's tiles: every kWaves-th of the visible tiles of all key ranges.
  int j = -1, t = 0, t1 = 0, f0 = 0, f1 = 0, skip = w;
  auto advance = [&]() __attribute__((always_inline)) -> bool {
    t += kWaves;
    while (t >= t1) {
      if (j >= 0) skip = t - t1;  // tiles still to pass over in the next range
      if (++j >= a.n_k) return false;
      key_tile_span(a, j, qr.stream, pq0, pq1, 16, t, t1, f0, f1);
      t += skip;
    }
    return true;
  };
  auto tile_of = [&](const void* base) __attribute__((always_inline)) {
    const KRangeArg& kr = a.kr[j];
    return row_tile<D>(base, (((int64_t)it.b * kr.bstride + t * 16) * HKV + kvh) * D, imin(16, kr.len - t * 16),
                       HKV * D);
  };
  t = t1 = -kWaves;  // the first call starts with range 0
  bool have = advance();
  if (have) load_rows<D>(kx, tile_of(a.kr[j].k), i, g);
  while (have) {
    const KRangeArg& kr = a.kr[j];
    const int tt = t;
    const bool full = tt >= f0 && tt < f1;
    const RowTile vt = tile_of(kr.v);
    ColOps<D> vx;
    vx.load(vt, i, g);
    int lo = 0, wid = 0;
    if (!full) lane_key_interval(a, j, qr.stream, pq, lo, wid);
    const int kbase = kr.pos0 + tt * 16 - lo;
    auto seen = [&](int row) { return full || (unsigned)(kbase + row) < (unsigned)wid; };

    f64x4 s = row_product<D>(kx, lds, lane) * c;
    // the next tile's K loads run under the softmax and the products below
    have = advance();
    if (have) load_rows<D>(kx, tile_of(a.kr[j].k), i, g);

    bool grow = false;
#pragma unroll
    for (int r = 0; r < 4; ++r) grow |= seen(4 * r + g) && !(s[r] <= m + kRescale);
    if (__builtin_amdgcn_ballot_w64(grow) != 0) {
      double mx = -INFINITY;
#pragma unroll
      for (int r = 0; r < 4; ++r) mx = seen(4 * r + g) ? fmax(mx, s[r]) : mx;
      const double mn = fmax(m, col_max(mx));
      const double al = m == -INFINITY ? 0.0 : exp2_f64(m - mn);
      l *= al;
      acc.scale(al);
      m = mn;
    }
    f64x4 p;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      p[r] = exp2_f64(seen(4 * r + g) ? s[r] - m : kHidden);
      l += p[r];
    }
    // hidden keys must not spread an infinity or NaN of V to rows that do not see them
    if (full || !vx.non_finite()) col_product<D>(acc, vx, p);
    else col_product_guarded<D>(acc, vt, p, seen, i, g);
  }

  // Merge the waves: common reference max, scaled sums.
  l = col_sum(l);
  if (g == 0) {
    red_m[w][i] = m;
    red_l[w][i] = l;
  }
  __syncthreads();  // also: every wave has left the walk, Q is no longer read
  double mt = red_m[0][i];
#pragma unroll
  for (int k = 1; k < kWaves; ++k) mt = fmax(mt, red_m[k][i]);
  acc.scale(m == -INFINITY ? 0.0 : exp2_f64(m - mt));
  acc_to_lds<D>(acc, lds + w * 16 * kRedRow<D>, i, g);
  __syncthreads();
  constexpr int EPT = 16 * D / (kWaves * 64);  // elements per thread
  const int q = tid / (D / EPT), d0 = (tid % (D / EPT)) * EPT;
  double M = red_m[0][q], lt = 0.0;
#pragma unroll
  for (int k = 1; k < kWaves; ++k) M = fmax(M, red_m[k][q]);
#pragma unroll
  for (int k = 0; k < kWaves; ++k) lt += red_m[k][q] == -INFINITY ? 0.0 : red_l[k][q] * exp2_f64(red_m[k][q] - M);
  const bool empty = !(lt > 0.0);
  const double inv = empty ? 0.0 : 1.0 / lt;
  if (q < nvalid) {
    float* op = (float*)qr.o + qoff + (int64_t)q * H * D + d0;
#pragma unroll
    for (int e4 = 0; e4 < EPT / 4; ++e4) {
      fl4 o;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        double x = 0.0;
#pragma unroll
        for (int k = 0; k < kWaves; ++k) x += lds[(k * 16 + q) * kRedRow<D> + d0 + 4 * e4 + e];
        o[e] = (float)(x * inv);
      }
      *(fl4*)(op + 4 * e4) = o;
    }
    if (d0 == 0)
      qr.lse[((int64_t)it.b * H + it.h) * qr.bstride + row0 + q] =
          empty ? -INFINITY : (float)((M + log2(lt)) * kLn2D);
  }
}

}  // namespace

hipError_t launch_fwd_f32(const AttnArgs& a, int head_dim, hipStream_t s) {
  const int n = workgroups_for(a.total_tiles * a.heads * a.batch);
  if (n == 0) return hipSuccess;
  if (head_dim == 128)
    hipLaunchKernelGGL((fwd_f32_kernel<128>), grid_of(n), dim3(kWaves * 64), 0, s, a);
  else
    hipLaunchKernelGGL((fwd_f32_kernel<64>), grid_of(n), dim3(kWaves * 64), 0, s, a);
  return hipGetLastError();
}

}  // namespace bdlm
