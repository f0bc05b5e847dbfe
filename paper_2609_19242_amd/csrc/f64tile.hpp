// fp64 matrix tiles for the fp32 path, gfx950.
//
// fp32 inputs are multiplied and summed in fp64 by v_mfma_f64_16x16x4_f64
// (16x16 tiles, 4 deep; 64 cycles per SIMD, 78 TFLOP/s on the whole chip, with
// two or more independent chains in flight; a stream of v_fma_f64 reaches 58).
// Lane layouts (checked on the GPU), i = lane % 16, g = lane / 16:
//  * A (16x4): lane holds row i, depth g;  B (4x16): depth g, column i;
//    C, register r: row 4 r + g, column i.
// The depth order of a product is free as long as A and B agree, which lets a
// lane read its operands from global memory as float4:
//  * row operands (contraction over head_dim): the float4 at element
//    16 c + 4 g of row i is the lane's operand of products 4 c .. 4 c + 3
//    (product 4 c + e contracts the elements 16 c + 4 g' + e, g' = 0..3);
//  * column operands (contraction over the tile's 16 rows, output rows =
//    head_dim): the float4 at element 64 h + 4 i of row 4 kk + g is the lane's
//    operand of step kk of the four output tiles (h, e), and output tile
//    (h, e), register r, holds head_dim element 64 h + 16 r + 4 g + e.  Step kk
//    contracts rows 4 kk + g', exactly what register kk of a C tile holds.
#pragma once

#include "common.hpp"
#include "device.hpp"

namespace bdlm {

typedef double f64x4 __attribute__((ext_vector_type(4)));
typedef double f64x2 __attribute__((ext_vector_type(2)));
typedef float fl4 __attribute__((ext_vector_type(4)));

constexpr double kLog2eD = 1.4426950408889634074;
constexpr double kLn2D = 0.69314718055994530942;

// c += A B as volatile inline assembly: that keeps the products in source order
// among the operand reads (as builtins, the compiler reads and converts every
// operand of a tile up front, which spills 258 VGPRs).  The s_nop covers the wait states
// between the conversion of an operand and the product that reads it, which
// the compiler does not pad inline assembly for.
__device__ __forceinline__ void mfma64(f64x4& c, double a, double b) {
  asm volatile("s_nop 1\n\tv_mfma_f64_16x16x4_f64 %0, %1, %2, %0" : "+v"(c) : "v"(a), "v"(b));
}
// Before vector code reads results of mfma64: the last product must have left
// the matrix core (19 wait states).  The compiler does not see the product in
// the inline assembly: any use of a result that it may add, a copy or a spill
// included, has to come after such a wait too.
#define BDLM_F64_WAIT "s_nop 15\n\ts_nop 2"

// Sum (or any reduction) partners of a C-layout column: lanes i, i+16, i+32, i+48.
__device__ __forceinline__ double shfl_d(double x, int src) {
  const uint64_t u = __builtin_bit_cast(uint64_t, x);
  const uint32_t lo = (uint32_t)__shfl((int)(uint32_t)u, src), hi = (uint32_t)__shfl((int)(uint32_t)(u >> 32), src);
  return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}
__device__ __forceinline__ double shfl_xor_d(double x, int m) {
  const uint64_t u = __builtin_bit_cast(uint64_t, x);
  const uint32_t lo = (uint32_t)__shfl_xor((int)(uint32_t)u, m), hi = (uint32_t)__shfl_xor((int)(uint32_t)(u >> 32), m);
  return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}
__device__ __forceinline__ double col_sum(double x) {
  x += shfl_xor_d(x, 16);
  return x + shfl_xor_d(x, 32);
}
__device__ __forceinline__ double col_max(double x) {
  x = fmax(x, shfl_xor_d(x, 16));
  return fmax(x, shfl_xor_d(x, 32));
}

// 2^t in fp64: t = n + f with n the nearest integer, 2^f by its Taylor series
// in f ln 2 to degree 13 (|f ln 2| <= 0.347: the remainder is below 2^-56),
// scaled by 2^n.  Infinite t give 0 and infinity, NaN stays NaN.
constexpr double kHidden = -2000.0;  // the exponent of a hidden pair: 2^kHidden is 0
__device__ __forceinline__ double exp2_f64(double t) {
  t = t > 1100.0 ? 1100.0 : t;
  t = t < -1100.0 ? -1100.0 : t;
  const double n = __builtin_rint(t);
  const double x = (t - n) * kLn2D;
  double p = 1.0 / 6227020800.0;
  p = __builtin_fma(p, x, 1.0 / 479001600.0);
  p = __builtin_fma(p, x, 1.0 / 39916800.0);
  p = __builtin_fma(p, x, 1.0 / 3628800.0);
  p = __builtin_fma(p, x, 1.0 / 362880.0);
  p = __builtin_fma(p, x, 1.0 / 40320.0);
  p = __builtin_fma(p, x, 1.0 / 5040.0);
  p = __builtin_fma(p, x, 1.0 / 720.0);
  p = __builtin_fma(p, x, 1.0 / 120.0);
  p = __builtin_fma(p, x, 1.0 / 24.0);
  p = __builtin_fma(p, x, 1.0 / 6.0);
  p = __builtin_fma(p, x, 0.5);
  p = __builtin_fma(p, x, 1.0);
  p = __builtin_fma(p, x, 1.0);
  return __builtin_ldexp(p, (int)n);
}

// A tile of 16 rows held in LDS as fp64 row operands, in the order the
// products consume them: product n of lane l is element (n * 64 + l) of pairs
// of products, [n / 2][l][n % 2].
template <int D>
__device__ __forceinline__ void stage_row_operands(double* dst, const float* rows, int64_t row_stride, int nrows,
                                                   int tid, int nthreads) {
  for (int it = tid; it < 64 * (D / 16); it += nthreads) {
    const int lane = it & 63, c = it >> 6, i = lane & 15, g = lane >> 4;
    const fl4 x = *(const fl4*)(rows + (int64_t)imin(i, nrows - 1) * row_stride + 16 * c + 4 * g);
#pragma unroll
    for (int e = 0; e < 4; ++e) dst[((2 * c + (e >> 1)) * 64 + lane) * 2 + (e & 1)] = (double)x[e];
  }
}

// C = A B over head_dim, A from the lane's row operand registers, B from LDS
// (stage_row_operands).  Two chains, so that a lone wave keeps the matrix core
// busy.
template <int D>
__device__ __forceinline__ f64x4 row_product(const fl4 (&x)[D / 16], const double* b, int lane) {
  constexpr int NC = D / 16;
  f64x4 c0 = {0, 0, 0, 0}, c1 = {0, 0, 0, 0};
  // B is read one step ahead; the address laundered at each step keeps the
  // compiler from reading all of B up front or keeping it over the walk.
  uint32_t at = lds_addr(b) + 16u * lane;
  f64x2 q[2][2];
  auto read = [&](int c) __attribute__((always_inline)) {
    asm volatile("" : "+v"(at));
    typedef __attribute__((address_space(3))) const f64x2* lp;
    q[c & 1][0] = *(lp)(uintptr_t)(at + 2048u * c);
    q[c & 1][1] = *(lp)(uintptr_t)(at + 2048u * c + 1024u);
  };
  read(0);
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    if (c + 1 < NC) read(c + 1);
    mfma64(c0, (double)x[c][0], q[c & 1][0][0]);
    mfma64(c1, (double)x[c][1], q[c & 1][0][1]);
    mfma64(c0, (double)x[c][2], q[c & 1][1][0]);
    mfma64(c1, (double)x[c][3], q[c & 1][1][1]);
  }
  asm volatile(BDLM_F64_WAIT : "+v"(c0), "+v"(c1));
  return c0 + c1;
}

// A tile of up to 16 rows in global memory: element 0 of its first row, the
// bytes to the end of its last row (later rows read as zeros) and the row
// stride in bytes.  Wave-uniform.
struct RowTile {
  __amdgpu_buffer_rsrc_t rsrc;
  uint32_t stride;
};
template <int D>
__device__ __forceinline__ RowTile row_tile(const void* base, int64_t first_row_elem, int nrows, int64_t row_elems) {
  return RowTile{make_rsrc((const float*)base + first_row_elem, (uint32_t)(((int64_t)(nrows - 1) * row_elems + D) * 4)),
                 (uint32_t)(row_elems * 4)};
}
// (the row's offset is part of voff: a scalar offset takes no part in the bounds check)
__device__ __forceinline__ fl4 buf_f4(__amdgpu_buffer_rsrc_t r, uint32_t voff) {
  return __builtin_bit_cast(fl4, __builtin_amdgcn_raw_buffer_load_b128(r, voff, 0, 0));
}
// The lane's row operands (row i).
template <int D>
__device__ __forceinline__ void load_rows(fl4 (&x)[D / 16], const RowTile& t, int i, int g) {
  uint32_t off = (uint32_t)i * t.stride + 16u * g;
  asm volatile("" : "+v"(off));  // (keeps the loads at this place among the products)
#pragma unroll
  for (int c = 0; c < D / 16; ++c) x[c] = buf_f4(t.rsrc, off + 64 * c);
}
// The lane's column operands (rows 4 kk + g).
template <int D>
struct ColOps {
  fl4 x[4][D / 64];
  __device__ __forceinline__ void load(const RowTile& t, int i, int g) {
    uint32_t off = (uint32_t)g * t.stride + 16u * i;
    asm volatile("" : "+v"(off));  // (keeps the loads at this place among the products)
#pragma unroll
    for (int kk = 0; kk < 4; ++kk)
#pragma unroll
      for (int h = 0; h < D / 64; ++h) x[kk][h] = buf_f4(t.rsrc, off + 4u * kk * t.stride + 256 * h);
  }
  // Does the tile hold an infinity or NaN?  (wave-uniform)
  __device__ __forceinline__ bool non_finite() const {
    bool bad = false;
#pragma unroll
    for (int kk = 0; kk < 4; ++kk)
#pragma unroll
      for (int h = 0; h < D / 64; ++h)
#pragma unroll
        for (int e = 0; e < 4; ++e) bad |= !__builtin_isfinite(x[kk][h][e]);
    return __builtin_amdgcn_ballot_w64(bad) != 0;
  }
};

// Accumulators of 16 columns x D head_dim elements: tile (h, e), see above.
template <int D>
struct AccTiles {
  f64x4 t[D / 16];
  __device__ __forceinline__ void zero() {
#pragma unroll
    for (int n = 0; n < D / 16; ++n) t[n] = f64x4{0, 0, 0, 0};
  }
  // Before vector code reads the accumulators (one wait for all of them).
  __device__ __forceinline__ void done() {
    if constexpr (D == 128)
      asm volatile(BDLM_F64_WAIT
                   : "+v"(t[0]), "+v"(t[1]), "+v"(t[2]), "+v"(t[3]), "+v"(t[4]), "+v"(t[5]), "+v"(t[6]), "+v"(t[7]));
    else
      asm volatile(BDLM_F64_WAIT : "+v"(t[0]), "+v"(t[1]), "+v"(t[2]), "+v"(t[3]));
  }
  __device__ __forceinline__ void scale(double s) {
    done();
#pragma unroll
    for (int n = 0; n < D / 16; ++n) t[n] = t[n] * s;
  }
};

// acc[d][column] += sum over the tile's 16 rows of X[row][d] w[row][column],
// w in C layout.  Ends with the wait for its products: where its callers' paths
// meet (col_product_guarded), the compiler copies or spills accumulators.
template <int D>
__device__ __forceinline__ void col_product(AccTiles<D>& acc, const ColOps<D>& x, const f64x4& w) {
#pragma unroll
  for (int kk = 0; kk < 4; ++kk)
#pragma unroll
    for (int h = 0; h < D / 64; ++h) {
#pragma unroll
      for (int e = 0; e < 4; ++e) mfma64(acc.t[4 * h + e], (double)x.x[kk][h][e], w[kk]);
    }
  acc.done();
}

// The same for a tile holding non-finite operands and hidden (row, column)
// pairs: in vector code, one row at a time, so that 0 * inf of a hidden pair
// does not reach the column.  vis(row): does this lane's column see the row?
template <int D, class Vis>
__device__ __forceinline__ void col_product_guarded(AccTiles<D>& acc, const RowTile& t, const f64x4& w, Vis&& vis,
                                                    int i, int g) {
  acc.done();
#pragma unroll 1
  for (int row = 0; row < 16; ++row) {
    const int kk = row >> 2;
    const double mine = kk == 0 ? w[0] : kk == 1 ? w[1] : kk == 2 ? w[2] : w[3];
    const double p = shfl_d(mine, 16 * (row & 3) + i);
    const bool seen = vis(row);
#pragma unroll
    for (int h = 0; h < D / 64; ++h)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const fl4 v = buf_f4(t.rsrc, (uint32_t)row * t.stride + 4u * (64 * h + 16 * r + 4 * g));
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const double old = acc.t[4 * h + e][r];
          acc.t[4 * h + e][r] = seen ? __builtin_fma(p, (double)v[e], old) : old;
        }
      }
  }
}

// Rows of the LDS area in which the waves' accumulators are summed: D + 2
// doubles apart, so that the 16 columns of a wave start in different banks.
template <int D>
constexpr int kRedRow = D + 2;

// Workgroup ids of a launch of n workgroups that may need two grid dimensions
// (a dimension holds fewer than 2^32 threads; 16-row tiles make many
// workgroups): rows of 2^23 workgroups, a multiple of the 8 XCDs.
constexpr int kGridRow = 1 << 23;
inline dim3 grid_of(int n) { return n <= kGridRow ? dim3(n) : dim3(kGridRow, (n + kGridRow - 1) / kGridRow); }
__device__ __forceinline__ int workgroup_id() { return (int)(blockIdx.y * (unsigned)kGridRow + blockIdx.x); }

template <int D>
__device__ __forceinline__ void acc_to_lds(AccTiles<D>& acc, double* dst, int i, int g) {
  acc.done();
#pragma unroll
  for (int h = 0; h < D / 64; ++h)
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
      for (int e2 = 0; e2 < 2; ++e2)
        *(f64x2*)(dst + i * kRedRow<D> + 64 * h + 16 * r + 4 * g + 2 * e2) =
            f64x2{acc.t[4 * h + 2 * e2][r], acc.t[4 * h + 2 * e2 + 1][r]};
}

}  // namespace bdlm
