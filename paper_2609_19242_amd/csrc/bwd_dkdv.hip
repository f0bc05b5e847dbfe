// dK and dV of the BDLM attention backward, key-major, bf16 inputs, fp32
// accumulation, gfx950: the software-pipelined kernel (single-term or adaptive
// two-term products, at most two query ranges).
//
// Exact gradients from the saved O and LSE (arXiv 2609.19242 App. C fused
// backward; eq:correctness-corrupted-gradient and eq:correctness-clean-gradient):
// with P = exp(scale Q K^T + mask - LSE) and D = rowsum(dO * O),
//   dV = P^T dO,  dS = P * (dO V^T - D),  dK = scale dS^T Q,
// summed over every query row that sees a key and over the query heads of the
// key's GQA group.  dQ comes from the query-major kernel (bwd_dq.hip).
//
// A workgroup owns 128 keys of one KV head (4 waves x 32 keys), holds their K
// and V rows in AGPRs as MFMA operands and accumulates dK^T and dV^T in AGPRs
// over its walk (or chunk of a walk, ktiles.hpp) of visible query steps.  A
// step is two sub-blocks of 32 query rows: the same rows of two query heads of
// an even GQA group, or 64 rows of one head of an odd one.
//
// At head_dim 128 one wave per SIMD fits (384 registers), and nothing else
// hides a wave's own dependency chain S, dP -> softmax -> dV, dK, so the step
// is written as four blocks of 16 matrix products each (8 at head_dim 64),
// with the vector and scalar work placed under them and the order fixed by
// scheduling fences (heads 0, 1 here: the sub-blocks):
//   A: S_0 = Q_0 K^T, dP_0 = dO_0 V^T (head 0)  under  the LDS-DMA copies of
//      the step three ahead and the copy plan of the step after
//   B: S_1, dP_1 (head 1)      under  P_0 = exp2(c S_0), dS_0 = P_0 dP_0, and
//      the first operand reads of C
//   C: dV += dO_0^T P_0, dK += Q_0^T dS_0   under  P_1 = exp2(c S_1)
//   D: dV += dO_1^T P_1, dK += Q_1^T dS_1   under  dS_1 = P_1 dP_1, the next
//      step's accumulator starts, and its first row reads (issued before the
//      step's barrier: that stage is complete from the barrier before)
// Row operands are read four products ahead, transpose operands eight (at
// head_dim 64 two and four, in the two-term forms one and two: at most 252
// registers, so two workgroups share a CU; the two-term form on odd groups
// takes 280 and runs alone).  The walk's bookkeeping is vector work: the descriptors of 64 steps (block,
// range, partial flag, copy resource words) sit in the lanes of a few VGPRs,
// computed every 56 steps from a closed form (walk_plan, walk_step), and a
// step reads its own with readlane, so a step issues about 27 scalar
// instructions where a scalar cursor took over a hundred.
// S and dP accumulate on top of -LSE/scale and -D read from LDS (the dQ
// kernel, which runs first, writes that form), so the softmax is one multiply
// and one exp2 per score and dS one multiply; rows the mask hides start at
// -inf.  LDS holds four stages, filled by LDS-DMA copies three steps ahead,
// so the next step's data is resident while a step runs; the copies are
// issued as inline assembly, which keeps the compiler from waiting on them
// before every LDS transpose read (it cannot tell which stage a DMA writes).
// The dV/dK products are inline-assembly MFMAs on AGPR accumulators (the S/dP
// products use VGPR accumulators, which the softmax reads).
// Bound by the matrix cores (and, at head_dim 64, the exponentials: one per
// product).  Measured against the general kernel of bwd_bf16.hip: 4K, batch 2,
// 32/8 heads, head_dim 64: 790 -> 590 us (whole walks 630; one wave per SIMD
// with the longer read-ahead 612); 3,000 tokens, 16/16 heads: 211 -> 179 us.
#include "common.hpp"
#include "device.hpp"
#include "ktiles.hpp"

namespace bdlm {

namespace {

constexpr int kSub = 32;     // query rows of a sub-block: a step is two of them
constexpr int kStages = 4;

// Shapes of one instantiation.  D: head_dim.  ROWS false: the two sub-blocks
// of a step are the same 32 rows of two query heads (even GQA groups); true:
// 64 consecutive rows of one head (odd groups).
template <int D, bool ROWS>
struct Shape {
  static constexpr int KS = D / 16;               // k-steps of 16 in a score product
  static constexpr int DT = D / 32;               // 32-wide d tiles of dK^T / dV^T
  static constexpr int BM = ROWS ? 2 * kSub : kSub;  // query rows per step
  static constexpr int HPS = ROWS ? 1 : 2;        // query heads per step
  static constexpr uint32_t RB = D * 2;           // bytes per row
  static constexpr uint32_t HB = kSub * RB;       // bytes per sub-block in a stage tile (8 KB at D = 128)
  static constexpr uint32_t TileB = 2 * HB;       // Q (or dO) tile of a stage (16 KB)
  // LDS: the four Q tiles, then the four dO tiles (each region 64 KB at D =
  // 128, so every read address is a per-lane register plus an immediate offset
  // below 2^16), then per stage -LSE/scale and -D of the step's 2 x 32 rows.
  static constexpr uint32_t QRegion = 0;
  static constexpr uint32_t DoRegion = kStages * TileB;
  static constexpr uint32_t StatRegion = 2 * kStages * TileB;
  static constexpr uint32_t StatB = 2 * 2 * kSub * 4;                   // 512 bytes per stage
  static constexpr uint32_t SpareRegion = StatRegion + kStages * StatB;  // empty copies of waves 0, 1
  static constexpr uint32_t LdsBytes = SpareRegion + 2 * 256;            // 133632 at D = 128, 68096 at D = 64
  // Copy plan: a tensor tile of a step is 64 rows x D / 8 16-byte slots;
  // waves 0-1 copy Q, waves 2-3 dO, IPW instructions of 64 lanes each; one
  // more dword instruction per wave copies the 64 floats of -LSE/scale (wave
  // 2) or -D (wave 3) (waves 0, 1: an empty copy).
  static constexpr int IPW = 64 * (D / 8) / 64 / 2;
};

__device__ __forceinline__ void mfma_agpr(f32x16& acc, const bf16x8& a, const bf16x8& b) {
  asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+a"(acc) : "v"(a), "v"(b));
}
// The same with the two wait states a VALU write of an operand needs before an
// MFMA reads it (the compiler does not pad inline assembly for it).
__device__ __forceinline__ void mfma_agpr_padded(f32x16& acc, const bf16x8& a, const bf16x8& b) {
  asm volatile("s_nop 1\n\tv_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+a"(acc) : "v"(a), "v"(b));
}

// Buffer resource as four SGPRs for the inline-assembly copies.
__device__ __forceinline__ u32x4 rsrc_words(const void* base, uint32_t bytes) {
  const uint64_t p = (uint64_t)(uintptr_t)base;
  u32x4 r;
  r[0] = (uint32_t)p;
  r[1] = (uint32_t)(p >> 32) & 0xffffu;
  r[2] = bytes;
  r[3] = 0x00020000u;
  return r;
}
// Global -> LDS copy: lane i's 16 (or 4) bytes at voff land at LDS byte
// address m0 + 16 i (4 i); offsets past the resource's end write zeros.
__device__ __forceinline__ void dma16(u32x4 rsrc, uint32_t lds_byte, uint32_t voff) {
  asm volatile("s_nop 0\n\tbuffer_load_dwordx4 %0, %1, 0 offen lds" ::"v"(voff), "s"(rsrc), "{m0}"(lds_byte)
               : "memory");
}
__device__ __forceinline__ void dma4(u32x4 rsrc, uint32_t lds_byte, uint32_t voff) {
  asm volatile("s_nop 0\n\tbuffer_load_dword %0, %1, 0 offen lds" ::"v"(voff), "s"(rsrc), "{m0}"(lds_byte)
               : "memory");
}

__device__ __forceinline__ void fence() { __builtin_amdgcn_sched_barrier(0); }

__device__ __forceinline__ f32x4 lds_f4(uint32_t a) {
  return *(__attribute__((address_space(3))) const f32x4*)(uintptr_t)a;
}

// Descriptors of step i of a key tile's walk (walk_step): its row block,
// q | partial << 1, and words 0-2 of the buffer resources of its tensor rows
// (BM rows x HPS heads from block s of range q, head group hp) and of its
// statistics row; steps past the end copy nothing and are not partial.  Plain
// scalar parameters: as a lambda over captured variables, the compiler turned
// the per-lane selects into indexed loads from a stack copy of the captures.
struct StepDesc {
  int s, flags;
  uint32_t t0, t1, t2, l0, l1, l2;
};
template <int D, bool ROWS>
__device__ __forceinline__ StepDesc step_desc(const WalkPlan& wp, int i, int64_t H, bool stats_wave, int len_0,
                                              int len_1, int f0_0, int f0_1, int f1_0, int f1_1, uint32_t lrec_0,
                                              uint32_t lrec_1, uint64_t tb_0, uint64_t tb_1, uint64_t lb_0,
                                              uint64_t lb_1) {
  constexpr int BM = Shape<D, ROWS>::BM, NH = Shape<D, ROWS>::HPS;
  const WalkStep ws = walk_step(wp, i);
  const bool live = ws.live;
  const int q = live ? ws.q : 0;
  const int blk = ws.s;
  const int row0 = live ? blk * BM : 0;
  const int len = q ? len_1 : len_0;
  const int nrows = imin(BM, len - row0);
  const int hoff = ws.hp * NH;
  StepDesc d;
  d.s = blk;
  const bool part = live && !(blk >= (q ? f0_1 : f0_0) && blk < (q ? f1_1 : f1_0));
  d.flags = q | (part ? 2 : 0);
  const uint64_t tp = (q ? tb_1 : tb_0) + (uint64_t)(((int64_t)row0 * H + hoff) * D * 2);
  d.t0 = (uint32_t)tp;
  d.t1 = (uint32_t)(tp >> 32) & 0xffffu;
  d.t2 = live ? (uint32_t)((nrows - 1) * (int)H + NH) * D * 2 : 0u;
  const int loff = live ? hoff * len + row0 : 0;
  const uint64_t lp = (q ? lb_1 : lb_0) + (uint64_t)loff * 4u;
  d.l0 = (uint32_t)lp;
  d.l1 = (uint32_t)(lp >> 32) & 0xffffu;
  d.l2 = (live && stats_wave) ? (q ? lrec_1 : lrec_0) - (uint32_t)loff * 4u : 0u;
  return d;
}

// ADAPT: a step also carries P - bf16(P) and dS - bf16(dS) of a head's
// 16-row half as second bf16 terms when some probability of that half reaches
// hilo_tau (8 more products: head 0's after block B, head 1's after block D,
// each while its P and dS are still in registers).
template <int D, bool ADAPT, bool ROWS>
__global__ __launch_bounds__(256) void dkdv_kernel(const AttnArgs a) {
  using Sh = Shape<D, ROWS>;
  constexpr int BN = kBwdKeysBf16, BM = Sh::BM, HPS = Sh::HPS, KS = Sh::KS, DT = Sh::DT, IPW = Sh::IPW;
  constexpr uint32_t RB = Sh::RB, HB = Sh::HB, TileB = Sh::TileB;
  static_assert(BN == 128, "tile shape");
  __shared__ __attribute__((aligned(1024))) unsigned char lds[Sh::LdsBytes];
  const uint32_t L0 = lds_addr(lds);

  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, half = lane >> 5;
  const int G = lane >> 4, sl = lane & 15;
  const int64_t H = a.heads, HKV = a.kv_heads;

  // ---- work item: (batch, KV head, key range, key tile, chunk of its walk); heaviest tiles first per XCD
  KeyTileItem it;
  if (!key_tile_item(a, blockIdx.x, it)) return;
  const int b = it.b, kvh = it.kvh, r = it.r, t = it.t;
  const KRangeArg& kr = a.kr[r];
  const int key0 = t * BN;
  const int nk = imin(BN, kr.len - key0);
  const bool ragged = nk < BN;
  const int mykey = w * 32 + l32;
  const bool key_ok = mykey < nk;
  const int pk = kr.pos0 + key0 + imin(mykey, nk - 1);
  const int kpos_first = kr.pos0 + key0, kpos_last = kr.pos0 + key0 + nk - 1;

  // ---- K, V rows of this wave's keys (B operands of the score products), in AGPRs
  bf16x8 kf[KS], vf[KS];
  {
    const int64_t eoff = (((int64_t)b * kr.bstride + key0) * HKV + kvh) * D;
    const uint32_t bytes = (uint32_t)(((int64_t)(nk - 1) * HKV * D + D) * 2);
    const auto rk = make_rsrc((const bf16*)kr.k + eoff, bytes);
    const auto rv = make_rsrc((const bf16*)kr.v + eoff, bytes);
    const uint32_t off = (uint32_t)(((int64_t)mykey * HKV * D + 8 * half) * 2);
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      kf[s] = __builtin_bit_cast(bf16x8, buf_load16(rk, off + 32 * s));
      vf[s] = __builtin_bit_cast(bf16x8, buf_load16(rv, off + 32 * s));
    }
  }
  // dK^T / dV^T accumulators (AGPRs, written only by the inline-assembly MFMAs)
  f32x16 dka[DT], dva[DT];
#pragma unroll
  for (int d = 0; d < DT; ++d) {
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      dka[d][i] = 0.f;
      dva[d][i] = 0.f;
    }
    asm volatile("" : "+a"(dka[d]), "+a"(dva[d]));
  }

  // ---- walk over (query range, head pair, step), steps from the end of the
  // ranges down (every range active at a step index, then the next index);
  // the call passes at most two query ranges (the ones with rows).
  struct Span {
    int s0, s1, f0, f1, pos0, qa, qw, len;
    const bf16* tb;
    const float* lb;
    uint32_t lrec;
  };
  auto make_span = [&](int q) __attribute__((always_inline)) -> Span {
    Span sp{0, 0, 0, 0, 0, 0, 0, 0, nullptr, nullptr, 0u};
    if (q >= a.n_q) return sp;
    const QRangeArg& qr = a.qr[q];
    sp.pos0 = qr.pos0;
    sp.len = qr.len;
    const int h0 = kvh * a.group;
    sp.tb = (const bf16*)(w < 2 ? qr.q : qr.dO) + ((int64_t)b * qr.bstride * H + h0) * D;
    const int64_t lrow = ((int64_t)b * H + h0) * qr.len;
    sp.lb = (w == 2 ? qr.l2 : qr.delta) + lrow;
    sp.lrec = (uint32_t)(((int64_t)a.batch * H * qr.len - lrow) * 4);
    int lo0, hi0, lo1, hi1;
    query_interval(qr.stream, kr.stream, kpos_first, rule_of(a), lo0, hi0);
    query_interval(qr.stream, kr.stream, kpos_last, rule_of(a), lo1, hi1);
    const int u0 = imax(lo0 - qr.pos0, 0), u1 = imin(hi1 - qr.pos0, qr.len);
    if (u1 > u0) {
      sp.s0 = u0 / BM;
      sp.s1 = (u1 + BM - 1) / BM;
      const int i0 = imax(lo1 - qr.pos0, 0), i1 = imin(hi0 - qr.pos0, qr.len);
      if (i1 > i0 && !ragged) {
        sp.f0 = (i0 + BM - 1) / BM;
        sp.f1 = i1 / BM;
      }
    }
    int lo, hi;
    query_interval(qr.stream, kr.stream, pk, rule_of(a), lo, hi);
    lo = imax(lo, qr.pos0);
    hi = imin(hi, qr.pos0 + qr.len);
    sp.qa = lo;
    sp.qw = key_ok ? imax(hi - lo, 0) : 0;
    return sp;
  };
  const Span R0 = make_span(0), R1 = make_span(1);
  auto sel2 = [](int q, auto v0, auto v1) { return q ? v1 : v0; };
#define BDLM_PICK(f, q) sel2((q), R0.f, R1.f)
  // The walk by step index (walk_plan, walk_step).
  WalkPlan wp = walk_plan(R0.s0, R0.s1, R1.s0, R1.s1, a.group / HPS);
  // This workgroup's chunk of it: steps [n0, n1).
  const int max_ch = a.split.chunks[r];
  const int nch = max_ch > 1 ? chunks_of(wp.nsteps, a.split.unit, max_ch) : 1;
  if (max_ch > 1 && it.chunk == 0 && tid == 0) a.split.counts[it.tile] = nch;
  if (it.chunk >= nch) return;
  const int n0 = it.chunk * a.split.unit, n1 = it.chunk + 1 < nch ? n0 + a.split.unit : wp.nsteps;
  wp.nsteps = n1;  // (steps past the chunk copy nothing)
  // At head_dim 128 the epilogue's scalars wait in VGPRs, of which the walk
  // leaves some free (it needs every SGPR: spilled ones, read back each step,
  // cost 2% at 32K).
  uint64_t partial_at =
      nch > 1 ? (uint64_t)(uintptr_t)a.split.partials + (uint64_t)partial_row<BN>(a, b, kvh, r, t, it.chunk) * (2 * D * 4)
              : 0;
  if constexpr (D == 128) {
    asm volatile("" : "+v"(partial_at));
    // So does the walk's plan, which only the (vector) step descriptors read.
    asm volatile("" : "+v"(wp.p0), "+v"(wp.p1), "+v"(wp.p2), "+v"(wp.p3), "+v"(wp.st1), "+v"(wp.st2), "+v"(wp.nsteps));
    asm volatile("" : "+v"(wp.cnt0), "+v"(wp.cnt1), "+v"(wp.cnt2), "+v"(wp.q00), "+v"(wp.q01), "+v"(wp.q02),
                      "+v"(wp.npairs));
  }

  // ---- copies.  Instruction i of a wave is instruction (w & 1) * IPW + i of
  // its tensor; the per-lane global offsets are constant over the walk.
  const int wodd = w & 1;
  uint32_t voff[IPW];
#pragma unroll
  for (int i = 0; i < IPW; ++i) {
    const int slot = (wodd * IPW + i) * 64 + lane;
    const int row = slot / (D / 8), ch = (slot % (D / 8)) ^ chunk_swz<D>(row);
    const int head = ROWS ? 0 : row / kSub, rr = ROWS ? row : row % kSub;
    voff[i] = (uint32_t)(((rr * H + head) * D + ch * 8) * 2);
  }
  // A step's copies: IPW 16-byte instructions of the wave's tensor and one
  // dword instruction of -LSE/scale (wave 2) or -D (wave 3); waves 0 and 1
  // issue an empty dword copy into a spare LDS row instead, so that every wave
  // has IPW + 1 copies per step in flight.
  struct CopyPlan {
    u32x4 rt, rl;   // resources: the wave's tensor rows, its -LSE/scale or -D row
    uint32_t lvo;   // per-lane offset of the dword copy
  };
  // Step descriptors, 64 steps at a time: lane l of a batch holds step
  // base + l (step_desc); a step reads them back with one readlane each.
  // Steps past the walk's end copy nothing (zero-size resources) and are not
  // partial.
  const int len_0 = R0.len, len_1 = R1.len, f0_0 = R0.f0, f0_1 = R1.f0, f1_0 = R0.f1, f1_1 = R1.f1;
  const uint32_t lrec_0 = R0.lrec, lrec_1 = R1.lrec;
  const uint64_t tb_0 = (uint64_t)(uintptr_t)R0.tb, tb_1 = (uint64_t)(uintptr_t)R1.tb;
  const uint64_t lb_0 = (uint64_t)(uintptr_t)R0.lb, lb_1 = (uint64_t)(uintptr_t)R1.lb;
  auto make_batch = [&](int base) __attribute__((always_inline)) -> StepDesc {
    return step_desc<D, ROWS>(wp, base + lane, H, w >= 2, len_0, len_1, f0_0, f0_1, f1_0, f1_1, lrec_0, lrec_1, tb_0, tb_1,
                     lb_0, lb_1);
  };
  StepDesc bt;
  int bbase = n0;
  // Per-lane offsets of the dword copy for each range (32 rows of two heads, or 64 rows of one).
  const uint32_t lvo0 = (uint32_t)(ROWS ? lane * 4 : ((lane >> 5) * R0.len + (lane & 31)) * 4);
  const uint32_t lvo1 = (uint32_t)(ROWS ? lane * 4 : ((lane >> 5) * R1.len + (lane & 31)) * 4);
  auto rl = [&](uint32_t v, int i) __attribute__((always_inline)) {
    return (uint32_t)__builtin_amdgcn_readlane((int)v, i - bbase);
  };
  // The copy resources of step i.
  auto copy_plan = [&](int i) __attribute__((always_inline)) -> CopyPlan {
    CopyPlan cp;
    cp.rt[0] = rl(bt.t0, i);
    cp.rt[1] = rl(bt.t1, i);
    cp.rt[2] = rl(bt.t2, i);
    cp.rt[3] = 0x00020000u;
    cp.rl[0] = rl(bt.l0, i);
    cp.rl[1] = rl(bt.l1, i);
    cp.rl[2] = rl(bt.l2, i);
    cp.rl[3] = 0x00020000u;
    cp.lvo = (rl((uint32_t)bt.flags, i) & 1) ? lvo1 : lvo0;
    return cp;
  };
  auto copy_issue = [&](const CopyPlan& cp, int st, int i) __attribute__((always_inline)) {
    if (i < IPW) {
      dma16(cp.rt, L0 + (w < 2 ? Sh::QRegion : Sh::DoRegion) + st * TileB + (wodd * IPW + i) * 1024, voff[i]);
    } else {
      const uint32_t ldst =
          w >= 2 ? L0 + Sh::StatRegion + st * Sh::StatB + (w == 2 ? 0u : 256u) : L0 + Sh::SpareRegion + w * 256;
      dma4(cp.rl, ldst, cp.lvo);
    }
  };
  // The resource words come from readlane, a vector instruction writing scalar
  // registers; a buffer access reading them needs five wait states after it,
  // which the compiler does not insert before inline assembly.  Every plan
  // therefore passes an s_nop 4 that takes its words as inputs before its copies.
  auto plan_ready = [](const CopyPlan& cp) __attribute__((always_inline)) {
    asm volatile("s_nop 4" ::"s"(cp.rt), "s"(cp.rl), "v"(cp.lvo));
  };
  auto copy_step = [&](int st, int i) __attribute__((always_inline)) {
    const CopyPlan cp = copy_plan(i);
    plan_ready(cp);
#pragma unroll
    for (int i = 0; i <= IPW; ++i) copy_issue(cp, st, i);
  };

  const float c = a.scale_log2;
  // Per-lane read addresses (loop-invariant; stage, head and tensor are immediate offsets).
  // Row reads: lane (half, l32) reads logical chunk 2k + half of row l32.
  // (The dO addresses are laundered through an empty asm statement: otherwise
  // the compiler re-derives them from the Q addresses with an add per read.)
  uint32_t yq[KS], yd[KS];
#pragma unroll
  for (int k = 0; k < KS; ++k) {
    yq[k] = (L0 + Sh::QRegion + swz_row_part<D>(l32, half)) ^ (32u * k);
    yd[k] = yq[k] + Sh::DoRegion;
    asm volatile("" : "+v"(yd[k]));
  }
  // Transpose reads: rows 16u + R0 and 16u + R0 + 8 of the head's tile, 8-byte
  // piece 8d + 4 (G & 1) + (sl & 3).
  uint32_t tq0[DT], tq1[DT], td0[DT], td1[DT];
#pragma unroll
  for (int d = 0; d < DT; ++d) {
    tq0[d] = (L0 + Sh::QRegion + swz_tr_part<D>(G, sl, 0)) ^ (64u * d);
    tq1[d] = (L0 + Sh::QRegion + swz_tr_part<D>(G, sl, 8)) ^ (64u * d);
    td0[d] = tq0[d] + Sh::DoRegion;
    td1[d] = tq1[d] + Sh::DoRegion;
    asm volatile("" : "+v"(td0[d]), "+v"(td1[d]));
  }
  // Accumulator starts of a step: for head j, register i of a lane holds query
  // row 8 (i / 4) + 4 half + i % 4 of the step.
  uint32_t ystat = L0 + Sh::StatRegion + (uint32_t)(4 * half) * 4;
  asm volatile("" : "+v"(ystat));  // one base register; stage, head and row offsets stay immediate

  f32x16 sa[2], da[2];
  // The first row-read pairs of a step, issued at the end of the step before
  // (its stage is complete from the barrier before that step on).
  constexpr int RA = D == 128 ? 4 : ADAPT ? 1 : 2;  // row-read pairs in flight ahead of the score products
  bf16x8 nq[RA], nd[RA];
  // Starts at -inf where the row mbase + (offset of register i) is hidden from the lane's key.
  auto mask_sub = [](f32x16& s, int mbase, int lane_qw) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      float x0 = s[i];
      uint32_t tmp;
      asm volatile(
          "v_add_u32 %1, %2, %3\n\t"
          "v_cmp_lt_u32 vcc, %1, %4\n\t"
          "v_mov_b32 %1, 0xff800000\n\t"
          "v_cndmask_b32 %0, %1, %0, vcc"
          : "+v"(x0), "=&v"(tmp)
          : "n"(8 * (i >> 2) + (i & 3)), "v"(mbase), "v"(lane_qw)
          : "vcc");
      s[i] = x0;
    }
  };
  // Load the starts of step i (stage st) and apply the mask of partly visible steps.
  auto load_starts = [&](int st, int si) __attribute__((always_inline)) {
    const uint32_t base = ystat + st * Sh::StatB;
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int g4 = 0; g4 < 4; ++g4) {
        const f32x4 l = lds_f4(base + (j * kSub + 8 * g4) * 4);
        const f32x4 dd = lds_f4(base + 256 + (j * kSub + 8 * g4) * 4);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          sa[j][4 * g4 + e] = l[e];
          da[j][4 * g4 + e] = dd[e];
        }
      }
    const int fl = (int)rl((uint32_t)bt.flags, si), q = fl & 1;
    // Partly visible steps: hidden scores start at -inf.  The compare and the
    // selects are inline assembly inside a wave-uniform branch: as plain code
    // the compiler speculates them onto every step.
    if (fl & 2) {
      const int mbase = BDLM_PICK(pos0, q) + (int)rl((uint32_t)bt.s, si) * BM + 4 * half - BDLM_PICK(qa, q);
      const int lane_qw = BDLM_PICK(qw, q);
      if constexpr (ROWS) {
        mask_sub(sa[0], mbase, lane_qw);
        mask_sub(sa[1], mbase + kSub, lane_qw);
      } else {
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          float x0 = sa[0][i], x1 = sa[1][i];
          uint32_t tmp;
          // hidden when (unsigned)(mbase + row offset of register i) >= lane_qw
          asm volatile(
              "v_add_u32 %2, %3, %4\n\t"
              "v_cmp_lt_u32 vcc, %2, %5\n\t"
              "v_mov_b32 %2, 0xff800000\n\t"
              "v_cndmask_b32 %0, %2, %0, vcc\n\t"
              "v_cndmask_b32 %1, %2, %1, vcc"
              : "+v"(x0), "+v"(x1), "=&v"(tmp)
              : "n"(8 * (i >> 2) + (i & 3)), "v"(mbase), "v"(lane_qw)
              : "vcc");
          sa[0][i] = x0;
          sa[1][i] = x1;
        }
      }
    }
  };

  // The starts of head j of step `cu` (stage st) into s, d, with the mask of
  // partly visible steps (the values load_starts gives that head).
  auto load_head_starts = [&](int st, int si, int j, f32x16& s, f32x16& d) __attribute__((always_inline)) {
    const uint32_t base = ystat + st * Sh::StatB;
#pragma unroll
    for (int g4 = 0; g4 < 4; ++g4) {
      const f32x4 l = lds_f4(base + (j * kSub + 8 * g4) * 4);
      const f32x4 dd = lds_f4(base + 256 + (j * kSub + 8 * g4) * 4);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        s[4 * g4 + e] = l[e];
        d[4 * g4 + e] = dd[e];
      }
    }
    const int fl = (int)rl((uint32_t)bt.flags, si), q = fl & 1;
    if (fl & 2) {
      const int mbase = BDLM_PICK(pos0, q) + (int)rl((uint32_t)bt.s, si) * BM + 4 * half - BDLM_PICK(qa, q);
      const int lane_qw = BDLM_PICK(qw, q);
      mask_sub(s, mbase + (ROWS ? j * kSub : 0), lane_qw);
    }
  };

  // One step on stage ST: the copies of step `cp` into stage CP go out under
  // its first products, the starts of step `nx` (stage NX) are loaded under its
  // last ones, and the walk advances under the softmax of head 0.
  constexpr int TA = D == 128 ? 8 : ADAPT ? 2 : 4;  // transpose-read pairs in flight ahead of the dV/dK products
  int i0 = n0;   // the current step
  CopyPlan cpl;  // copies of step i0 + 3, planned during the step before
  auto run_step = [&](auto st_c, auto nx_c, int cp_stage) __attribute__((always_inline)) {
    constexpr int ST = decltype(st_c)::value, NX = decltype(nx_c)::value;
    constexpr uint32_t SO = ST * TileB;  // stage offset inside a tensor region
    // ---- A and B: S_j = Q_j K^T + start, dP_j = dO_j V^T + start, j = 0, 1 (32
    // products), the softmax of head 0 under the products of head 1.
    bf16x8 rq[RA + 1], rd[RA + 1];
    auto rowq = [&](int n) { return lds_load16(yq[n % KS] + SO + (n / KS) * HB); };
    auto rowd = [&](int n) { return lds_load16(yd[n % KS] + SO + (n / KS) * HB); };
#pragma unroll
    for (int n = 0; n < RA; ++n) {
      rq[n] = nq[n];
      rd[n] = nd[n];
    }
    // Transpose reads of blocks C and D: rows 16u .. 16u + 15 of head j.
    auto trd = [&](int j, int u, int d) {
      const uint32_t o = SO + j * HB + u * 16 * RB;
      return cat(lds_read_tr_at(td0[d] + o), lds_read_tr_at(td1[d] + o));
    };
    auto trq = [&](int j, int u, int d) {
      const uint32_t o = SO + j * HB + u * 16 * RB;
      return cat(lds_read_tr_at(tq0[d] + o), lds_read_tr_at(tq1[d] + o));
    };
    // product m of a sub-block: m < MD -> dV (u = m / DT, d = m % DT), else dK
    constexpr int MD = 2 * DT;
    auto opnd = [&](int j, int m) { return m < MD ? trd(j, m / DT, m % DT) : trq(j, (m - MD) / DT, (m - MD) % DT); };
    bf16x8 tf[TA + 1];
    bf16x8 pb[2][2], dsb[2][2];
    float pm[2][2] = {{0.f, 0.f}, {0.f, 0.f}};  // ADAPT: largest P per head and 16-row half
#pragma unroll
    for (int n = 0; n < 2 * KS; ++n) {
      if (n + RA < 2 * KS) {
        rq[(n + RA) % (RA + 1)] = rowq(n + RA);
        rd[(n + RA) % (RA + 1)] = rowd(n + RA);
      }
      if (n >= 2 * KS - TA) tf[n - (2 * KS - TA)] = opnd(0, n - (2 * KS - TA));  // block C's first operands
      const int j = n / KS, k = n % KS;
      sa[j] = mfma32(rq[n % (RA + 1)], kf[k], sa[j]);
      da[j] = mfma32(rd[n % (RA + 1)], vf[k], da[j]);
      if (n <= IPW) copy_issue(cpl, cp_stage, n);
      if (n == IPW + (D == 128 ? 3 : 1)) cpl = copy_plan(i0 + 4);
      if (n == IPW + (D == 128 ? 4 : 2)) plan_ready(cpl);

      if (j == 1) {
        // softmax of sub-block 0: SPP scores per product pair
        constexpr int SPP = 16 / KS;
#pragma unroll
        for (int e = 0; e < SPP; ++e) {
          const int i = SPP * k + e;
          const float p = exp2f_fast(sa[0][i] * c);
          da[0][i] = p * da[0][i];
          sa[0][i] = p;
          if constexpr (ADAPT) pm[0][i >> 3] = fmaxf(pm[0][i >> 3], p);
        }
        if ((SPP * (k + 1)) % 4 == 0) {
          const int i0 = SPP * (k + 1) - 4;
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            pb[0][(i0 + e) >> 3][(i0 + e) & 7] = to_bf16(sa[0][i0 + e]);
            dsb[0][(i0 + e) >> 3][(i0 + e) & 7] = to_bf16(da[0][i0 + e]);
          }
        }
      }
      fence();
    }
    // ---- C and D: dV^T += dO_j^T P_j, dK^T += Q_j^T dS_j (queries are the
    // contraction index), head 0 under the softmax of head 1, head 1 under
    // dS_1 and the next step's starts.  Per product: two transpose reads.
    // ADAPT: the 16-row half u of head j also carries P - bf16(P) and
    // dS - bf16(dS) (from P_j and dS_j, still in sa[j], da[j]) as second bf16
    // terms when some probability of that half reaches hilo_tau: 4 dV and 4 dK
    // products more.
    auto second_terms = [&](int j) __attribute__((always_inline)) {
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        if (__builtin_amdgcn_ballot_w64(pm[j][u] >= a.hilo_tau) != 0) {
          // All eight operands are read before the residuals are formed, whose
          // vector work covers the reads' latency (8K, 32/4 heads: the kernel
          // 3.36 -> 3.14 ms against reading each before its product).
          bf16x8 od[DT], oq[DT];
#pragma unroll
          for (int d = 0; d < DT; ++d) od[d] = trd(j, u, d);
#pragma unroll
          for (int d = 0; d < DT; ++d) oq[d] = trq(j, u, d);
          fence();
          bf16x8 pl, dl;
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            const float p = sa[j][8 * u + e], ds = da[j][8 * u + e];
            pl[e] = to_bf16(p - (float)to_bf16(p));
            dl[e] = to_bf16(ds - (float)to_bf16(ds));
          }
#pragma unroll
          for (int d = 0; d < DT; ++d) mfma_agpr_padded(dva[d], od[d], pl);
#pragma unroll
          for (int d = 0; d < DT; ++d) mfma_agpr_padded(dka[d], oq[d], dl);
        }
      }
    };
    if constexpr (ADAPT) {
      second_terms(0);
      fence();
    }
#pragma unroll
    for (int n = 0; n < 4 * MD; ++n) {
      if (n + TA < 4 * MD) tf[(n + TA) % (TA + 1)] = opnd((n + TA) / (2 * MD), (n + TA) % (2 * MD));
      const int j = n / (2 * MD), m = n % (2 * MD);
      if (m < MD) mfma_agpr(dva[m % DT], tf[n % (TA + 1)], pb[j][m / DT]);
      else mfma_agpr(dka[(m - MD) % DT], tf[n % (TA + 1)], dsb[j][(m - MD) / DT]);
      if (j == 0) {
        // P_1 = exp2(c S_1): SP scores per product
        constexpr int SP = 16 / (2 * MD);
#pragma unroll
        for (int e = 0; e < SP; ++e) {
          const int i = SP * m + e;
          sa[1][i] = exp2f_fast(sa[1][i] * c);
          if constexpr (ADAPT) pm[1][i >> 3] = fmaxf(pm[1][i >> 3], sa[1][i]);
          if (i & 1) {
            pb[1][i >> 3][(i - 1) & 7] = to_bf16(sa[1][i - 1]);
            pb[1][i >> 3][i & 7] = to_bf16(sa[1][i]);
          }
        }
      } else if (m < MD) {
        // dS_1 = P_1 dP_1 under the dV products of sub-block 1
        constexpr int SD = 16 / MD;
#pragma unroll
        for (int e = 0; e < SD; ++e) {
          const int i = SD * m + e;
          da[1][i] = sa[1][i] * da[1][i];
        }
        if ((SD * (m + 1)) % 4 == 0) {
          const int i0 = SD * (m + 1) - 4;
#pragma unroll
          for (int e = 0; e < 4; ++e) dsb[1][(i0 + e) >> 3][(i0 + e) & 7] = to_bf16(da[1][i0 + e]);
        }
      } else if (m == MD) {
        if constexpr (!ADAPT) load_starts(NX, i0 + 1);
        else load_head_starts(NX, i0 + 1, 0, sa[0], da[0]);
      }
      fence();
    }
    if constexpr (ADAPT) {
      // head 1's second terms need P_1 and dS_1, which its next starts
      // overwrite: both come after the products here
      second_terms(1);
      load_head_starts(NX, i0 + 1, 1, sa[1], da[1]);
      fence();
    }
#pragma unroll
    for (int i = 0; i < RA; ++i) {
      nq[i] = lds_load16(yq[i] + NX * TileB);
      nd[i] = lds_load16(yd[i] + NX * TileB);
    }
    asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(IPW + 1) : "memory");
    ++i0;
  };

  // ---- the walk: four LDS stages, copies three steps ahead.  At the barrier
  // closing step i every wave has waited for its copies of step i + 2 (only
  // those of step i + 3 stay in flight) and has finished reading stage i,
  // which the copies issued next overwrite.
  // A batch covers steps bbase .. bbase + 63 and is renewed every 56 steps: an
  // iteration of the loop below starting at step i0 reads steps up to i0 + 7.
  bt = make_batch(n0);
  cpl = copy_plan(n0 + 3);
  plan_ready(cpl);
  copy_step(0, n0);
  copy_step(1, n0 + 1);
  copy_step(2, n0 + 2);
  asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(IPW + 1) : "memory");  // steps 0 and 1 landed
  // K and V are pinned in AGPRs only now: pinning reads them, so their loads
  // (issued first) are waited for here, after the walk set-up and the first
  // copies, instead of before them.
#pragma unroll
  for (int s = 0; s < KS; ++s) asm volatile("" : "+a"(kf[s]), "+a"(vf[s]));
  load_starts(0, n0);
#pragma unroll
  for (int i = 0; i < RA; ++i) {
    nq[i] = lds_load16(yq[i]);
    nd[i] = lds_load16(yd[i]);
  }
  using I0 = std::integral_constant<int, 0>;
  using I1 = std::integral_constant<int, 1>;
  using I2 = std::integral_constant<int, 2>;
  using I3 = std::integral_constant<int, 3>;
  while (i0 < n1) {
    if (i0 - bbase >= 56) {
      bbase = i0;
      bt = make_batch(bbase);
    }
    run_step(I0{}, I1{}, 3);
    if (i0 >= n1) break;
    run_step(I1{}, I2{}, 0);
    if (i0 >= n1) break;
    run_step(I2{}, I3{}, 1);
    if (i0 >= n1) break;
    run_step(I3{}, I0{}, 2);
  }
  // Copies still in flight target stages nobody reads; they must land before
  // the workgroup's LDS is released.  The last dV/dK products must finish
  // before their accumulators are read.
  asm volatile("s_waitcnt vmcnt(0)\n\ts_nop 15\n\ts_nop 15" ::: "memory");
#undef BDLM_PICK

  // ---- epilogue: dK = scale dK^T^T, dV (bf16 or fp32); unseen keys get zeros
#pragma unroll
  for (int d = 0; d < DT; ++d) asm volatile("" : "+a"(dka[d]), "+a"(dva[d]));
  // A key that no query sees keeps zeros whatever its rows hold: a non-finite K
  // or V row makes NaN of its hidden pairs.
  const bool unseen = (R0.qw | R1.qw) == 0;
  if (__builtin_amdgcn_ballot_w64(unseen) != 0) {
#pragma unroll
    for (int d = 0; d < DT; ++d)
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        dka[d][i] = unseen ? 0.f : dka[d][i];
        dva[d][i] = unseen ? 0.f : dva[d][i];
      }
  }
  const uint64_t part = ((uint64_t)__builtin_amdgcn_readfirstlane((int)(partial_at >> 32)) << 32) |
                        (uint32_t)__builtin_amdgcn_readfirstlane((int)partial_at);
  if (part != 0) {
    // The chunk's partial sums: 16-byte piece 4 d + g4 of dK, then of dV, of
    // each half, [piece][half][key], so that a store writes 512-byte runs.
    if (key_ok) {
      f32x4* pp = (f32x4*)(uintptr_t)part;
      const uint32_t at = (uint32_t)(half * nk + mykey);
#pragma unroll
      for (int d = 0; d < DT; ++d)
#pragma unroll
        for (int g4 = 0; g4 < 4; ++g4) {
          f32x4 vk, vv;
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            vk[e] = dka[d][4 * g4 + e];
            vv[e] = dva[d][4 * g4 + e];
          }
          pp[at + (uint32_t)((4 * d + g4) * 2 * nk)] = vk;
          pp[at + (uint32_t)((4 * DT + 4 * d + g4) * 2 * nk)] = vv;
        }
    }
  } else if (a.out_f32) {
    if (key_ok) {
      const int64_t off = (((int64_t)b * kr.bstride + key0 + mykey) * HKV + kvh) * D;
      float* dkp = (float*)kr.dk + off;
      float* dvp = (float*)kr.dv + off;
#pragma unroll
      for (int d = 0; d < DT; ++d)
#pragma unroll
        for (int g4 = 0; g4 < 4; ++g4) {
          f32x4 vk, vv;
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            vk[e] = dka[d][4 * g4 + e] * a.scale;
            vv[e] = dva[d][4 * g4 + e];
          }
          *(f32x4*)(dkp + 32 * d + 8 * g4 + 4 * half) = vk;
          *(f32x4*)(dvp + 32 * d + 8 * g4 + 4 * half) = vv;
        }
    }
  } else {
    // Each wave's 32 rows of dK and dV go through its own 16 KB of LDS (in the
    // Q stages, free once every wave has left the walk), so that a store
    // writes 4 whole rows instead of 16 bytes of each of 32 rows.  Chunk c
    // (16 bytes) of row r sits at chunk c ^ (r & 15): conflict-free reads.
    asm volatile("s_barrier" ::: "memory");
    const uint32_t sw = L0 + Sh::QRegion + (uint32_t)w * (2 * HB);
    constexpr int CH = D / 8;  // 16-byte chunks per row
#pragma unroll
    for (int d = 0; d < DT; ++d)
#pragma unroll
      for (int g4 = 0; g4 < 4; ++g4) {
        bf16x4 vk, vv;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          vk[e] = to_bf16(dka[d][4 * g4 + e] * a.scale);
          vv[e] = to_bf16(dva[d][4 * g4 + e]);
        }
        const uint32_t o = (uint32_t)l32 * RB + (((uint32_t)(4 * d + g4) ^ (uint32_t)(l32 & (CH - 1))) * 16u) + 8u * half;
        lds_store8(sw + o, vk);
        lds_store8(sw + HB + o, vv);
      }
#pragma unroll
    for (int i = 0; i < CH / 2; ++i) {
      const int r = i * (64 / CH) + lane / CH, c = lane % CH;
      const uint32_t o = (uint32_t)r * RB + (((uint32_t)c ^ (uint32_t)(r & (CH - 1))) * 16u);
      const bf16x8 xk = lds_load16(sw + o), xv = lds_load16(sw + HB + o);
      if (w * 32 + r < nk) {
        const int64_t go = (((int64_t)b * kr.bstride + key0 + w * 32 + r) * HKV + kvh) * D + c * 8;
        *(bf16x8*)((bf16*)kr.dk + go) = xk;
        *(bf16x8*)((bf16*)kr.dv + go) = xv;
      }
    }
  }
}

// dK, dV of the chunked key tiles: the chunks' partial sums added in chunk
// order.  A thread owns 8 consecutive head_dim elements of one key of dK or
// dV, two 16-byte pieces of each partial; kSumWgs workgroups per tile.  HBM
// (mostly L2 and MALL) traffic: the partials once.
template <int D>
constexpr int kSumWgs = 4 * 2 * D / 32 * 4 * 32 / 256;
template <int D>
__global__ __launch_bounds__(256) void dkdv_sum_kernel(const AttnArgs a) {
  constexpr int DT = D / 32, PIECES = 2 * DT * 4;  // per 32 keys: dK's 4 d + g4, then dV's
  SumItem it;
  sum_item(a, blockIdx.x / kSumWgs<D>, it);
  const int nch = a.split.counts[blockIdx.x / kSumWgs<D>];
  if (nch <= 1) return;
  const int n = (blockIdx.x % kSumWgs<D>) * 256 + threadIdx.x;
  const int l32 = n & 31, piece = (n >> 5) % PIECES, w = (n >> 5) / PIECES;
  const KRangeArg& kr = a.kr[it.r];
  const int key0 = it.t * kBwdKeysBf16, nk = imin(kBwdKeysBf16, kr.len - key0);
  if (w * 32 + l32 >= nk) return;
  const int key = key0 + w * 32 + l32, at = piece * 2 * nk + w * 32 + l32;
  f32x4 lo = {0.f, 0.f, 0.f, 0.f}, hi = lo;
  for (int ch = 0; ch < nch; ++ch) {
    const f32x4* pp = (const f32x4*)((const float*)a.split.partials +
                                     partial_row<kBwdKeysBf16>(a, it.b, it.kvh, it.r, it.t, ch) * (2 * D));
    lo += pp[at];
    hi += pp[at + nk];
  }
  const bool is_dv = piece >= 4 * DT;
  const float sc = is_dv ? 1.f : a.scale;
  const int64_t off = (((int64_t)it.b * kr.bstride + key) * a.kv_heads + it.kvh) * D + (piece & (4 * DT - 1)) * 8;
  void* out = is_dv ? kr.dv : kr.dk;
  if (a.out_f32) {
    *(f32x4*)((float*)out + off) = lo * sc;
    *(f32x4*)((float*)out + off + 4) = hi * sc;
  } else {
    bf16x8 v;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      v[e] = to_bf16(lo[e] * sc);
      v[4 + e] = to_bf16(hi[e] * sc);
    }
    *(bf16x8*)((bf16*)out + off) = v;
  }
}

}  // namespace

hipError_t launch_bwd_dkdv_sum(const AttnArgs& a, int head_dim, hipStream_t s) {
  const int n = a.split.tiles_per_pair * a.kv_heads * a.batch;
  if (n == 0) return hipSuccess;
  if (head_dim == 128) hipLaunchKernelGGL(dkdv_sum_kernel<128>, dim3(n * kSumWgs<128>), dim3(256), 0, s, a);
  else hipLaunchKernelGGL(dkdv_sum_kernel<64>, dim3(n * kSumWgs<64>), dim3(256), 0, s, a);
  return hipGetLastError();
}

namespace {

template <int D, bool ADAPT>
void launch_rows(const AttnArgs& a, int n, hipStream_t s) {
  if (a.group % 2 == 0) hipLaunchKernelGGL((dkdv_kernel<D, ADAPT, false>), dim3(n), dim3(256), 0, s, a);
  else hipLaunchKernelGGL((dkdv_kernel<D, ADAPT, true>), dim3(n), dim3(256), 0, s, a);
}

}  // namespace

hipError_t launch_bwd_dkdv(const AttnArgs& a, int head_dim, hipStream_t s) {
  const int n = workgroups_for(a.split.wgs_per_pair * a.kv_heads * a.batch);
  if (n == 0) return hipSuccess;
  // at most two query ranges (the walk state stays in registers), no two-term products on every step
  const bool two_terms = a.hilo & kHiloDkDv;
  if (a.n_q > 2 || (two_terms && !(a.hilo & kHiloAdaptive))) return hipErrorInvalidValue;
  if (head_dim == 128) two_terms ? launch_rows<128, true>(a, n, s) : launch_rows<128, false>(a, n, s);
  else two_terms ? launch_rows<64, true>(a, n, s) : launch_rows<64, false>(a, n, s);
  return hipGetLastError();
}

}  // namespace bdlm
