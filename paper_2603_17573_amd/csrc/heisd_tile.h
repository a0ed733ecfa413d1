// Projections of M > 8 rows as one kernel of two-dimensional tiles (the records of heisd_batch.h times the packed weights).
//
// A workgroup owns TA weight tiles x TC column tiles (16 x 16 accumulators each) over one run of the reduction.  Both operands
// go from memory to LDS with direct transfers, a k-step (32 values of the reduction: 1 KB per tile of either kind) per slot of a
// ring; every wave issues its share of the transfers and every wave multiplies AW x CW accumulator tiles from fragments read out of
// LDS.  What bounds it, measured on one MI355X with the 24 x 14 tile at 448 rows x 22016 weight rows, launches repeated by
// themselves, on the loop that issued its transfers in front of rows of products: with the products left out it took 95 us (a compute unit's memory path answers about 54 B/ns
// of mixed HBM and L2 reads), with the transfers left out 118 us, products alone 104 us (the chip holds about 1.5 PFLOP/s of them), all together 124 us, 1.3
// PFLOP/s.  Inside steps the launch takes 125 us on today's loop (mean of 1120; 127 before).  So:
//   * no wave only moves data: the four SIMDs share the products evenly (six multiplying and two moving waves, the arrangement
//     before, left two SIMDs half idle: 167 us);
//   * three waves where the weights are what takes time: 6 weight tiles per workgroup give 5.4 tiles per compute unit of the 7B
//     gate/up, 2.7 rounded up to 3 pairs, a unit each (230 workgroups; 56 rows, inside a step: 44 us; before today's loop 45, the 8 x 7 tile's 172 workgroups 50);
//   * large tiles where there are rows and weights enough for every compute unit to have one (bytes per product are
//     1/TA + 1/TC), small ones where there are not: the choice is tile_plan's, from the tables of measured step times;
//   * transfers and the reads of the next fragments stand BETWEEN the products, one or two behind each: issued in front of a row of products, the matrix
//     core of a SIMD with one wave had nothing to do meanwhile.  Clocks per k-step, before and now: 12 x 14 tile 1105 / 878 (its products take
//     672), 16 x 7 868 / 754 (448; 23 KB of transfers in that time are 58 B/ns at 1.9 GHz: the memory path's limit), 24 x 9 1319 / 1154 (864), 24 x 14 with two waves per SIMD
//     1574 / 1472 (1344).  The chip then clocks lower (2.0 -> 1.6 to 1.9 GHz), so that in time 448 rows of QKV took 73 -> 63 us of loop, down 76 -> 69, gate/up 108 -> 106.
//     Whole launches inside 32-layer steps, means of 1120: QKV 84.6 -> 79.1 us, down 77.8 -> 76.8, gate/up 127.0 -> 124.7, O-projection (8 x 7) 43.5 -> 43.0;
//   * one barrier per k-step, in the middle of it: behind it the next step's fragments may be read before this step's products are
//     done, and the slot of the step before may be filled again.
//
// Three- and four-wave tiles have one wave per SIMD and up to 64 accumulators of it in accumulation registers; each product is written
// as assembly because the compiler copies such accumulators back and forth between the two halves of the register file (260 moves per 84 products).
#pragma once
#include <type_traits>
#include <utility>

#include "heisd_batch.h"

namespace heisd {

// One product into an accumulator of the second register half.  `fresh`: two wait states for a fragment the compiler may just have moved (the first
// product of a row; nothing else of the loop writes fragments but LDS reads, which are waited for).
template <bool FRESH>
__device__ __forceinline__ void tile_mul(f32x4 &c, const u32x4 a, const u32x4 b) {
  if (FRESH) asm volatile("s_nop 1\n\tv_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(c) : "v"(a), "v"(b));
  else asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(c) : "v"(a), "v"(b));
}
// The last products are written before anything reads them.
template <int CW>
__device__ __forceinline__ void tile_settle(f32x4 (&c)[CW]) {
  asm volatile("s_nop 15\n\ts_nop 15" : "+a"(c[0]));
#pragma unroll
  for (int i = 1; i < CW; ++i) asm volatile("" : "+a"(c[i]));
}

// WA x WC waves, each AW weight tiles x CW column tiles; OCC workgroups share a compute unit.
template <int WA_, int WC_, int AW_, int CW_, int OCC_>
struct TileShape {
  static constexpr int WA = WA_, WC = WC_, AW = AW_, CW = CW_, OCC = OCC_;
  static constexpr int NW = WA * WC, TA = WA * AW, TC = WC * CW;
  static constexpr int ST = TA + TC;                               // transfers (and KB) per k-step
  static constexpr int OPS = (ST + NW - 1) / NW;                   // of one wave (a surplus one repeats the last)
  static constexpr int kFit = (OCC == 2 ? 78 : 156) / ST;
  static constexpr int NB = kFit > 8 ? 8 : kFit;                   // slots of the ring
  static constexpr size_t kLds = (size_t)NB * ST * 1024;
  static constexpr bool kAcc = NW <= 4;                            // one wave per SIMD (and OCC): accumulators in the second register half
  static constexpr int kPerSimd = (OCC * NW + 3) / 4;
  static_assert(TA % NW == 0, "the first TA / NW transfers of every wave are weights, the others column tiles");
  static_assert(NB >= 4 && (NB - 2) * OPS <= 63 && AW >= 2 && AW * CW <= 64, "ring and accumulators");
};

// f(integral_constant<int, 0>), .. f(integral_constant<int, N - 1>).
template <int N, class F>
__device__ __forceinline__ void unrolled(F f) {
  [&]<int... I>(std::integer_sequence<int, I...>) __attribute__((always_inline)) { (f(std::integral_constant<int, I>{}), ...); }(std::make_integer_sequence<int, N>{});
}

// What is issued behind product (row t, column tile c) of a k-step: op[t * CW + c], in this order.  A row's operations - the weight tile two rows
// on, from row TB on the next step's column tiles, the transfers (those of a step go to rows TB, .. AW - 1, 0, ..) - are spread over its products.
enum { kOpNone = 0, kOpWeights = 1, kOpColumn = 2, kOpTransfer = 32 };
template <class T>
struct TileOrder {
  static constexpr int AW = T::AW, CW = T::CW, OPS = T::OPS;
  static constexpr int kHalf = AW / 2;
  static constexpr int TB = kHalf < AW - 1 ? kHalf : AW - 2;         // the barrier stands before row TB of a step's products
  static constexpr int kMost = 4;
  int op[AW * CW][kMost] = {};
  static constexpr int transfer_row(int o) { return (TB + o * AW / OPS) % AW; }
  constexpr TileOrder() {
    for (int t = 0; t < AW; ++t) {
      int list[1 + CW + OPS] = {kOpWeights}, n = 1;
      for (int c = 0; c < CW; ++c)
        if (t >= TB && c * (AW - TB) / CW == t - TB) list[n++] = kOpColumn + c;
      for (int o = 0; o < OPS; ++o)
        if (transfer_row(o) == t) list[n++] = kOpTransfer + o;
      for (int k = 0; k < n; ++k) {
        int (&at)[kMost] = op[t * CW + k * CW / n];
        int i = 0;
        while (at[i] != kOpNone) ++i;                                // (more than kMost: not a constant expression)
        at[i] = list[k];
      }
    }
  }
};

// The projection's epilogue for columns 4*q .. 4*q+3 of unit `unit` of row `jr` of column tile `ct`: s the sums (u: of the up tile), x the residual
// stream's old values, gain the next norm's gains.  The four lanes q = 0..3 of a row call it together: lanes 16 apart (ADJ = false:
// accumulator layout) or adjacent ones (ADJ).  SINGLE: one bf16 per activation, 16 rows per column tile.  `on`: the lane has a row.
template <bool ADJ, bool SINGLE>
__device__ __forceinline__ void tile_emit(const BatGemm &g, int unit, int ct, int jr, int q, f32x4 s, f32x4 u, float sc, f32x4 x, f32x4 gain,
                                          bool on) {
  const int m = ct * (SINGLE ? 16 : 8) + jr;
  const bool live = on && m < g.M;
  float *out = g.out + (size_t)m * g.ldo + unit * 16 + 4 * q;
  f32x4 a = f32x4{0.f, 0.f, 0.f, 0.f};
  if (g.epi == FEPI_STORE_ROWS) {
#pragma unroll
    for (int i = 0; i < 4; ++i) a[i] = s[i] * sc;
    if (live) *reinterpret_cast<f32x4 *>(out) = a;
    return;
  }
  if (g.epi == FEPI_SWIGLU) {
    if (live) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float gv = s[i] * sc;
        a[i] = gv / (1.0f + expf(-gv)) * (u[i] * sc);
      }
    }
  } else {
    if (live) {
#pragma unroll
      for (int i = 0; i < 4; ++i) a[i] = x[i] + s[i] * sc;
      *reinterpret_cast<f32x4 *>(out) = a;
    }
    // the row's sum of squares over the tile's 16 columns: pairs, then a tree over them
    float p0 = fmaf(a[1], a[1], a[0] * a[0]), p1 = fmaf(a[3], a[3], a[2] * a[2]);
    asm volatile("" : "+v"(p0), "+v"(p1));           // two sums of two squares each, not one chain of four
    float t = p0 + p1;
    if (ADJ) {
      t += dpp_move<kDppXor1>(t);
      t += dpp_move<kDppXor2>(t);
    } else {
      t = sum_xor16(t);
      t = sum_xor32(t);
    }
    if (q == 0 && on) g.ssq_out[(size_t)unit * (g.CTS * 8) + m] = t;
#pragma unroll
    for (int i = 0; i < 4; ++i) a[i] *= gain[i];
  }
  uint32_t h[4], l[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) split_bf16(a[i], h[i], l[i]);
  if (!on) return;
  uint16_t *rec = g.o_planes + ((size_t)unit * g.CTS + ct) * 256 + jr * 16 + 4 * q;
  *reinterpret_cast<uint2 *>(rec) = make_uint2(h[0] | (h[1] << 16), h[2] | (h[3] << 16));
  if (!SINGLE) *reinterpret_cast<uint2 *>(rec + 128) = make_uint2(l[0] | (l[1] << 16), l[2] | (l[3] << 16));
}
__device__ __forceinline__ f32x4 tile_old_x(const BatGemm &g, int unit, int m, int q) {
  if (g.epi != FEPI_RESID_NORM || m >= g.M) return f32x4{0.f, 0.f, 0.f, 0.f};
  return *reinterpret_cast<const f32x4 *>(g.out + (size_t)m * g.ldo + unit * 16 + 4 * q);
}
__device__ __forceinline__ f32x4 tile_gain(const BatGemm &g, int unit, int q) {
  if (g.epi != FEPI_RESID_NORM) return f32x4{0.f, 0.f, 0.f, 0.f};
  return *reinterpret_cast<const f32x4 *>(g.next_gain + unit * 16 + 4 * q);
}

// A wave's end: its accumulators through the epilogue, or, in a split reduction, its sums to part.
// Heads and tails (SINGLE = false): accumulator column j holds row j's head sums (j < 8) or row j - 8's tail sums.  They are added across the 16
// lanes; two column tiles make a full wave of rows (lanes 0-7 of 16 the even tile's, 8-15 the odd one's).  SINGLE: column j is row j.
template <class T, bool SINGLE>
__device__ __forceinline__ void tile_end(const BatGemm &g, f32x4 (&acc)[T::AW][T::CW], int tile0, int n_tiles, int ct0, int wc, const float *tab,
                                         int ks, int run, float *part, int lane) {
  constexpr int AW = T::AW, CW = T::CW, CS = SINGLE ? 1 : 2, kSlots = (CW + CS - 1) / CS, RPT = SINGLE ? 16 : 8;
  const int lr = lane & 15, lg = lane >> 4;
  const int jr = SINGLE ? lr : (lr & 7), codd = SINGLE ? 0 : lr >> 3;
  const bool swiglu = g.epi == FEPI_SWIGLU;
  auto sums = [&](const f32x4(&v)[CW], int i) __attribute__((always_inline)) {
    if (SINGLE) return v[i];
    f32x4 e = v[2 * i < CW ? 2 * i : 0], o = v[2 * i + 1 < CW ? 2 * i + 1 : 0];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      e[r] += dpp_move<0x128>(e[r]);                               // row_ror 8
      o[r] += dpp_move<0x128>(o[r]);
      e[r] = lr < 8 ? e[r] : o[r];
    }
    return e;
  };
#pragma unroll
  for (int t = 0; t < AW; ++t) {
    __builtin_amdgcn_sched_barrier(0);                             // one weight tile's values in registers at a time
    if constexpr (T::kAcc)                                         // the last products are written before anything reads them, and no
      if (t % 2 == 0) {                                            // copy out of the accumulation registers happens earlier
        tile_settle<CW>(acc[t]);
        if (t + 1 < AW) tile_settle<CW>(acc[t + 1 < AW ? t + 1 : t]);
      }
    const int tile = tile0 + t;
    if (tile >= n_tiles) continue;                                 // uniform over the wave
    if (swiglu && (t & 1)) continue;                               // a pair is emitted from its gate tile
    const int unit = swiglu ? tile >> 1 : tile;
    if (ks > 1) {
#pragma unroll
      for (int i = 0; i < kSlots; ++i) {
        const int c = i * CS + codd, m = (ct0 + c) * RPT + jr;
        const f32x4 s = sums(acc[t], i);
        if (c < CW && m < g.M)
          *reinterpret_cast<f32x4 *>(part + ((size_t)run * g.CT * RPT + m) * (g.n_units * 16) + unit * 16 + 4 * lg) = s;
      }
      continue;
    }
    f32x4 x[kSlots];                                               // requested before the first store: a load behind a store waits for it
#pragma unroll
    for (int i = 0; i < kSlots; ++i) x[i] = tile_old_x(g, unit, (ct0 + i * CS + codd) * RPT + jr, lg);
    const f32x4 gain = tile_gain(g, unit, lg);
#pragma unroll
    for (int i = 0; i < kSlots; ++i) {
      const int c = i * CS + codd, ct = ct0 + c;
      const f32x4 s = sums(acc[t], i);
      f32x4 u = s;
      if (swiglu) u = sums(acc[t + 1 < AW ? t + 1 : t], i);
      const float sc = g.scale_tag ? tab[min(c + wc * CW, T::TC - 1) * RPT + jr] : 1.0f;
      tile_emit<false, SINGLE>(g, unit, ct, jr, lg, s, u, sc, x[i], gain, c < CW && ct < g.CT);
    }
  }
}

// n_blk: blocks of TC column tiles; ks runs of `per` k-steps each.  ks > 1: the sums go to part[run][row][column] and
// bat_split_finish adds the runs in their order and applies the epilogue.
template <class T, bool SINGLE>
__global__ __launch_bounds__(64 * T::NW) __attribute__((amdgpu_waves_per_eu(T::kPerSimd, T::kPerSimd))) void bat_gemm_wide(
    BatGemm g, int n_blk, int ks, int per, float *part) {
  constexpr int NW = T::NW, TA = T::TA, TC = T::TC, AW = T::AW, CW = T::CW, ST = T::ST, OPS = T::OPS, NB = T::NB;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char *)smem;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lr = lane & 15, lg = lane >> 4;
  const bool swiglu = g.epi == FEPI_SWIGLU;
  const int n_tiles = swiglu ? 2 * g.n_units : g.n_units;          // SwiGLU: gate and up tiles of a unit follow each other
  const int n_groups = (n_tiles + TA - 1) / TA;
  // workgroup -> (weight group, row block, run): those of a weight group differ by 8 in the launch order, so they run next to
  // each other on one XCD and find its weights in that L2
  const int id = blockIdx.x, q8 = id >> 3;
  const int inner = q8 % (n_blk * ks), blk = inner % n_blk, run = inner / n_blk, grp = (q8 / (n_blk * ks)) * 8 + (id & 7);
  if (grp >= n_groups) {
    bat_scales_produce(g);
    return;
  }
  const int ktot = (g.Kd + 31) / 32, k0 = run * per;
  const int steps = min(per, ktot - k0);                           // >= 1: no run is empty
  const int wa = wave % T::WA, wc = wave / T::WA;
  // this wave's transfers of a k-step: fragments wave, wave + NW, ... (weight tiles, then column tiles)
  const unsigned char *src[OPS];
  uint32_t off[OPS];
  const uint32_t stride_b = (uint32_t)g.CTS * 1024u;
  const uint32_t off_a = lane * 16, off_b = ((uint32_t)(lg >> 1) * g.CTS * 256 + lr * 16 + (lg & 1) * 8) * 2;
#pragma unroll
  for (int o = 0; o < OPS; ++o) {
    const int f = min(o * NW + wave, ST - 1);
    const int tile = min(grp * TA + f, n_tiles - 1);               // surplus tiles: a valid one, the results are dropped
    int seg, in_seg;
    if (swiglu) { seg = tile & 1; in_seg = tile >> 1; }
    else { seg = (tile >= g.seg_tiles) + (tile >= 2 * g.seg_tiles); in_seg = tile - seg * g.seg_tiles; }
    const uint16_t *w = seg == 0 ? g.w[0] : (seg == 1 ? g.w[1] : g.w[2]);
    const int ct = max(0, min(blk * TC + f - TA, g.CTS - 1));
    const bool is_a = o < TA / NW;
    src[o] = is_a ? reinterpret_cast<const unsigned char *>(w) + ((size_t)in_seg * ktot + k0) * 1024
                  : reinterpret_cast<const unsigned char *>(g.b + ((size_t)2 * k0 * g.CTS + ct) * 256);
    off[o] = is_a ? off_a : off_b;
  }
  constexpr TileOrder<T> kOrder;
  constexpr int TB = TileOrder<T>::TB;
  // The transfers of a step are issued from its barrier on, the last ones in the first rows of the next step
  // (their slot is free until the next barrier).  Past the run's end the last k-step is transferred again: never read, and the count
  // of transfers in flight stays the same at every wait.
  constexpr uint32_t kSlot = ST * 1024, kRing = NB * kSlot;
  int fs = 0;
  uint32_t fslot = 0;
  auto transfer = [&](int o) __attribute__((always_inline)) {
    lds_dma16_s(src[o], off[o], __builtin_amdgcn_readfirstlane(lds0 + fslot + min(o * NW + wave, ST - 1) * 1024));
    src[o] += fs < steps - 1 ? (o < TA / NW ? 1024u : stride_b) : 0u;
  };
  f32x4 acc[AW][CW];
#pragma unroll
  for (int t = 0; t < AW; ++t)
#pragma unroll
    for (int c = 0; c < CW; ++c) acc[t][c] = f32x4{0.f, 0.f, 0.f, 0.f};
  wait_vmcnt_all();                                                // no wait of the compiler's between the transfers
  constexpr int kLate = [] {
    int n = 0;
    for (int o = 0; o < OPS; ++o) n += TileOrder<T>::transfer_row(o) < TB;
    return n;
  }();                                                             // transfers of a step issued in the next one
#pragma unroll 1
  for (; fs < NB - 2; ++fs, fslot += kSlot) {
#pragma unroll
    for (int o = 0; o < OPS; ++o) transfer(o);
  }
#pragma unroll
  for (int o = 0; o < OPS - kLate; ++o) transfer(o);
  bat_scales_produce(g);                                           // behind the first transfers: they are on their way meanwhile
  wait_vmcnt<(NB - 3) * OPS + OPS - kLate>();                      // step 0 has arrived
  __builtin_amdgcn_s_waitcnt(0xC07F);                              // lgkmcnt 0: with scalar loads pending the compiler could not count LDS reads in the loop
  asm volatile("s_barrier" ::: "memory");
  const unsigned char *pa = smem + wa * AW * 1024 + lane * 16, *pb = smem + (TA + wc * CW) * 1024 + lane * 16;
  u32x4 b0[CW], b1[CW], a0, a1;
#pragma unroll
  for (int c = 0; c < CW; ++c) b0[c] = *reinterpret_cast<const u32x4 *>(pb + c * 1024);
  a0 = *reinterpret_cast<const u32x4 *>(pa);
  a1 = *reinterpret_cast<const u32x4 *>(pa + 1024);
  uint32_t cur = 0, nxt = kSlot;
  // One k-step.  Everything else a row needs - fragments ahead (the weight tile two rows on; behind the barrier the next step's column tiles), its
  // share of the transfers - is issued BETWEEN its products, spread over them (TileOrder): a product keeps the matrix core busy for 16 clocks, in
  // which the wave can issue a few other instructions, and where a SIMD has one wave nobody else would.
  auto step = [&](u32x4(&b)[CW], u32x4(&bn)[CW]) __attribute__((always_inline)) {
    const unsigned char *pac = pa + cur, *pan = pa + nxt, *pbn = pb + nxt;
    unrolled<AW>([&](auto row) __attribute__((always_inline)) {
      constexpr int t = decltype(row)::value;
      if constexpr (t == TB) {
        wait_vmcnt<(NB - 3) * OPS>();                              // step s + 1 has arrived (this wave's part)
        asm volatile("s_barrier" ::: "memory");                    // everybody's part; and nobody reads step s - 1 any more
        ++fs;
        fslot = fslot + kSlot == kRing ? 0u : fslot + kSlot;
      }
      u32x4 an;
      unrolled<CW>([&](auto column) __attribute__((always_inline)) {
        constexpr int c = decltype(column)::value;
        if constexpr (T::kAcc) tile_mul<c == 0>(acc[t][c], a0, b[c]);
        else acc[t][c] = fast_mfma(a0, b[c], acc[t][c]);
        __builtin_amdgcn_sched_barrier(0);
        unrolled<TileOrder<T>::kMost>([&](auto place) __attribute__((always_inline)) {
          constexpr int op = kOrder.op[t * CW + c][decltype(place)::value];
          if constexpr (op == kOpWeights) an = *reinterpret_cast<const u32x4 *>(t + 2 < AW ? pac + (t + 2) * 1024 : pan + (t + 2 - AW) * 1024);
          else if constexpr (op >= kOpTransfer) transfer(op - kOpTransfer);
          else if constexpr (op >= kOpColumn) bn[op - kOpColumn] = *reinterpret_cast<const u32x4 *>(pbn + (op - kOpColumn) * 1024);
          if constexpr (op != kOpNone) __builtin_amdgcn_sched_barrier(0);      // it stays here
        });
      });
      a0 = a1;
      a1 = an;
    });
    cur = nxt;
    nxt = nxt + kSlot == kRing ? 0u : nxt + kSlot;
  };
  int s = 0;
  for (; s + 1 < steps; s += 2) {
    step(b0, b1);
    step(b1, b0);
  }
  if (s < steps) step(b0, b1);
  wait_vmcnt<0>();                                                 // nothing may land in LDS after the ring changes hands
  constexpr int rpt = SINGLE ? 16 : 8;
  float *tab = reinterpret_cast<float *>(smem);                    // 1/rms of the block's rows, one round trip for all of them
  __syncthreads();
  if (ks == 1 && g.scale_tag) {
    for (int i = threadIdx.x; i < TC * rpt; i += 64 * NW) tab[i] = bat_row_scale(g, blk * TC * rpt + i);
    __syncthreads();
  }
  const int tile0 = grp * TA + wa * AW, ct0 = blk * TC + wc * CW;
  tile_end<T, SINGLE>(g, acc, tile0, n_tiles, ct0, wc, tab, ks, run, part, lane);
}

// Second half of a split reduction: four adjacent lanes take a row's 16 columns of a unit; a wave two (unit, column tile) pairs, one if a
// column tile has 16 rows.  The runs are added in their order.
__global__ __launch_bounds__(256) void bat_split_finish(BatGemm g, int ks, const float *part) {
  const int lane = threadIdx.x & 63, rpt = g.single ? 16 : 8;
  const int per_wave = 16 / rpt;
  const int waves_per_ct = (g.n_units + per_wave - 1) / per_wave;
  const int w = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (w >= waves_per_ct * g.CT) return;                            // uniform over the wave
  const int ct = w / waves_per_ct, q = lane & 3;                   // neighbouring waves: neighbouring columns of the same rows
  const int jr = (lane >> 2) & (rpt - 1);
  int unit = (w - ct * waves_per_ct) * per_wave + (lane >> 2) / rpt;
  const bool on = unit < g.n_units;
  unit = min(unit, g.n_units - 1);
  const int m = ct * rpt + jr;
  const f32x4 x = tile_old_x(g, unit, m, q), gain = tile_gain(g, unit, q);
  const float sc = bat_row_scale(g, m);
  const size_t run = (size_t)g.CT * rpt * g.n_units * 16;
  const float *mine = part + (size_t)min(m, g.M - 1) * (g.n_units * 16) + unit * 16 + 4 * q;
  f32x4 s = f32x4{0.f, 0.f, 0.f, 0.f};
  for (int k0 = 0; k0 < ks; k0 += 8) {                             // eight runs requested together
    f32x4 v[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) v[k] = *reinterpret_cast<const f32x4 *>(mine + (size_t)min(k0 + k, ks - 1) * run);
#pragma unroll
    for (int k = 0; k < 8; ++k)
      if (k0 + k < ks) s += v[k];
  }
  if (g.single) tile_emit<true, true>(g, unit, ct, jr, q, s, s, sc, x, gain, on);
  else tile_emit<true, false>(g, unit, ct, jr, q, s, s, sc, x, gain, on);
}

// Greedy bin after the last of every episode's n new rows (and that row's logits), straight from the LM head's runs: their sums are added in
// their order and scaled as bat_split_finish does it, for the one row per episode that is wanted, without its launch (prefill of 276
// rows and decode steps of more than 8 episodes, 4 to 5 us per call).  row0: rows of the call in front of part's first.  Otherwise as last_row_argmax.
__global__ __launch_bounds__(256) void last_row_argmax_runs(BatGemm g, int ks, const float *part, int row0, int n, int32_t *pred,
                                                            float *last_logits, const int32_t *prefix_len, int cap, unsigned *err) {
  __shared__ float s_best[4];
  __shared__ int s_bin[4];
  const int b = blockIdx.x, tid = threadIdx.x, n_bins = g.n_units * 16;
  if (episode_overflows(prefix_len, b, n, cap)) {
    if (last_logits)
      for (int t = tid; t < n_bins; t += 256) last_logits[(size_t)b * n_bins + t] = __uint_as_float(0x7FC00000u);
    if (tid == 0) {
      pred[b] = -1;
      atomicOr(err, kErrOverflow);
    }
    return;
  }
  const int m = b * n + n - 1 - row0;
  const float sc = bat_row_scale(g, m);
  const size_t run = (size_t)g.CT * (g.single ? 16 : 8) * n_bins;
  float best = -INFINITY;
  int bi = 0x7FFFFFFF;
  for (int t = tid; t < n_bins; t += 256) {
    const float *mine = part + (size_t)m * n_bins + t;
    float s = 0.f;
    for (int k0 = 0; k0 < ks; k0 += 8) {                           // eight runs requested together
      float v[8];
#pragma unroll
      for (int k = 0; k < 8; ++k) v[k] = mine[(size_t)min(k0 + k, ks - 1) * run];
#pragma unroll
      for (int k = 0; k < 8; ++k)
        if (k0 + k < ks) s += v[k];
    }
    s *= sc;
    if (last_logits) last_logits[(size_t)b * n_bins + t] = s;
    if (s != s) s = -INFINITY;
    if (s > best || (s == best && t < bi)) { best = s; bi = t; }
  }
  const float top = wave_max(best);
  bi = wave_argmax(best, bi);
  if ((tid & 63) == 0) {
    s_best[tid >> 6] = top;
    s_bin[tid >> 6] = bi;
  }
  __syncthreads();
  if (tid != 0) return;
  best = s_best[0];
  bi = s_bin[0];
  for (int w = 1; w < 4; ++w)
    if (s_best[w] > best || (s_best[w] == best && s_bin[w] < bi)) { best = s_best[w]; bi = s_bin[w]; }
  pred[b] = bi == 0x7FFFFFFF ? 0 : bi;
}

}  // namespace heisd
