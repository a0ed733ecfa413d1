// The retrieval branch's nearest-neighbour search (paper App. C: C.1 database construction, C.2 performance): cosine Top-K of a query embedding
// over the database of L2-normalised embeddings, as an exact brute-force scan.  The database is read
// once per group of up to 64 queries (2.4 GB at the paper's size: an HBM stream), the scores go to
// a small buffer, and the K best per query are selected in two rounds.
#pragma once
#include "heisd_common.h"

namespace heisd {

constexpr int kScanThreads = 512;      // 8 wavefronts per workgroup
constexpr int kTopChunk = 2048;        // scores per workgroup in the first selection round
constexpr int kTopMaxK = 64;

// scores[q][i] = <db[i], queries[q]>, q < NQ.  A wavefront takes two database rows per iteration (the
// query slices it reads from LDS serve both); lane l covers elements 256 t + 4 l .. + 3 of a row, one
// 8-byte load each, so a wavefront's loads are 512 contiguous bytes.
template <int NQ>
__global__ __launch_bounds__(kScanThreads) void retrieve_scores(const uint16_t *db, long long N, int d, const float *queries,
                                                               float *scores, long long ld_scores) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  float *qs = reinterpret_cast<float *>(smem);          // [NQ][d]
  const int tid = threadIdx.x, lane = tid & 63;
  for (int i = tid * 4; i < NQ * d; i += kScanThreads * 4)
    *reinterpret_cast<float4 *>(qs + i) = *reinterpret_cast<const float4 *>(queries + i);
  __syncthreads();
  const long long waves = (long long)gridDim.x * (kScanThreads / 64);
  const long long gw = (long long)blockIdx.x * (kScanThreads / 64) + (tid >> 6);
  const int steps = (d + 255) / 256;
  for (long long pr = gw; 2 * pr < N; pr += waves) {
    const long long r0 = 2 * pr, r1 = min(2 * pr + 1, N - 1);       // an odd tail computes its last row twice
    const uint16_t *p0 = db + r0 * d, *p1 = db + r1 * d;
    float acc0[NQ], acc1[NQ];
#pragma unroll
    for (int q = 0; q < NQ; ++q) acc0[q] = acc1[q] = 0.f;
#pragma unroll 4
    for (int t = 0; t < steps; ++t) {
      const int c = t * 256 + lane * 4;
      if (c < d) {
        const uint2 a = *reinterpret_cast<const uint2 *>(p0 + c);
        const uint2 b = *reinterpret_cast<const uint2 *>(p1 + c);
        const float a0 = __uint_as_float(a.x << 16), a1 = __uint_as_float(a.x & 0xFFFF0000u);
        const float a2 = __uint_as_float(a.y << 16), a3 = __uint_as_float(a.y & 0xFFFF0000u);
        const float b0 = __uint_as_float(b.x << 16), b1 = __uint_as_float(b.x & 0xFFFF0000u);
        const float b2 = __uint_as_float(b.y << 16), b3 = __uint_as_float(b.y & 0xFFFF0000u);
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
          const float4 w = *reinterpret_cast<const float4 *>(qs + q * d + c);
          acc0[q] = fmaf(a0, w.x, fmaf(a1, w.y, fmaf(a2, w.z, fmaf(a3, w.w, acc0[q]))));
          acc1[q] = fmaf(b0, w.x, fmaf(b1, w.y, fmaf(b2, w.z, fmaf(b3, w.w, acc1[q]))));
        }
      }
    }
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
      const float s0 = wave_sum(acc0[q]), s1 = wave_sum(acc1[q]);
      if (lane == 0) {
        scores[q * ld_scores + r0] = s0;
        scores[q * ld_scores + r1] = s1;
      }
    }
  }
}

// ---- three or more queries: the scan on the matrix cores ----------------------------------------------
// scores[q][i] = <db[i], queries[q]> for up to 16 QT queries per launch, with the database streamed once.
// A tile of 16 database rows is the A operand of v_mfma_f32_16x16x32_bf16 straight from memory; the queries are the
// B operand, each fp32 value as THREE bf16 parts that add up to it exactly (8 + 8 + 8 bits of its 24, cut off and not
// rounded, so that no part overflows): every product is the fp32 product and nothing of a query is lost.  The
// products of the leading part are summed by themselves, and every FLUSH k-steps their sum goes into a total
// whose rounding error is kept (a two-sum) together with the small sum of the other parts.
// A workgroup (one per compute unit) owns a contiguous range of tiles and walks them in passes of 8 waves x NT tiles; all waves
// cut the query parts of the next chunk of k-steps and put them into LDS (double buffered).  What it is bound by: reading
// (6 TB/s with the loads alone), and beside it what the queries cost a compute unit, whose loads share one path
// with about 64 KB in flight: hence 16 tiles per reading of the queries, both halves of a 128-byte line requested
// together (459 instead of 510 us at 4 queries).  Four waves that only
// fill and four that only multiply measured slower (460 and 646 us against 399 and 563 us on the same data).
// Every row is walked from its first column on, in every workgroup: equal entries of the database have equal scores, to the
// bit, and tie.  (Workgroups that start at different columns spread the reading of the queries over the L2's channels, but
// add up in different orders: 8 queries of 4096 x 100000 entries 166 -> 157 us, of 2048 x 200000 173 -> 167, elsewhere nothing.)
// 273465 x 4352, whole calls: 4 queries 507 -> 411 us, 16: 1950 -> 431 us, 64: 7734 -> 689 us.
// With 17 queries and more it is not reading that bounds it but what goes with the products (273465 x 4352, 64 queries: matrix cores busy 45 % of
// the time, other vector instructions - the totals, the cutting of the queries - another 28 %, and waits between two barriers): three
// tiles per wave share one reading and cutting of the queries.  With 64 queries the ring is half as deep and a chunk has
// two k-steps, which is what registers and LDS allow.  64 queries 675 -> 607 us (601 with shorter cutting), 24 queries
// 486 -> 448.
constexpr int kScanMulWaves = kScanThreads / 64;
template <int QT, int NT>
constexpr int scan_ring() { return QT == 4 && NT > 2 ? 4 : 8; }       // k-steps of database rows a wave requests ahead
template <int QT, int NT>
constexpr int scan_chunk() { return QT == 4 ? (NT > 2 ? 2 : 4) : 8; }     // k-steps of query parts per LDS buffer (two buffers)
template <int QT, int NT>
constexpr bool scan_sums_in_lds() { return QT * NT > 4; }       // the totals, where there are no registers left for them
template <int QT, int NT>
constexpr size_t scan_mfma_lds_bytes() {
  return (size_t)2 * scan_chunk<QT, NT>() * 3 * QT * 1024 + (scan_sums_in_lds<QT, NT>() ? (size_t)kScanMulWaves * NT * QT * 1024 : 0);
}

typedef unsigned int ru32x4 __attribute__((ext_vector_type(4)));
typedef ru32x4 ru32x4_a8 __attribute__((aligned(8)));      // rows start at multiples of 8 bytes
typedef const ru32x4_a8 __attribute__((address_space(1))) *gptr_ru4;
typedef const f32x4 __attribute__((address_space(1))) *gptr_f4;
typedef const float __attribute__((address_space(1))) *gptr_f1;

// 8 fp32 values as three fragments of 8 bf16 that add up to them exactly.  An infinity or a NaN (made a quiet one, whose bit is in
// the leading part) leaves NaN in the others, which only meet totals that it makes infinite or NaN itself: those are taken without them.
// (Guards against that were every sixth of the vector instructions that are no products: 64 queries of 4352 x 273465 entries 615 -> 601 us.)
__device__ __forceinline__ void split3(const float (&x)[8], ru32x4 (&part)[3]) {
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    uint32_t b[3][2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const float v = __builtin_canonicalizef(x[2 * i + h]);
      const float r1 = v - __uint_as_float(__float_as_uint(v) & 0xFFFF0000u);
      b[0][h] = __float_as_uint(v);
      b[1][h] = __float_as_uint(r1);
      b[2][h] = __float_as_uint(r1 - __uint_as_float(b[1][h] & 0xFFFF0000u));
    }
#pragma unroll
    for (int p = 0; p < 3; ++p) part[p][i] = __builtin_amdgcn_perm(b[p][1], b[p][0], 0x07060302u);   // the two upper halves
  }
}

template <int QT, int NT, int FLUSH>
__global__ __launch_bounds__(kScanThreads) __attribute__((amdgpu_waves_per_eu(2, 2))) void retrieve_scan_mfma(
    const uint16_t *db, long long N, int d, const float *queries, int nq, float *scores, long long ld_scores) {
  constexpr bool SUMS_IN_LDS = scan_sums_in_lds<QT, NT>();
  constexpr int RING = scan_ring<QT, NT>(), C = scan_chunk<QT, NT>(), BUF = C * 3 * QT * 1024, CPR = RING / C;
  constexpr int EVERY = FLUSH > RING ? FLUSH / RING : 1;             // revolutions between two totals, if one is too short
  static_assert(RING % C == 0 && C % 2 == 0 && (FLUSH <= RING ? RING % FLUSH == 0 : FLUSH % RING == 0), "revolutions");
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lr = lane & 15, lg = lane >> 4;
  const long long tiles = (N + 15) / 16, per = tiles / gridDim.x, extra = tiles % gridDim.x;
  const long long t0 = blockIdx.x * per + min((long long)blockIdx.x, extra);
  const int mine = (int)(per + (blockIdx.x < extra ? 1 : 0));       // tiles of this workgroup
  const int passes = (mine + kScanMulWaves * NT - 1) / (kScanMulWaves * NT);
  // Whole revolutions of the ring (256 or 128 values of a row) run through a loop without a branch; what is left of a row
  // (less than a revolution, the last k-step cut short by a multiple of 4) is added behind it, chunk by chunk.
  const int revs = d / (RING * 32), main_chunks = revs * CPR;
  const int chunks = (d + 32 * C - 1) / (32 * C);

  // Query parts of a chunk: thread f takes 8 consecutive values of one query (a lane's B fragment) at a time, requests them
  // two chunks before they are multiplied and cuts them into parts one chunk before.  (A wave's loads return in order; at that
  // distance the wait for them covers only database rows that are due anyway.)
  constexpr int PIECES = C * QT * 64 / kScanThreads;
  static_assert(C * QT * 64 % kScanThreads == 0, "pieces");
  f32x4 qv[PIECES][2];
  int ahead = 0, k_held = 0;                                        // next chunk to request; first k of the one in qv
  auto fill_load = [&]() __attribute__((always_inline)) {
    k_held = ahead * C * 32;
#pragma unroll
    for (int p = 0; p < PIECES; ++p) {
      const int f = tid + p * kScanThreads, qt = (f >> 6) % QT, s = (f >> 6) / QT, k = k_held + s * 32 + (f >> 4 & 3) * 8;
      const uint32_t q0 = (uint32_t)(min(qt * 16 + (f & 15), nq - 1) * d);                // columns past the last query repeat it
      qv[p][0] = *reinterpret_cast<gptr_f4>(reinterpret_cast<gptr_f1>(reinterpret_cast<uintptr_t>(queries)) + (q0 + min(k, d - 4)));
      qv[p][1] = *reinterpret_cast<gptr_f4>(reinterpret_cast<gptr_f1>(reinterpret_cast<uintptr_t>(queries)) + (q0 + min(k + 4, d - 4)));
    }
    ahead = ahead + 1 == chunks ? 0 : ahead + 1;
  };
  auto fill_store = [&](int g) __attribute__((always_inline)) {
    unsigned char *buf = smem + (size_t)(g & 1) * BUF;
#pragma unroll
    for (int p = 0; p < PIECES; ++p) {
      const int f = tid + p * kScanThreads, qt = (f >> 6) % QT, s = (f >> 6) / QT, k = k_held + s * 32 + (f >> 4 & 3) * 8;
      const bool in0 = k < d, in1 = k + 4 < d;                      // past the row's end: zero (d is a multiple of 4)
      const float x[8] = {in0 ? qv[p][0].x : 0.f, in0 ? qv[p][0].y : 0.f, in0 ? qv[p][0].z : 0.f, in0 ? qv[p][0].w : 0.f,
                          in1 ? qv[p][1].x : 0.f, in1 ? qv[p][1].y : 0.f, in1 ? qv[p][1].z : 0.f, in1 ? qv[p][1].w : 0.f};
      ru32x4 part[3];
      split3(x, part);
#pragma unroll
      for (int a = 0; a < 3; ++a) *reinterpret_cast<ru32x4 *>(buf + (size_t)((s * 3 + a) * QT + qt) * 1024 + (f & 63) * 16) = part[a];
    }
  };

  f32x4 *const lsum = reinterpret_cast<f32x4 *>(smem + 2 * BUF + (size_t)wave * NT * QT * 1024) + lane;
  int g = 0;                                                        // chunks done
  struct Place {                                                    // this wave's tiles of a pass
    const uint16_t *row[NT];
    long long first;
    int cnt;
  };
  int done = 0;
  auto place = [&](int pass) __attribute__((always_inline)) {
    Place p;
    const int left = max(passes - pass, 1);
    const int now = (mine - done + left - 1) / left;                // spread evenly over the passes and waves
    const int share = now / kScanMulWaves, rest = now % kScanMulWaves;
    p.cnt = share + (wave < rest ? 1 : 0);
    p.first = t0 + done + wave * share + min(wave, rest);
    done += now;
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      const long long tile = min(p.first + min(t, max(p.cnt - 1, 0)), tiles - 1);  // a wave with fewer tiles repeats its last
      p.row[t] = db + min(tile * 16 + lr, N - 1) * (long long)d + lg * 8;
    }
    return p;
  };
  auto ld = [&](const uint16_t *row, int s) __attribute__((always_inline)) {
    return *reinterpret_cast<gptr_ru4>(reinterpret_cast<uintptr_t>(row + s * 32));
  };
  ru32x4 A[RING][NT];
  Place now = place(0);
  fill_load();
  fill_store(0);
  fill_load();
  if (revs > 0)
#pragma unroll
    for (int u = 0; u < RING; ++u)
#pragma unroll
      for (int t = 0; t < NT; ++t) A[u][t] = ld(now.row[t], u);
  lds_barrier();                                                    // chunk 0 is in LDS
  for (int pass = 0; pass < passes; ++pass) {
    float zero = 0.f;
    asm volatile("" : "+v"(zero));                                  // a constant vector for LDS would be kept, in scratch, over the loop
    f32x4 hi[NT][QT], lo[NT][QT], sum[SUMS_IN_LDS ? 1 : NT][SUMS_IN_LDS ? 1 : QT];
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int q = 0; q < QT; ++q) {
        hi[t][q] = lo[t][q] = f32x4{0.f, 0.f, 0.f, 0.f};
        if (SUMS_IN_LDS) lsum[(t * QT + q) * 64] = f32x4{zero, zero, zero, zero};
        else sum[t][q] = hi[t][q];
      }
    // One k-step: the QT fragments of the next part are requested from LDS before the products of the current one.
    auto products = [&](const ru32x4 (&a_)[NT], int s, const unsigned char *buf) __attribute__((always_inline)) {
      ru32x4 B[2][QT];
#pragma unroll
      for (int q = 0; q < QT; ++q) B[0][q] = *reinterpret_cast<const ru32x4 *>(buf + (size_t)(s * 3 * QT + q) * 1024);
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        if (a < 2)
#pragma unroll
          for (int q = 0; q < QT; ++q) B[(a + 1) & 1][q] = *reinterpret_cast<const ru32x4 *>(buf + (size_t)((s * 3 + a + 1) * QT + q) * 1024);
        __builtin_amdgcn_sched_barrier(0);                          // requested here, not at their use
#pragma unroll
        for (int q = 0; q < QT; ++q)
#pragma unroll
          for (int t = 0; t < NT; ++t) {
            f32x4 &acc = a == 0 ? hi[t][q] : lo[t][q];
            acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a_[t]), __builtin_bit_cast(bf16x8, B[a & 1][q]), acc, 0, 0, 0);
          }
      }
    };
    auto flush = [&]() __attribute__((always_inline)) {             // sum += hi, the rounding error goes to lo
#pragma unroll
      for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int q = 0; q < QT; ++q) {
          const f32x4 was = SUMS_IN_LDS ? lsum[(t * QT + q) * 64] : sum[t][q];
          f32x4 is;
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const float a = was[i], b = hi[t][q][i], s = a + b, bb = s - a;
            lo[t][q][i] += (a - (s - bb)) + (b - bb);
            is[i] = s;
            hi[t][q][i] = 0.f;
          }
          if (SUMS_IN_LDS) lsum[(t * QT + q) * 64] = is;
          else sum[t][q] = is;
        }
    };
    const Place then = place(pass + 1);                             // after the last pass: valid rows, never used
    for (int rev = 0; rev < revs; ++rev) {
      const bool last = rev == revs - 1;                            // the ring is refilled from the start of the next pass
      const uint16_t *from[NT];
#pragma unroll
      for (int t = 0; t < NT; ++t) from[t] = (last ? then.row[t] : now.row[t]) + (last ? 0 : rev + 1) * RING * 32;
#pragma unroll
      for (int cc = 0; cc < CPR; ++cc) {
        fill_store(g + 1);
        fill_load();
        __builtin_amdgcn_sched_barrier(0);
        const unsigned char *buf = smem + (size_t)(g & 1) * BUF + lane * 16;
#pragma unroll
        for (int s = 0; s < C; ++s) {
          const int u = cc * C + s;
          products(A[u], s, buf);
          __builtin_amdgcn_sched_barrier(0);                        // a fragment's registers are free when it is requested anew
          if (u & 1)                                                // two k-steps are one 128-byte line of every row:
#pragma unroll
            for (int t = 0; t < NT; ++t) {                          // requested together, it crosses to the L1 once
              A[u - 1][t] = ld(from[t], u - 1);
              A[u][t] = ld(from[t], u);
            }
          __builtin_amdgcn_sched_barrier(0);                        // the requests stay in this step
          if (FLUSH <= RING ? (u + 1) % FLUSH == 0 : (u == RING - 1 && ((rev + 1) % EVERY == 0 || last))) flush();
        }
        lds_barrier();                                              // the next chunk is in LDS, this one is free
        ++g;
      }
    }
    for (int c = main_chunks; c < chunks; ++c) {                    // the rest of the rows
      fill_store(g + 1);
      fill_load();
      const unsigned char *buf = smem + (size_t)(g & 1) * BUF + lane * 16;
#pragma unroll
      for (int s = 0; s < C; ++s) {
        const int k = (c * C + s) * 32 + lg * 8;
        ru32x4 rest[NT];                                            // the ring already holds the next pass
#pragma unroll
        for (int t = 0; t < NT; ++t) {
          uint2 a = make_uint2(0u, 0u), b = a;
          if (k < d) a = *reinterpret_cast<const uint2 *>(now.row[t] + (c * C + s) * 32);
          if (k + 4 < d) b = *reinterpret_cast<const uint2 *>(now.row[t] + (c * C + s) * 32 + 4);
          rest[t] = ru32x4{a.x, a.y, b.x, b.y};
        }
        products(rest, s, buf);
        if ((s + 1) % FLUSH == 0 || s == C - 1) flush();
      }
      lds_barrier();
      ++g;
    }
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      if (t >= now.cnt) continue;                                     // uniform over the wave
      // lane: rows r0 .. r0+3 against query lr of its group.  (The group's part of the address is uniform: a lane address per group would
      // be kept, in scratch, over the loop.)
      const long long r0 = (now.first + t) * 16 + lg * 4, at = lr * ld_scores + r0;
#pragma unroll
      for (int q = 0; q < QT; ++q) {
        if (q * 16 + lr >= nq) continue;
        f32x4 v;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          // An infinite or NaN element, of a row or a query, is in the leading parts' total as it should be; the other parts (its own, its
          // product with a part that is zero, the rounding error of an infinite total) would make a NaN of it.  (An overflow stays one.)
          const float total = SUMS_IN_LDS ? lsum[(t * QT + q) * 64][i] : sum[t][q][i];
          v[i] = (__float_as_uint(total) & 0x7F800000u) == 0x7F800000u ? total : total + lo[t][q][i];
        }
        *reinterpret_cast<f32x4 *>(scores + q * 16 * ld_scores + at) = v;          // rows past N stay inside this query's padded row
      }
    }
    wait_vmcnt_all();                                               // the loop's waits can count exactly again (stores count, too)
    now = then;
  }
}

// (value, index) order of the search: higher value first, equal values by lower index; a NaN counts as -inf.
__device__ __forceinline__ bool top_before(float v, int i, float bv, int bi) { return v > bv || (v == bv && i < bi); }

// The K best of `n` (value, index) pairs (in LDS or in global memory), by K rounds of a workgroup-wide arg-max; the
// winner of a round is taken out.  Results to out_val/out_idx [K] (index -1, value -inf when fewer
// than K pairs exist).  All 256 threads call this.
__device__ __forceinline__ void top_select(float *val, const int *idx, int n, int K, float *out_val, int *out_idx,
                                           float *red_v, int *red_i, int *red_p) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  for (int k = 0; k < K; ++k) {
    float bv = -INFINITY;
    int bi = 0x7FFFFFFF, bp = -1;
    for (int p = tid; p < n; p += 256) {
      const float v = val[p];
      const int i = idx ? idx[p] : p;
      if (i >= 0 && (top_before(v, i, bv, bi) || (bp < 0 && v == -INFINITY))) { bv = v; bi = i; bp = p; }
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
      const float ov = __shfl_xor(bv, o, kWave);
      const int oi = __shfl_xor(bi, o, kWave), op = __shfl_xor(bp, o, kWave);
      if (op >= 0 && (bp < 0 || top_before(ov, oi, bv, bi))) { bv = ov; bi = oi; bp = op; }
    }
    if (lane == 0) { red_v[wave] = bv; red_i[wave] = bi; red_p[wave] = bp; }
    __syncthreads();
    if (tid == 0) {
      for (int w = 1; w < 4; ++w)
        if (red_p[w] >= 0 && (red_p[0] < 0 || top_before(red_v[w], red_i[w], red_v[0], red_i[0]))) {
          red_v[0] = red_v[w]; red_i[0] = red_i[w]; red_p[0] = red_p[w];
        }
      if (red_p[0] >= 0) {
        out_val[k] = red_v[0];
        out_idx[k] = red_i[0];
        val[red_p[0]] = -INFINITY;
        // taken out: an index of -1 can never be chosen again
        if (idx) const_cast<int *>(idx)[red_p[0]] = -1;
      } else {
        out_val[k] = -INFINITY;
        out_idx[k] = -1;
      }
    }
    __syncthreads();
  }
}

// First round: one wavefront per chunk of kTopChunk scores of one query, all of them in registers (32 per lane) as integers
// of the same order.  A lane keeps the best of each of its four groups of 8; a round finds the wave's best lane by
// lane exchanges in the vector ALU, and only the group the winner came from is looked through again.  No LDS, no
// barrier: K = 4 of 64 x 273465 scores 79 -> 25 us (K rounds of a workgroup over LDS before), which is mostly
// the reading of the scores.  Among equal scores the lowest index wins; NaN counts as -inf.
constexpr uint32_t kTopTaken = 0u;       // below every score's integer: nothing left
__device__ __forceinline__ uint32_t top_order(float v) {
  const uint32_t u = __float_as_uint(v + 0.f);                    // -0 and +0 are equal
  if (v != v) return 0x007FFFFFu;                                 // NaN: as -inf
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
__device__ __forceinline__ float top_value(uint32_t o) { return __uint_as_float((o & 0x80000000u) ? (o & 0x7FFFFFFFu) : ~o); }
template <int CTRL>
__device__ __forceinline__ uint32_t dpp_move_u(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xf, 0xf, true);
}
__device__ __forceinline__ uint32_t wave_max_u(uint32_t v) {
  v = max(v, dpp_move_u<kDppXor1>(v));
  v = max(v, dpp_move_u<kDppXor2>(v));
  v = max(v, dpp_move_u<kDppHalfMirror>(v));
  v = max(v, dpp_move_u<kDppMirror>(v));
  const uint32_t a = max((uint32_t)__builtin_amdgcn_readlane((int)v, 0), (uint32_t)__builtin_amdgcn_readlane((int)v, 16));
  const uint32_t b = max((uint32_t)__builtin_amdgcn_readlane((int)v, 32), (uint32_t)__builtin_amdgcn_readlane((int)v, 48));
  return max(a, b);
}

__global__ __launch_bounds__(256) void retrieve_top_chunks(const float *scores, long long ld_scores, long long N, int K,
                                                          float *cand_val, int *cand_idx, int n_chunks) {
  constexpr int PER = kTopChunk / kWave, GROUPS = 4, GS = PER / GROUPS;
  const int lane = threadIdx.x & 63, chunk = blockIdx.x * 4 + (threadIdx.x >> 6), q = blockIdx.y;
  if (chunk >= n_chunks) return;                                  // uniform over the wave
  const long long base = (long long)chunk * kTopChunk;
  const int n = (int)min((long long)kTopChunk, N - base);
  const float *src = scores + q * ld_scores + base;               // element j of this lane: 64 j + lane of the chunk
  uint32_t v[PER];
#pragma unroll
  for (int j = 0; j < PER; ++j) v[j] = __float_as_uint(src[min(j * kWave + lane, n - 1)]);
#pragma unroll
  for (int j = 0; j < PER; ++j) v[j] = j * kWave + lane < n ? top_order(__uint_as_float(v[j])) : kTopTaken;
  uint32_t best[GROUPS];
#pragma unroll
  for (int g = 0; g < GROUPS; ++g) {
    best[g] = v[g * GS];
#pragma unroll
    for (int j = 1; j < GS; ++j) best[g] = max(best[g], v[g * GS + j]);
  }
  float *out_val = cand_val + ((size_t)q * n_chunks + chunk) * K;
  int *out_idx = cand_idx + ((size_t)q * n_chunks + chunk) * K;
  for (int k = 0; k < K; ++k) {
    uint32_t mine = max(max(best[0], best[1]), max(best[2], best[3]));
    const uint32_t top = wave_max_u(mine);
    if (top == kTopTaken) {                                       // fewer than K scores in this chunk
      for (int r = k + lane; r < K; r += kWave) { out_val[r] = -INFINITY; out_idx[r] = -1; }
      return;
    }
    // the lowest element with that score: 64 j + lane, so the lowest j first, then the lowest lane
    int at = PER;
#pragma unroll
    for (int j = PER - 1; j >= 0; --j) at = v[j] == top ? j : at;
    const unsigned long long has = __ballot(mine == top);
    int j0 = PER, winner = 0;
    for (unsigned long long m = has; m; m &= m - 1) {             // one lane, or a few with the same score
      const int l = __ffsll((long long)m) - 1, jl = __builtin_amdgcn_readlane(at, l);
      if (jl < j0) { j0 = jl; winner = l; }
    }
    if (lane == 0) {
      out_val[k] = top_value(top);
      out_idx[k] = (int)(base + j0 * kWave + winner);
    }
    // take it out
    if (lane == winner)
#pragma unroll
      for (int j = 0; j < PER; ++j) v[j] = j == j0 ? kTopTaken : v[j];
#pragma unroll
    for (int g = 0; g < GROUPS; ++g)
      if (j0 / GS == g) {                                         // uniform
        uint32_t b = v[g * GS];
#pragma unroll
        for (int j = 1; j < GS; ++j) b = max(b, v[g * GS + j]);
        best[g] = b;
      }
  }
}

// Second round: the chunks' lists are sorted, so the K best of a query are a merge of their heads.  One workgroup per query; a
// thread holds the heads of up to kMergeLists lists (list l belongs to thread l % 256), and each head's successor is
// already on its way when the head is taken.  Also fetches the winners' payload rows.
constexpr int kMergeLists = 4;
__global__ __launch_bounds__(256) void retrieve_top_merge_lists(const float *cand_val, const int *cand_idx, int n_chunks, int K,
                                                               float *top_val, int *top_idx, const int32_t *payload,
                                                               int payload_len, int32_t *top_payload) {
  __shared__ unsigned long long red[2][4];
  __shared__ int picked[kTopMaxK];
  const int q = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const float *val = cand_val + (size_t)q * n_chunks * K;
  const int *idx = cand_idx + (size_t)q * n_chunks * K;
  // a head: score order in the upper half, the complement of the index below it (larger = better); 0 = list empty
  auto entry = [&](int l, int p) __attribute__((always_inline)) -> unsigned long long {
    if (l >= n_chunks || p >= K) return 0ull;
    const int i = idx[(size_t)l * K + p];
    const float v = val[(size_t)l * K + p];
    return i < 0 ? 0ull : ((unsigned long long)top_order(v) << 32) | (uint32_t)~i;
  };
  unsigned long long head[kMergeLists], next[kMergeLists];
  int pos[kMergeLists];
#pragma unroll
  for (int s = 0; s < kMergeLists; ++s) {
    head[s] = entry(tid + s * 256, 0);
    next[s] = entry(tid + s * 256, 1);
    pos[s] = 1;
  }
  for (int k = 0; k < K; ++k) {
    unsigned long long mine = head[0];
#pragma unroll
    for (int s = 1; s < kMergeLists; ++s) mine = mine > head[s] ? mine : head[s];
    const uint32_t hi = wave_max_u((uint32_t)(mine >> 32));
    const uint32_t lo = wave_max_u((uint32_t)(mine >> 32) == hi ? (uint32_t)mine : 0u);
    if (lane == 0) red[k & 1][wave] = ((unsigned long long)hi << 32) | lo;
    __syncthreads();
    unsigned long long top = red[k & 1][0];
#pragma unroll
    for (int w = 1; w < 4; ++w) top = top > red[k & 1][w] ? top : red[k & 1][w];
    if (tid == 0) {
      const int i = top ? (int)~(uint32_t)top : -1;
      top_val[(size_t)q * K + k] = top ? top_value((uint32_t)(top >> 32)) : -INFINITY;
      top_idx[(size_t)q * K + k] = i;
      picked[k] = i;
    }
#pragma unroll
    for (int s = 0; s < kMergeLists; ++s)
      if (top && head[s] == top) {                                // indices are distinct: one list of one thread
        head[s] = next[s];
        ++pos[s];
        next[s] = entry(tid + s * 256, pos[s]);
      }
  }
  if (payload && top_payload) {
    __syncthreads();
    for (int e = tid; e < K * payload_len; e += 256) {
      const int i = picked[e / payload_len];
      top_payload[(size_t)q * K * payload_len + e] = i >= 0 ? payload[(size_t)i * payload_len + e % payload_len] : -1;
    }
  }
}

// The second round for more lists than a workgroup holds heads of (over 2 million vectors): arg-max over all winners.
__global__ __launch_bounds__(256) void retrieve_top_merge(float *cand_val, int *cand_idx, int n_cand, int K, float *top_val,
                                                         int *top_idx, const int32_t *payload, int payload_len,
                                                         int32_t *top_payload) {
  __shared__ float red_v[4];
  __shared__ int red_i[4], red_p[4];
  const int q = blockIdx.x, tid = threadIdx.x;
  top_select(cand_val + (size_t)q * n_cand, cand_idx + (size_t)q * n_cand, n_cand, K, top_val + (size_t)q * K,
             top_idx + (size_t)q * K, red_v, red_i, red_p);
  if (payload && top_payload) {
    __threadfence_block();
    __syncthreads();
    for (int e = tid; e < K * payload_len; e += 256) {
      const int i = top_idx[(size_t)q * K + e / payload_len];
      top_payload[(size_t)q * K * payload_len + e] = i >= 0 ? payload[(size_t)i * payload_len + e % payload_len] : -1;
    }
  }
}

}  // namespace heisd
