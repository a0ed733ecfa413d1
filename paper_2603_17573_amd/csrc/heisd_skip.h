// The verify-skip decision (paper Sec. 4.1, Alg. 1): features of the final layer, their cosine
// similarity over pairs of trajectory points, the offline stage's minimum acceptable similarity and
// its point distance, and the per-episode decision that produces the skip mask the verify step
// consumes.  Small fp32 kernels.
#pragma once
#include "heisd_common.h"

namespace heisd {

// feat[b][:] = RMSNorm(x[m][:]; gain, eps) for row m = b * rows_per_ep + row[b] (the last row of the
// episode when `row` is null): the LM head's input of that row.  One workgroup per episode.
__global__ __launch_bounds__(256) void export_features(const float *x, const int32_t *row, int rows_per_ep, int d,
                                                      const float *gain, float eps, float *feat) {
  __shared__ float part[4];
  const int b = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  int r = row ? row[b] : rows_per_ep - 1;
  r = max(0, min(r, rows_per_ep - 1));
  const float *src = x + ((size_t)b * rows_per_ep + r) * d;
  float ss = 0.f;
  for (int c = tid * 4; c < d; c += 256 * 4) {
    const float4 v = *reinterpret_cast<const float4 *>(src + c);
    ss += v.x * v.x + v.y * v.y + v.z * v.z + v.w * v.w;
  }
  ss = wave_sum(ss);
  if (lane == 0) part[wave] = ss;
  __syncthreads();
  const float inv = rsqrtf((part[0] + part[1] + part[2] + part[3]) / (float)d + eps);
  for (int c = tid * 4; c < d; c += 256 * 4) {
    const float4 v = *reinterpret_cast<const float4 *>(src + c);
    const float4 g = *reinterpret_cast<const float4 *>(gain + c);
    *reinterpret_cast<float4 *>(feat + (size_t)b * d + c) = make_float4(v.x * inv * g.x, v.y * inv * g.y, v.z * inv * g.z, v.w * inv * g.w);
  }
}

// ---- one arithmetic for every similarity ------------------------------------------------------------
// The threshold min_S of the offline stage IS the similarity of one pair, and the online decision compares with >=: that
// pair itself has to pass.  So a similarity is the same bits whichever kernel computes it - the tile kernel, the
// kernel of a few pairs, the decision -, by one order of additions:
//   channel c = 512 r + 64 w + 16 g + 4 y + x   (w < 8; g, y, x < 4; channels past d count as zeros)
//   product   128 fp32 chains (w, y, x) of FMAs, r ascending and g ascending inside it: what v_mfma_f32_16x16x4_f32 does with k = g (checked
//             against chains of FMAs on 5 million elements, denormals, infinities and NaN among them: the same bits); the
//             sum over x in fp32, the rest in fp64: y, then w, as trees
//   lengths   512 fp32 chains (w, g, y, x) of the squares over r; the sum over x in fp32, the rest in fp64: g, y, then w, as trees
//   cosine    product / sqrt(length a x length b) in fp64, rounded once; 0 if either vector is all zero
// Error against 64 bits (2-norm, 300 x 300 x 4096) 2.3e-8; one wavefront's fp32 dot product and lengths 6.8e-8.
// A pair and its mirror image are the same bits (FMAs commute in their factors).
__device__ __forceinline__ float pair_cosine(double dot, double la, double lb) {
  return (la == 0. || lb == 0.) ? 0.f : (float)(dot / sqrt(la * lb));
}

__device__ __forceinline__ double sum4_tree(float a, float b, float c, float d) { return (double)((a + b) + (c + d)); }

// Sum over 32 lanes as the tree of neighbours, pairs of neighbours, ..: the same in all 32.  Exchanges in the vector ALU; in the
// mirrored halves every lane of the other half already holds that half's sum.
template <int CTRL>
__device__ __forceinline__ double dpp_add64(double v) {
  const uint64_t u = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)u, CTRL, 0xf, 0xf, true);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(u >> 32), CTRL, 0xf, 0xf, true);
  return v + __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}
__device__ __forceinline__ double half_wave_tree(double v) {
  v = dpp_add64<kDppXor1>(v);
  v = dpp_add64<kDppXor2>(v);
  v = dpp_add64<kDppHalfMirror>(v);
  v = dpp_add64<kDppMirror>(v);
  const uint64_t u = __builtin_bit_cast(uint64_t, v);
  const auto lo = __builtin_amdgcn_permlane16_swap((uint32_t)u, (uint32_t)u, false, false);
  const auto hi = __builtin_amdgcn_permlane16_swap((uint32_t)(u >> 32), (uint32_t)(u >> 32), false, false);
  return __builtin_bit_cast(double, ((uint64_t)hi[0] << 32) | lo[0]) + __builtin_bit_cast(double, ((uint64_t)hi[1] << 32) | lo[1]);
}

// Cosine of two d-vectors by 32 lanes (lane l = 4 w + y of them: four neighbours read 64 consecutive bytes); all 32 get it.
// Two groups of 512 channels are requested together.
__device__ __forceinline__ float half_wave_cosine(const float *a, const float *b, int d, int l) {
  float p[4] = {0.f, 0.f, 0.f, 0.f}, qa[4][4] = {}, qb[4][4] = {};         // [x], [g][x]
  auto take = [&](const f32x4 (&u)[4], const f32x4 (&v)[4]) __attribute__((always_inline)) {
#pragma unroll
    for (int g = 0; g < 4; ++g)
#pragma unroll
      for (int x = 0; x < 4; ++x) {
        p[x] = fmaf(u[g][x], v[g][x], p[x]);
        qa[g][x] = fmaf(u[g][x], u[g][x], qa[g][x]);
        qb[g][x] = fmaf(v[g][x], v[g][x], qb[g][x]);
      }
  };
  constexpr int U = 2;
  const int lane_c = (l >> 2) * 64 + (l & 3) * 4;
  int c = 0;
  for (; c + 512 * U <= d; c += 512 * U) {
    f32x4 u[U][4], v[U][4];
#pragma unroll
    for (int r = 0; r < U; ++r)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        u[r][g] = *reinterpret_cast<const f32x4 *>(a + lane_c + c + r * 512 + g * 16);
        v[r][g] = *reinterpret_cast<const f32x4 *>(b + lane_c + c + r * 512 + g * 16);
      }
    __builtin_amdgcn_sched_barrier(0);                         // all of them requested before the first is used
#pragma unroll
    for (int r = 0; r < U; ++r) take(u[r], v[r]);
  }
  for (; c < d; c += 512) {                                    // the last groups, the very last perhaps cut short
    f32x4 u[4], v[4];
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const int k = c + lane_c + g * 16;
      u[g] = *reinterpret_cast<const f32x4 *>(a + min(k, d - 4));
      v[g] = *reinterpret_cast<const f32x4 *>(b + min(k, d - 4));
      if (k >= d) u[g] = v[g] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    take(u, v);
  }
  double dot = sum4_tree(p[0], p[1], p[2], p[3]);
  double la = (sum4_tree(qa[0][0], qa[0][1], qa[0][2], qa[0][3]) + sum4_tree(qa[1][0], qa[1][1], qa[1][2], qa[1][3])) +
              (sum4_tree(qa[2][0], qa[2][1], qa[2][2], qa[2][3]) + sum4_tree(qa[3][0], qa[3][1], qa[3][2], qa[3][3]));
  double lb = (sum4_tree(qb[0][0], qb[0][1], qb[0][2], qb[0][3]) + sum4_tree(qb[1][0], qb[1][1], qb[1][2], qb[1][3])) +
              (sum4_tree(qb[2][0], qb[2][1], qb[2][2], qb[2][3]) + sum4_tree(qb[3][0], qb[3][1], qb[3][2], qb[3][3]));
  return pair_cosine(half_wave_tree(dot), half_wave_tree(la), half_wave_tree(lb));
}

// Floats as unsigned integers of the same order.
__device__ __forceinline__ uint32_t ordered_bits(float f) {
  const uint32_t u = __float_as_uint(f);
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
__device__ __forceinline__ float from_ordered_bits(uint32_t o) {
  return __uint_as_float((o & 0x80000000u) ? (o & 0x7FFFFFFFu) : ~o);
}

__global__ void skip_key_init(unsigned long long *key) { *key = ~0ull; }

// S[i][j] = cosine(a[i], b[j]).
// SAME (a and b are the same points): only pairs i <= j are computed, one off the diagonal is stored twice.
// With `key` given (offline stage of Alg. 1; SAME): every pair i < j whose similarity exceeds T offers
// (similarity, i, j - i) to a 64-bit minimum, so that the smallest similarity above T wins and, among
// equals, the pair found first by the algorithm's loops (i ascending, then distance ascending).
__device__ __forceinline__ unsigned long long pair_offer(float s, int i, int j) {
  return ((unsigned long long)ordered_bits(s) << 32) | ((unsigned long long)i << 16) | (unsigned long long)(j - i);
}

// A few pairs: 32 lanes per pair, one wave per workgroup: the pairs spread over the compute units.  Bound by the L1, which gives a
// pair's 2 x 4 d bytes at 64 bytes a clock.  Of two sets, consecutive workgroups of an XCD take the same columns against row after
// row of the other side, so that a column comes from that XCD's L2 (blockIdx.x % 8 is the XCD).
constexpr int kFewPerGroup = 2;
template <bool SAME>
__global__ __launch_bounds__(kFewPerGroup * 32) __attribute__((amdgpu_waves_per_eu(3, 3))) void pair_similarity_few(const float *a, const float *b, int n, int m, int d, float *S,
                                                                         float T, unsigned long long *key) {
  int i = blockIdx.y, j = i + blockIdx.x * kFewPerGroup;
  if (!SAME) {
    i = (int)(blockIdx.x / 8 % (unsigned)n);
    j = (int)(blockIdx.x / 8 / (unsigned)n * 8 + blockIdx.x % 8) * kFewPerGroup;
  }
  j += (int)(threadIdx.x >> 5);
  if (j >= m) return;
  const float s = half_wave_cosine(a + (size_t)i * d, b + (size_t)j * d, d, threadIdx.x & 31);
  if (threadIdx.x & 31) return;
  if (S) {
    S[(size_t)i * m + j] = s;
    if (SAME) S[(size_t)j * m + i] = s;
  }
  if (SAME && key && i < j && s > T) atomicMin(key, pair_offer(s, i, j));
}

// Many pairs: one workgroup per 16 x 16 tile of them on the fp32 matrix instruction, 512 channels of the 32 rows at a time through LDS (two
// buffers; the next group on its way in registers): a lane that reads its own row from memory costs the L1 a tag look-up per 16 bytes, and
// the 16 lanes next to each other in an operand are 16 rows (1.7 us per 512 channels of a workgroup that way; 0.95 us now: copying into
// LDS, reading from it and 32 matrix instructions a SIMD, one after the other between two barriers).  One tile per compute unit at a
// time: 12.5 us at d = 4096 up to 256 tiles; heisd_skip_offline, 300 points: 21.4 -> 17.7 us (one wavefront per pair 98.8 us).  Wave 2 w + e takes the elements y = 2 e, 2 e + 1 of group w: lane (lr, g) =
// (l % 16, l / 16) reads them of row lr of either side, element (y, x) goes to accumulator (y, x), and the squared lengths come from the
// same reads.
constexpr int kPairTile = 16, kPairWaves = 16, kPairStep = 512, kPairRow = kPairStep + 4;   // floats; rows 16 bytes apart in the banks
// Rows up to this long are read straight from memory: once, by 12 waves at most, which costs less than the way through
// LDS (128 to 250 points of 256 values: 5.5 -> 4.5 us; of 512 values both ways 5.2).
constexpr int kPairDirect = 384;
template <bool SAME>
__global__ __launch_bounds__(kPairWaves * 64) __attribute__((amdgpu_waves_per_eu(4, 4))) void pair_similarity(const float *a, const float *b, int n, int m, int d, float *S,
                                                                   float T, unsigned long long *key) {
  __shared__ __attribute__((aligned(16))) float stage[2 * 32 * kPairRow];
  __shared__ double len[2][kPairWaves][kPairTile];
  __shared__ unsigned long long least;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, lr = lane & 15, lg = lane >> 4;
  int ti = blockIdx.y, tj = blockIdx.x;
  if (SAME) {                                                  // blockIdx.x counts the tiles on and above the diagonal, row by row
    const int nt = (n + kPairTile - 1) / kPairTile;
    ti = 0;
    int rest = blockIdx.x;
    // rows 0 .. ti-1 hold ti nt - ti (ti - 1) / 2 tiles
    const float h = nt + 0.5f;
    ti = max(0, min((int)(h - sqrtf(fmaxf(h * h - 2.f * rest, 0.f))), nt - 1));
    while (ti > 0 && (long long)ti * nt - (long long)ti * (ti - 1) / 2 > rest) --ti;
    while ((long long)(ti + 1) * nt - (long long)(ti + 1) * ti / 2 <= rest) ++ti;
    tj = ti + (int)(rest - ((long long)ti * nt - (long long)ti * (ti - 1) / 2));
  }
  const int i0 = ti * kPairTile, j0 = tj * kPairTile;
  // staging: 128 threads copy a row, each 16 bytes of it; rows row, row + 8 of either side
  const int row = tid >> 7, k0 = (tid & 127) * 4;
  const float *src[4];
#pragma unroll
  for (int p = 0; p < 4; ++p) {
    const int r = row + (p & 1) * 8;
    src[p] = p < 2 ? a + (size_t)min(i0 + r, n - 1) * d : b + (size_t)min(j0 + r, m - 1) * d;
  }
  f32x4 st[4];
  auto load = [&](int c) __attribute__((always_inline)) {
#pragma unroll
    for (int p = 0; p < 4; ++p) st[p] = *reinterpret_cast<const f32x4 *>(src[p] + min(c + k0, d - 4));   // d is a multiple of 4
  };
  auto store = [&](int c, int buf) __attribute__((always_inline)) {
#pragma unroll
    for (int p = 0; p < 4; ++p) {
      f32x4 x = st[p];
      if (c + k0 >= d) x = f32x4{0.f, 0.f, 0.f, 0.f};          // past the rows' end
      *reinterpret_cast<f32x4 *>(stage + (size_t)(buf * 32 + row + p * 8) * kPairRow + k0) = x;
    }
  };
  f32x4 acc[2][4], qa[2], qb[2];                               // [y][x], [y][x of the vector]
#pragma unroll
  for (int y = 0; y < 2; ++y) {
    qa[y] = qb[y] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int x = 0; x < 4; ++x) acc[y][x] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  const int mine = (wave >> 1) * 64 + lg * 16 + (wave & 1) * 8;  // this lane's channels of a group of 512
  f32x4 u[2], v[2];
  auto multiply = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int y = 0; y < 2; ++y)
#pragma unroll
      for (int x = 0; x < 4; ++x) {
        acc[y][x] = __builtin_amdgcn_mfma_f32_16x16x4f32(u[y][x], v[y][x], acc[y][x], 0, 0, 0);
        qa[y][x] = fmaf(u[y][x], u[y][x], qa[y][x]);
        qb[y][x] = fmaf(v[y][x], v[y][x], qb[y][x]);
      }
  };
  if (d <= kPairDirect) {
    const float *ra = a + (size_t)min(i0 + lr, n - 1) * d, *rb = b + (size_t)min(j0 + lr, m - 1) * d;
#pragma unroll
    for (int y = 0; y < 2; ++y) {
      const int k = mine + 4 * y;
      u[y] = v[y] = f32x4{0.f, 0.f, 0.f, 0.f};
      if (k < d) {
        u[y] = *reinterpret_cast<const f32x4 *>(ra + k);
        v[y] = *reinterpret_cast<const f32x4 *>(rb + k);
      }
    }
    multiply();
  } else {
    load(0);
    store(0, 0);
    if (kPairStep < d) load(kPairStep);
    lds_barrier();
    int buf = 0;
    for (int c = 0; c < d; c += kPairStep, buf ^= 1) {
      const float *ra = stage + (size_t)(buf * 32 + lr) * kPairRow + mine, *rb = ra + 16 * kPairRow;
#pragma unroll
      for (int y = 0; y < 2; ++y) {
        u[y] = *reinterpret_cast<const f32x4 *>(ra + 4 * y);
        v[y] = *reinterpret_cast<const f32x4 *>(rb + 4 * y);
      }
      multiply();
      if (c + kPairStep < d) store(c + kPairStep, buf ^ 1);    // read last before the barrier behind us
      if (c + 2 * kPairStep < d) load(c + 2 * kPairStep);
      lds_barrier();
    }
  }
  double *part = reinterpret_cast<double *>(stage);            // [wave][element i][lane]; nobody reads the rows any more
#pragma unroll
  for (int i = 0; i < 4; ++i)
    part[(wave * 4 + i) * 64 + lane] = sum4_tree(acc[0][0][i], acc[0][1][i], acc[0][2][i], acc[0][3][i]) +
                                       sum4_tree(acc[1][0][i], acc[1][1][i], acc[1][2][i], acc[1][3][i]);
  double la[2], lb[2];
#pragma unroll
  for (int y = 0; y < 2; ++y) {
    la[y] = sum4_tree(qa[y][0], qa[y][1], qa[y][2], qa[y][3]);
    lb[y] = sum4_tree(qb[y][0], qb[y][1], qb[y][2], qb[y][3]);
#pragma unroll
    for (int o = 16; o < 64; o <<= 1) {                        // g
      la[y] += __shfl_xor(la[y], o, kWave);
      lb[y] += __shfl_xor(lb[y], o, kWave);
    }
  }
  if (lg == 0) {
    len[0][wave][lr] = la[0] + la[1];
    len[1][wave][lr] = lb[0] + lb[1];
  }
  if (tid == 0) least = ~0ull;
  __syncthreads();
  // thread (row, column) of the tile; accumulator element i of lane l is row 4 (l / 16) + i, column l % 16
  if (tid < kPairTile * kPairTile) {
    const int r = tid >> 4, col = tid & 15, i = i0 + r, j = j0 + col;
    double s3[3][kPairWaves];
#pragma unroll
    for (int w = 0; w < kPairWaves; ++w) {
      s3[0][w] = part[(w * 4 + (r & 3)) * 64 + (r >> 2) * 16 + col];
      s3[1][w] = len[0][w][r];
      s3[2][w] = len[1][w][col];
    }
#pragma unroll
    for (int e = 0; e < 3; ++e)
#pragma unroll
      for (int o = 1; o < kPairWaves; o <<= 1)                 // y, then w: neighbours, then pairs of neighbours, ..
#pragma unroll
        for (int w = 0; w < kPairWaves; w += 2 * o) s3[e][w] += s3[e][w + o];
    if (i < n && j < m) {
      const float s = pair_cosine(s3[0][0], s3[1][0], s3[2][0]);
      if (S) {
        S[(size_t)i * m + j] = s;
        if (SAME && ti != tj) S[(size_t)j * m + i] = s;
      }
      if (SAME && key && i < j && s > T) atomicMin(&least, pair_offer(s, i, j));
    }
  }
  if (!SAME || !key) return;
  __syncthreads();
  if (tid == 0 && least != ~0ull) atomicMin(key, least);       // one offer per tile
}

__global__ void skip_key_decode(const unsigned long long *key, float *min_s, int32_t *o_dist) {
  const unsigned long long k = *key;
  if (k == ~0ull) {
    *min_s = INFINITY;          // nothing above the boundary: never skip
    *o_dist = 0;
  } else {
    *min_s = from_ordered_bits((uint32_t)(k >> 32));
    *o_dist = (int32_t)(k & 0xFFFFull);
  }
}

// skip[b] = dist[b] <= O_dist and cosine(feat_prev[b], feat_last[b]) >= min_S.  32 lanes per episode.
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(2, 2))) void skip_decide(const float *feat_prev, const float *feat_last, const int32_t *dist, int batch,
                                                  int d, const float *min_s, const int32_t *o_dist, uint8_t *skip,
                                                  float *S_out) {
  const int b = blockIdx.x * 2 + (int)(threadIdx.x >> 5);
  if (b >= batch) return;
  const float s = half_wave_cosine(feat_prev + (size_t)b * d, feat_last + (size_t)b * d, d, threadIdx.x & 31);
  if (threadIdx.x & 31) return;
  if (S_out) S_out[b] = s;
  skip[b] = (dist[b] <= *o_dist && s >= *min_s) ? 1 : 0;
}

}  // namespace heisd
