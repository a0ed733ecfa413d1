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

// Cosine similarity of two d-vectors by one wavefront; 0 if either is all zero.
__device__ __forceinline__ float wave_cosine(const float *a, const float *b, int d, int lane) {
  float ab = 0.f, aa = 0.f, bb = 0.f;
  for (int c = lane * 4; c < d; c += kWave * 4) {
    const float4 u = *reinterpret_cast<const float4 *>(a + c);
    const float4 v = *reinterpret_cast<const float4 *>(b + c);
    ab += u.x * v.x + u.y * v.y + u.z * v.z + u.w * v.w;
    aa += u.x * u.x + u.y * u.y + u.z * u.z + u.w * u.w;
    bb += v.x * v.x + v.y * v.y + v.z * v.z + v.w * v.w;
  }
  ab = wave_sum(ab);
  aa = wave_sum(aa);
  bb = wave_sum(bb);
  return (aa == 0.f || bb == 0.f) ? 0.f : ab / (sqrtf(aa) * sqrtf(bb));
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

// S[i][j] = cosine(a[i], b[j]), one workgroup per 16 x 16 tile of pairs on the fp32 matrix instruction
// v_mfma_f32_16x16x4_f32 (fp32 products and sums).  The 16 waves take every sixteenth group of 32 channels; a lane
// loads 2 x 16 bytes of one row of each side and feeds component x of half h of both to accumulator (h, x): eight short sums per
// wave (error against 64 bits no larger than that of one wavefront's dot product), added up in a fixed order.  The rows' squared lengths
// come from the same loads.  Bound: each tile reads 32 rows from the L2 (512 KB at d = 4096, at 64 bytes a clock 3.9 us);
// one wavefront per pair read both rows for every pair: 300 x 300 x 4096 311 us, 22 us now (error against
// 64 bits 6.8e-8, 5.7e-8 now).
// SAME (a and b are the same points): only tiles on and above the diagonal are computed, a tile above it is stored twice
// (a product and its mirror image are the same bits).
// With `key` given (offline stage of Alg. 1; SAME): every pair i < j whose similarity exceeds T offers
// (similarity, i, j - i) to a 64-bit minimum, so that the smallest similarity above T wins and, among
// equals, the pair found first by the algorithm's loops (i ascending, then distance ascending).
constexpr int kPairTile = 16, kPairWaves = 16;
template <bool SAME>
__global__ __launch_bounds__(kPairWaves * 64) __attribute__((amdgpu_waves_per_eu(4, 4))) void pair_similarity(const float *a, const float *b, int n, int m, int d, float *S,
                                                                   float T, unsigned long long *key) {
  __shared__ f32x4 part[kPairWaves][64];
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
  const float *pa = a + (size_t)min(i0 + lr, n - 1) * d, *pb = b + (size_t)min(j0 + lr, m - 1) * d;
  const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
  f32x4 acc[2][4];
  double aa = 0., bb = 0.;                                     // in 64 bits: the diagonal's 1 rests on them
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int x = 0; x < 4; ++x) acc[h][x] = zero;
  // 32 channels (one 128-byte line of each row) at a time: lane (lr, lg) loads channels c + 4 lg .. + 3 and c + 16 + 4 lg .. + 3;
  // d is a multiple of 4
  for (int c = wave * 32; c < d; c += kPairWaves * 32) {         // (three groups requested together: no faster)
    f32x4 u[2], v[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int k = min(c + h * 16 + lg * 4, d - 4);
      u[h] = *reinterpret_cast<const f32x4 *>(pa + k);
      v[h] = *reinterpret_cast<const f32x4 *>(pb + k);
    }
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const bool in = c + h * 16 + lg * 4 < d;
#pragma unroll
      for (int x = 0; x < 4; ++x) {
        const float a1 = in ? u[h][x] : 0.f, b1 = in ? v[h][x] : 0.f;
        acc[h][x] = __builtin_amdgcn_mfma_f32_16x16x4f32(a1, b1, acc[h][x], 0, 0, 0);
        aa = fma((double)a1, (double)a1, aa);
        bb = fma((double)b1, (double)b1, bb);
      }
    }
  }
  part[wave][lane] = ((acc[0][0] + acc[0][1]) + (acc[0][2] + acc[0][3])) + ((acc[1][0] + acc[1][1]) + (acc[1][2] + acc[1][3]));
  aa += __shfl_xor(aa, 16, kWave);
  aa += __shfl_xor(aa, 32, kWave);
  bb += __shfl_xor(bb, 16, kWave);
  bb += __shfl_xor(bb, 32, kWave);
  if (lg == 0) {
    len[0][wave][lr] = aa;
    len[1][wave][lr] = bb;
  }
  if (tid == 0) least = ~0ull;
  __syncthreads();
  // thread (row, column) of the tile; accumulator element i of lane l is row 4 (l / 16) + i, column l % 16
  if (tid < kPairTile * kPairTile) {
    const int r = tid >> 4, col = tid & 15, i = i0 + r, j = j0 + col;
    double dot = 0., la = 0., lb = 0.;
#pragma unroll
    for (int w = 0; w < kPairWaves; ++w) {
      const int l = (r >> 2) * 16 + col;
      dot += part[w][l][r & 3];
      la += len[0][w][r];
      lb += len[1][w][col];
    }
    if (i < n && j < m) {
      const float fa = (float)la, fb = (float)lb;
      const float s = (fa == 0.f || fb == 0.f) ? 0.f : (float)dot / (sqrtf(fa) * sqrtf(fb));
      if (S) {
        S[(size_t)i * m + j] = s;
        if (SAME && ti != tj) S[(size_t)j * m + i] = s;
      }
      if (SAME && key && i < j && s > T)
        atomicMin(&least, ((unsigned long long)ordered_bits(s) << 32) | ((unsigned long long)i << 16) | (unsigned long long)(j - i));
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

// skip[b] = dist[b] <= O_dist and cosine(feat_prev[b], feat_last[b]) >= min_S.  One wavefront per episode.
__global__ __launch_bounds__(64) void skip_decide(const float *feat_prev, const float *feat_last, const int32_t *dist,
                                                  int d, const float *min_s, const int32_t *o_dist, uint8_t *skip,
                                                  float *S_out) {
  const int b = blockIdx.x, lane = threadIdx.x;
  const float s = wave_cosine(feat_prev + (size_t)b * d, feat_last + (size_t)b * d, d, lane);
  if (lane != 0) return;
  if (S_out) S_out[b] = s;
  skip[b] = (dist[b] <= *o_dist && s >= *min_s) ? 1 : 0;
}

}  // namespace heisd
