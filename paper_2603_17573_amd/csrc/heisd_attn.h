// Verify attention with fused RoPE and KV-append (paper Sec. 2.2: the target scores all K
// drafts in one pass; App. A.2: causal attention over visual, text and earlier action
// tokens).  One workgroup per (episode, head).
//
//   1. rotate this head's new keys (rotate-half, absolute position prefix_len + j), round
//      keys and values to bf16 and append them to the episode's cache rows; the rotated keys
//      are also kept in fp32 (in LDS, or in place in the projection scratch) so that the block attends
//      to its own rows at full precision and only the prefix is read as bf16;
//   2. per block of 8 queries: scores, softmax and weighted values on the matrix cores, every wave over its own tiles
//      of cached keys, the waves' results added at the end (attn_verify).
// Skipped episodes (verify-skip, Sec. 4.1) touch neither the cache nor the scores.
//
// Tree verification (Sec. 4.2: chains of a sequence-wise draft tree are checked in one pass):
// with `depth` and `anc` given, new row j sits at position prefix_len + depth[j] and sees, among
// the new rows, exactly those whose bit is set in its 256-bit ancestor mask (itself included).
// Its key and value still go to cache row prefix_len + j.
#pragma once
#include "heisd_common.h"

namespace heisd {

constexpr int kAttnQB = 8;  // queries per block

struct AttnArgs {
  float *qkv;                // [M][3*d] fp32: q | k | v of the new rows, not yet rotated; k is rotated in place
  uint16_t *k_cache;         // this layer: bf16 [batch][H][cap][HD]
  uint16_t *v_cache;
  const int32_t *prefix_len; // [batch]
  const uint8_t *skip;       // [batch] or nullptr
  const float2 *rope;        // [cap][HD/2] (cos, sin) of position * theta_i
  float *out;                // [M][d] fp32 rows, or nullptr
  uint16_t *o_planes;        // or: records [d/16][CTS][16][16] bf16 (head rows 0-7, tail rows 8-15 of each
  int CTS;                   //     column tile of 8 activation rows), the B-operand format of the GEMMs
  int single;                // records hold ONE bf16 per value: 16 activation rows per column tile (see BatGemm::single)
  int K, H, cap, d;
  float scale;               // 1/sqrt(HD)
  const int32_t *depth;              // tree mode: [batch][K] tokens between the prefix and row j; else nullptr
  const unsigned long long *anc;     // tree mode: [batch][K][4] visibility bits over the K new rows
};

// LDS of attn_verify: queries, the block's own rows or (split) room for the scores of K new rows, the waves' results.
inline size_t attn_lds_bytes(int hd, int K, int waves, bool split) {
  const size_t floats = (size_t)kAttnQB * hd + (split ? 0 : (size_t)2 * kAttnQB * hd) + (size_t)kAttnQB * (split ? K : kAttnQB) +
                        (size_t)waves * 2 * kAttnQB;
  return (floats * sizeof(float) + 15) / 16 * 16 + (size_t)waves * kAttnQB * hd * sizeof(float);
}

// Attention output element (row m, column col).
__device__ __forceinline__ void attn_store(const AttnArgs &a, int m, int col, float v) {
  if (a.out) a.out[(size_t)m * a.d + col] = v;
  if (a.o_planes) {
    uint32_t hi, lo;
    split_bf16(v, hi, lo);
    if (a.single) {
      a.o_planes[((size_t)(col >> 4) * a.CTS + (m >> 4)) * 256 + (m & 15) * 16 + (col & 15)] = (uint16_t)hi;
      return;
    }
    uint16_t *rec = a.o_planes + ((size_t)(col >> 4) * a.CTS + (m >> 3)) * 256 + (m & 7) * 16 + (col & 15);
    rec[0] = (uint16_t)hi;
    rec[128] = (uint16_t)lo;
  }
}

// Two neighbouring elements (col even): one 4-byte store per half of the record.
__device__ __forceinline__ void attn_store2(const AttnArgs &a, int m, int col, float v0, float v1) {
  if (a.out) *reinterpret_cast<float2 *>(a.out + (size_t)m * a.d + col) = make_float2(v0, v1);
  if (a.o_planes) {
    uint32_t h0, l0, h1, l1;
    split_bf16(v0, h0, l0);
    split_bf16(v1, h1, l1);
    if (a.single) {
      *reinterpret_cast<uint32_t *>(a.o_planes + ((size_t)(col >> 4) * a.CTS + (m >> 4)) * 256 + (m & 15) * 16 + (col & 15)) = h0 | (h1 << 16);
      return;
    }
    uint32_t *rec = reinterpret_cast<uint32_t *>(a.o_planes + ((size_t)(col >> 4) * a.CTS + (m >> 3)) * 256 + (m & 7) * 16 + (col & 15));
    rec[0] = h0 | (h1 << 16);
    rec[64] = l0 | (l1 << 16);
  }
}

// RoPE on the new keys of (episode b, head h), in place in fp32, and the append of keys and values
// (bf16) to the episode's cache rows P .. P+K-1.
template <int HD, bool TREE>
__device__ __forceinline__ void attn_append_rows(const AttnArgs &a, int b, int h, int P, int tid, int nthreads,
                                                 int jb, int je) {
  constexpr int HALF = HD / 2;
  const int K = a.K, d = a.d, row0 = b * K;
  uint16_t *kc = a.k_cache + ((size_t)(b * a.H + h) * a.cap) * HD;
  uint16_t *vc = a.v_cache + ((size_t)(b * a.H + h) * a.cap) * HD;
  for (int idx = tid + jb * HALF; idx < je * HALF; idx += nthreads) {
    const int j = idx / HALF, i = idx - j * HALF;
    float *src = a.qkv + (size_t)(row0 + j) * 3 * d + h * HD;
    const float2 cs = a.rope[(size_t)(P + (TREE ? a.depth[row0 + j] : j)) * HALF + i];
    const float k1 = src[d + i], k2 = src[d + i + HALF];
    const float kr1 = k1 * cs.x - k2 * cs.y, kr2 = k2 * cs.x + k1 * cs.y;
    src[d + i] = kr1;
    src[d + i + HALF] = kr2;
    uint16_t *kr = kc + (size_t)(P + j) * HD;
    kr[i] = (uint16_t)f32_to_bf16_bits(kr1);
    kr[i + HALF] = (uint16_t)f32_to_bf16_bits(kr2);
    uint16_t *vr = vc + (size_t)(P + j) * HD;
    vr[i] = (uint16_t)f32_to_bf16_bits(src[2 * d + i]);
    vr[i + HALF] = (uint16_t)f32_to_bf16_bits(src[2 * d + i + HALF]);
  }
}

// The append alone, one workgroup per (head, episode, 8 new rows): first half of a step whose attention
// runs with one workgroup per block of 8 queries (attn_verify with SPLIT).
template <int HD, bool TREE>
__global__ __launch_bounds__(256) void attn_append(AttnArgs a) {
  const int h = blockIdx.x, b = blockIdx.y;
  if (episode_sits_out(a.skip, a.prefix_len, b, a.K, a.cap)) return;
  int P = a.prefix_len[b];
  P = max(0, min(P, a.cap - a.K));
  const int jb = (int)blockIdx.z * kAttnQB;
  attn_append_rows<HD, TREE>(a, b, h, P, threadIdx.x, 256, jb, min(a.K, jb + kAttnQB));
}

// Attention of one block of at most 8 queries of one (head, episode); blockIdx.z names the block.  Every wave takes every
// W-th tile of 32 cached keys (and every W-th new row) from scores to weighted values by itself, with a running maximum; the
// waves meet once at the end.
//   scores   S^T = K q^T on v_mfma_f32_16x16x32_bf16: 16 keys are the A operand straight from the cache (lane l: key l % 16, 8 consecutive
//            channels), the 8 queries the B operand, each fp32 query as a bf16 head (columns 0-7) and a bf16 tail (columns
//            8-15); one lane rotation adds the two, so that lane (lr, lg) = (l % 16, l / 16) holds the scores of keys 4 lg .. + 3 of
//            both 16-key halves against query lr % 8.
//   weights  p = exp(s - m) in fp32, cut into three bf16 parts that add up to it exactly: lanes lr < 8 keep the first, lanes lr >= 8 the
//            second - which IS the A operand of the value product (rows 0-7 and 8-15, k = the lane's 8 keys), without any
//            exchange -, and a second product adds the third.
//   values   O = p V: lane (lr, lg) loads its 8 keys' channels HD/16 lr .. (whole cache rows per 16 lanes) and turns the 8 x HD/16 block
//            around in registers (v_perm); the j-th product's column lr is channel HD/16 lr + j.
// The block's own new rows stay fp32 on both sides (scores and values by FMAs).
// What it is bound by: with few episodes the chain of dependent steps (round trips for the lengths, the rows, the cache), with
// many the reading of the cache.  The version before had scores, softmax and values in three passes with a barrier
// between them, the values by FMAs and 128 lane exchanges at the end.  us per layer at 32 heads of 128, before and
// now: 8 episodes x 7 rows 21.5 / 14.2, 64 x 7 88 / 67.6 (326 MB of cache: 4.8 TB/s), 16 x 14 (prefix up to 532) 51 / 34 with the append,
// 76-token tree 33 / 16.7, prefill of 276 rows 52 / 33.
// Every workgroup appends its own queries' keys and values to the cache.  SPLIT = false: the episode has a single block, whose new rows
// the waves read from LDS; SPLIT = true: several blocks per episode, and a block rotates the earlier blocks' keys as it
// reads them (a launch for that, attn_append, was 5-6 us per layer).  The last blocks see most of the new rows and
// start first, not by themselves at the end (whole calls: prefill of 276 rows 1197 -> 1191 us, of 400 rows with 8 heads 275 -> 270, 76-token tree 691 -> 686).
// TREE: tree mode compiled in (the linear kernel carries none of its registers).
template <int HD, int W, bool TREE, bool SPLIT>
__global__ __launch_bounds__(W * 64) __attribute__((amdgpu_waves_per_eu(W == 8 ? 2 : 3, W == 8 ? 2 : 3))) void attn_verify(AttnArgs a) {
  constexpr int THREADS = W * 64, HALF = HD / 2, KS = HD / 32, CPL = HD / 16, QB = kAttnQB;
  typedef unsigned int au32x4 __attribute__((ext_vector_type(4)));
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  float *qs = reinterpret_cast<float *>(smem);             // [QB][HD] rotated, scaled queries
  float *own = qs + QB * HD;                               // !SPLIT: [2][QB][HD] the block's new keys (rotated) and values
  float *so = own + (SPLIT ? 0 : 2 * QB * HD);             // [QB][own_ld] scores, then weights, of the new rows
  const int own_ld = SPLIT ? a.K : QB;
  float *ml = so + QB * own_ld;                            // [W][2][QB] the waves' maxima and sums
  float *om = reinterpret_cast<float *>(smem + ((size_t)(reinterpret_cast<unsigned char *>(ml + W * 2 * QB) - smem) + 15) / 16 * 16);   // [W][QB][HD]

  const int h = blockIdx.x, b = blockIdx.y;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lr = lane & 15, lg = lane >> 4;
  const int K = a.K, d = a.d, cap = a.cap;
  const int row0 = b * K, j0 = SPLIT ? (int)(gridDim.z - 1 - blockIdx.z) * QB : 0, nq = min(QB, K - j0);   // this workgroup's queries
  if (episode_sits_out(a.skip, a.prefix_len, b, K, cap)) {
    for (int idx = tid; idx < nq * HD; idx += THREADS) attn_store(a, row0 + j0 + idx / HD, h * HD + (idx % HD), 0.f);
    return;
  }
  int P = a.prefix_len[b];
  P = max(0, min(P, cap - K));  // never index past the cache, whatever the caller passed
  uint16_t *kc = a.k_cache + ((size_t)(b * a.H + h) * cap) * HD;
  uint16_t *vc = a.v_cache + ((size_t)(b * a.H + h) * cap) * HD;

  const int n_tiles = (P + 31) / 32;
  au32x4 kf[2][KS];
  uint2 vf[8][CPL / 4];
  auto load_k = [&](int t) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const uint16_t *kr = kc + (size_t)min(t * 32 + u * 16 + lr, max(P - 1, 0)) * HD + lg * 8;      // rows past the prefix repeat its last row
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) kf[u][ks] = *reinterpret_cast<const au32x4 *>(kr + ks * 32);
    }
  };
  auto load_v = [&](int t) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int r = t * 32 + (i >> 2) * 16 + lg * 4 + (i & 3);
      const uint16_t *vr = vc + (size_t)min(r, max(P - 1, 0)) * HD + lr * CPL;
      if constexpr (CPL == 8) {
        const uint4 v = *reinterpret_cast<const uint4 *>(vr);
        vf[i][0] = make_uint2(v.x, v.y);
        vf[i][1] = make_uint2(v.z, v.w);
      } else {
        vf[i][0] = *reinterpret_cast<const uint2 *>(vr);
      }
    }
  };
  // The block's queries (rotated, scaled), new keys (rotated) and values; the last two are appended to the cache.  Requested before the
  // first tile's cache rows (loads return in order), rotated while those are on their way.
  constexpr int NI = (QB * HALF + THREADS - 1) / THREADS;
  float2 cs[NI], qx[NI], kx[NI], vx[NI];
#pragma unroll
  for (int n = 0; n < NI; ++n) {
    const int idx = tid + n * THREADS, j = idx / HALF, i = idx - j * HALF, jc = min(j, nq - 1);
    const float *src = a.qkv + (size_t)(row0 + j0 + jc) * 3 * d + h * HD;
    cs[n] = a.rope[(size_t)(P + (TREE ? a.depth[row0 + j0 + jc] : j0 + jc)) * HALF + i];
    qx[n] = make_float2(src[i], src[i + HALF]);
    kx[n] = make_float2(src[d + i], src[d + i + HALF]);
    vx[n] = make_float2(src[2 * d + i], src[2 * d + i + HALF]);
  }
  __builtin_amdgcn_sched_barrier(0);
  load_k(wave);
  if (!SPLIT) load_v(wave);
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int n = 0; n < NI; ++n) {
    const int idx = tid + n * THREADS, j = idx / HALF, i = idx - j * HALF;
    if (j >= QB) break;
    const bool in = j < nq;
    qs[j * HD + i] = in ? (qx[n].x * cs[n].x - qx[n].y * cs[n].y) * a.scale : 0.f;
    qs[j * HD + i + HALF] = in ? (qx[n].y * cs[n].x + qx[n].x * cs[n].y) * a.scale : 0.f;
    if (in) {
      const float kr1 = kx[n].x * cs[n].x - kx[n].y * cs[n].y, kr2 = kx[n].y * cs[n].x + kx[n].x * cs[n].y;
      if (!SPLIT) {
        own[j * HD + i] = kr1;
        own[j * HD + i + HALF] = kr2;
        own[(QB + j) * HD + i] = vx[n].x;
        own[(QB + j) * HD + i + HALF] = vx[n].y;
      }
      uint16_t *kr = kc + (size_t)(P + j0 + j) * HD, *vr = vc + (size_t)(P + j0 + j) * HD;
      kr[i] = (uint16_t)f32_to_bf16_bits(kr1);
      kr[i + HALF] = (uint16_t)f32_to_bf16_bits(kr2);
      vr[i] = (uint16_t)f32_to_bf16_bits(vx[n].x);
      vr[i + HALF] = (uint16_t)f32_to_bf16_bits(vx[n].y);
    }
  }
  lds_barrier();

  // ---- scores of the new rows j = wave, wave + W, .. against all queries, kept in LDS (read back by this wave only) ----
  const int n_own = j0 + nq;                               // new rows the block's last query sees
  float m;                                                 // lane (lr, lg): the largest so far of query lr % 8
  if constexpr (!SPLIT) {                                  // from LDS: lane (q, part) = (lane / 8, lane % 8) sums HD / 8 channels
    const int q = lane >> 3, oc = (lane & 7) * (HD / 8);
    float best = -INFINITY;
    unsigned long long seen = 0ull;                        // at most 8 new rows
    if (TREE && q < nq) seen = a.anc[(size_t)(row0 + j0 + q) * 4];
    for (int j = wave; j < n_own; j += W) {
      float t = 0.f;
#pragma unroll
      for (int i = 0; i < HD / 32; ++i) {
        const float4 k4 = *reinterpret_cast<const float4 *>(own + j * HD + oc + 4 * i);
        const float4 q4 = *reinterpret_cast<const float4 *>(qs + q * HD + oc + 4 * i);
        t = fmaf(q4.x, k4.x, fmaf(q4.y, k4.y, fmaf(q4.z, k4.z, fmaf(q4.w, k4.w, t))));
      }
      t = sum8(t);
      t = (TREE ? ((seen >> j) & 1ull) != 0 : j <= j0 + q) ? t : -INFINITY;
      best = fmaxf(best, t);
      if ((lane & 7) == 0) so[q * own_ld + j] = t;
    }
    m = __shfl(best, (lr & 7) * 8, kWave);
  } else {
    // From memory: four rows at a time, lane (row, part) = (lg, lr) multiplies HD / 16 channels with all 8 queries; the 8 sums
    // over 16 lanes are halved three times on the way (a lane keeps the queries of its own bits 3, 2, 1), 8 values in 25 instructions.
    float qv[QB][CPL];
#pragma unroll
    for (int q = 0; q < QB; ++q)
#pragma unroll
      for (int c = 0; c < CPL; c += 4) {
        const float4 x = *reinterpret_cast<const float4 *>(qs + q * HD + lr * CPL + c);
        qv[q][c] = x.x; qv[q][c + 1] = x.y; qv[q][c + 2] = x.z; qv[q][c + 3] = x.w;
      }
    const int q = lr >> 1;                                 // the query this lane ends up with
    const bool b3 = lr & 8, b2 = lr & 4, b1 = lr & 2;
    unsigned long long seen[4] = {0ull, 0ull, 0ull, 0ull};
    if (TREE && q < nq)
#pragma unroll
      for (int w = 0; w < 4; ++w) seen[w] = a.anc[(size_t)(row0 + j0 + q) * 4 + w];
    float best = -INFINITY;
    constexpr int UB = 1;                                  // groups of four rows requested together (two: too many registers)
    for (int jb = wave; jb < n_own; jb += 4 * UB * W) {
      // The projection's rows are not rotated (each block rotates what it reads: no launch of its own for that): channel i
      // and channel i + HD / 2 are 8 lanes apart.
      float k[UB][CPL];
      float2 rt[UB][CPL];
#pragma unroll
      for (int u = 0; u < UB; ++u) {
        const int j = min(jb + (4 * u + lg) * W, n_own - 1);
        const float *kr = a.qkv + (size_t)(row0 + j) * 3 * d + d + h * HD + lr * CPL;
        const float2 *ro = a.rope + (size_t)(P + (TREE ? a.depth[row0 + j] : j)) * HALF + (lr & 7) * CPL;
#pragma unroll
        for (int c = 0; c < CPL; c += 4) {
          const float4 x = *reinterpret_cast<const float4 *>(kr + c);
          k[u][c] = x.x; k[u][c + 1] = x.y; k[u][c + 2] = x.z; k[u][c + 3] = x.w;
        }
#pragma unroll
        for (int c = 0; c < CPL; c += 2) {
          const float4 x = *reinterpret_cast<const float4 *>(ro + c);
          rt[u][c] = make_float2(x.x, x.y);
          rt[u][c + 1] = make_float2(x.z, x.w);
        }
      }
#pragma unroll
      for (int u = 0; u < UB; ++u)
#pragma unroll
        for (int c = 0; c < CPL; ++c) {
          const float other = dpp_move<0x128>(k[u][c]);
          k[u][c] = k[u][c] * rt[u][c].x + (lr < 8 ? -other : other) * rt[u][c].y;
        }
#pragma unroll
      for (int u = 0; u < UB; ++u) {
        const int j = jb + (4 * u + lg) * W;
        float s8[QB], s4[4], s2[2];
#pragma unroll
        for (int x = 0; x < QB; ++x) {
          s8[x] = 0.f;
#pragma unroll
          for (int c = 0; c < CPL; ++c) s8[x] = fmaf(qv[x][c], k[u][c], s8[x]);
        }
#pragma unroll
        for (int x = 0; x < 4; ++x) s4[x] = (b3 ? s8[x + 4] : s8[x]) + dpp_move<0x128>(b3 ? s8[x] : s8[x + 4]);
#pragma unroll
        for (int x = 0; x < 2; ++x) s2[x] = (b2 ? s4[x + 2] : s4[x]) + dpp_move<kDppHalfMirror>(b2 ? s4[x] : s4[x + 2]);
        float t = (b1 ? s2[1] : s2[0]) + dpp_move<kDppXor2>(b1 ? s2[0] : s2[1]);
        t += dpp_move<kDppXor1>(t);
        bool sees = j <= j0 + q;
        if (TREE) {
          const unsigned long long w = j < 128 ? (j < 64 ? seen[0] : seen[1]) : (j < 192 ? seen[2] : seen[3]);
          sees = ((w >> (j & 63)) & 1ull) != 0;
        }
        t = sees && j < n_own ? t : -INFINITY;
        best = fmaxf(best, t);
        if (!(lr & 1) && j < n_own) so[q * own_ld + j] = t;
      }
    }
    best = max_xor32(max_xor16(best));
    m = __shfl(best, (lr & 7) * 2, kWave);
  }

  // the queries as the B operand of the scores
  au32x4 qb[KS];
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) {
    const float4 x0 = *reinterpret_cast<const float4 *>(qs + (lr & 7) * HD + ks * 32 + lg * 8);
    const float4 x1 = *reinterpret_cast<const float4 *>(qs + (lr & 7) * HD + ks * 32 + lg * 8 + 4);
    const float x[8] = {x0.x, x0.y, x0.z, x0.w, x1.x, x1.y, x1.z, x1.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      uint32_t h0, l0, h1, l1;
      split_bf16(x[2 * i], h0, l0);
      split_bf16(x[2 * i + 1], h1, l1);
      qb[ks][i] = lr < 8 ? (h0 | (h1 << 16)) : (l0 | (l1 << 16));
    }
  }

  if (SPLIT) load_v(wave);                                 // (before the new rows' scores they are 32 registers too many: scratch in the loop)

  // lane (lr, lg): running maximum m and sum l (this lane's keys only) of query lr % 8; accumulator j: rows 4 lg + i (query, or query + 8: the
  // second part's product), channel CPL lr + j
  float l = 0.f;
  f32x4 acc[CPL];
#pragma unroll
  for (int j = 0; j < CPL; ++j) acc[j] = f32x4{0.f, 0.f, 0.f, 0.f};
  for (int t = wave; t < n_tiles; t += W) {
    float s[8];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      f32x4 c = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int ks = 0; ks < KS; ++ks)
        c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, kf[u][ks]), __builtin_bit_cast(bf16x8, qb[ks]), c, 0, 0, 0);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float v = c[i] + dpp_move<0x128>(c[i]);      // head column + tail column (a rotation of the row of 16 lanes by 8)
        s[u * 4 + i] = t * 32 + u * 16 + lg * 4 + i < P ? v : -INFINITY;
      }
    }
    const bool more = t + W < n_tiles;                     // uniform
    if (more) load_k(t + W);
    float mx = s[0];
#pragma unroll
    for (int i = 1; i < 8; ++i) mx = fmaxf(mx, s[i]);
    mx = max_xor32(max_xor16(mx));
    const float mn = fmaxf(m, mx);                         // finite: the tile holds a key of the prefix (or a NaN score, which stays one)
    const float ref = mn == -INFINITY ? 0.f : mn;
    const float f = expf(m - ref);
    m = mn;
    l *= f;
    // the rows of this lane's accumulators belong to queries (4 lg + i) % 8
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float fi = __shfl(f, (lg * 4 + i) & 7, kWave);
#pragma unroll
      for (int j = 0; j < CPL; ++j) acc[j][i] *= fi;
    }
    au32x4 pa, pb;                                         // parts: [first | second], [third | 0]
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      uint32_t w1[2], w3[2];
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        const float p = expf(s[2 * i + e] - ref);
        l += p;
        const float r1 = p - __uint_as_float(__float_as_uint(p) & 0xFFFF0000u);
        const float r2 = r1 - __uint_as_float(__float_as_uint(r1) & 0xFFFF0000u);
        w1[e] = lr < 8 ? __float_as_uint(p) : __float_as_uint(r1);
        w3[e] = lr < 8 ? __float_as_uint(r2) : 0u;
      }
      pa[i] = __builtin_amdgcn_perm(w1[1], w1[0], 0x07060302u);
      pb[i] = __builtin_amdgcn_perm(w3[1], w3[0], 0x07060302u);
    }
    if (t * 32 + 32 > P) {                                 // uniform: rows past the prefix count for nothing, whatever they hold
#pragma unroll
      for (int i = 0; i < 8; ++i)
        if (t * 32 + (i >> 2) * 16 + lg * 4 + (i & 3) >= P)
#pragma unroll
          for (int c = 0; c < CPL / 4; ++c) vf[i][c] = make_uint2(0u, 0u);
    }
#pragma unroll
    for (int j = 0; j < CPL; ++j) {
      au32x4 vt;                                           // channel CPL lr + j of the lane's 8 keys
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const uint2 v0 = vf[2 * i][j >> 2], v1 = vf[2 * i + 1][j >> 2];
        vt[i] = __builtin_amdgcn_perm((j & 2) ? v1.y : v1.x, (j & 2) ? v0.y : v0.x, (j & 1) ? 0x07060302u : 0x05040100u);
      }
      acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, pa), __builtin_bit_cast(bf16x8, vt), acc[j], 0, 0, 0);
      acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, pb), __builtin_bit_cast(bf16x8, vt), acc[j], 0, 0, 0);
    }
    if (more) load_v(t + W);
  }
  l = sum_xor32(sum_xor16(l));

  // ---- the new rows' values, two rows at a time: lanes 0-31 (whose accumulator rows are the queries) one, lanes 32-63 (whose rows
  // are added to them at the end) the other; lane (q, r) = (lane / 8, lane % 8) makes the weight of row r of eight for query q ----
  const float m_ref = m == -INFINITY ? 0.f : m;
  const float m_row = __shfl(m_ref, lane >> 3, kWave);     // maximum of query lane / 8 (held by lane lr = query)
  float lo = 0.f;
  constexpr int PAIRS = SPLIT ? 4 : 1;                     // (without split a wave has two rows at most)
  for (int jb = wave; jb < n_own; jb += 2 * PAIRS * W) {
    float v[PAIRS][CPL];
#pragma unroll
    for (int u = 0; u < PAIRS; ++u) {
      const int j = min(jb + (2 * u + (lane >> 5)) * W, n_own - 1);
      const float *vr = (SPLIT ? a.qkv + (size_t)(row0 + j) * 3 * d + 2 * d + h * HD : own + (QB + j) * HD) + lr * CPL;
#pragma unroll
      for (int c = 0; c < CPL; c += 4) {
        const float4 x = *reinterpret_cast<const float4 *>(vr + c);
        v[u][c] = x.x; v[u][c + 1] = x.y; v[u][c + 2] = x.z; v[u][c + 3] = x.w;
      }
    }
    const int jp = jb + (lane & 7) * W;
    const bool in = (lane & 7) < 2 * PAIRS && jp < n_own;
    const float p = in ? expf(so[(lane >> 3) * own_ld + min(jp, n_own - 1)] - m_row) : 0.f;
    lo += p;
#pragma unroll
    for (int u = 0; u < PAIRS; ++u) {
      if (jb + 2 * u * W >= n_own) break;                  // uniform
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float pi = __shfl(p, ((lg * 4 + i) & 7) * 8 + 2 * u + (lane >> 5), kWave);
#pragma unroll
        for (int c = 0; c < CPL; ++c) acc[c][i] = fmaf(pi, v[u][c], acc[c][i]);
      }
    }
  }
  l += __shfl(sum8(lo), (lr & 7) * 8, kWave);
  if (lane < QB) {
    ml[(wave * 2) * QB + lane] = m;
    ml[(wave * 2 + 1) * QB + lane] = l;
  }
  // rows q and q + 8 (lanes 32 apart) are two parts of the same output
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    float o[CPL];
#pragma unroll
    for (int j = 0; j < CPL; ++j) o[j] = sum_xor32(acc[j][i]);
    if (lg < 2)
#pragma unroll
      for (int j = 0; j < CPL; j += 4)
        *reinterpret_cast<float4 *>(om + ((size_t)wave * QB + lg * 4 + i) * HD + lr * CPL + j) = make_float4(o[j], o[j + 1], o[j + 2], o[j + 3]);
  }
  lds_barrier();

  // ---- the waves' results together: thread (query, two channels) ----
  for (int idx = tid; idx < nq * HALF; idx += THREADS) {
    const int q = idx / HALF, c = (idx - q * HALF) * 2;
    float M = -INFINITY;
#pragma unroll
    for (int w = 0; w < W; ++w) M = fmaxf(M, ml[(w * 2) * QB + q]);
    if (M == -INFINITY) M = 0.f;
    float L = 0.f, o0 = 0.f, o1 = 0.f;
#pragma unroll
    for (int w = 0; w < W; ++w) {
      const float e = expf(ml[(w * 2) * QB + q] - M);
      L = fmaf(ml[(w * 2 + 1) * QB + q], e, L);
      const float2 o = *reinterpret_cast<const float2 *>(om + ((size_t)w * QB + q) * HD + c);
      o0 = fmaf(o.x, e, o0);
      o1 = fmaf(o.y, e, o1);
    }
    const float inv = 1.0f / L;
    attn_store2(a, row0 + j0 + q, h * HD + c, o0 * inv, o1 * inv);
  }
}

// ---- single-bf16 activations ------------------------------------------------------------------------
// The kernel of HEISD_ACT_BF16: prefix scores on the matrix cores, softmax, values by fp32 FMAs, in three passes over LDS.
// attn_verify above is 23 % faster at 64 episodes (88 / 67.6 us per layer) and as exact, but adds in another order, and with one
// bf16 per activation ANY change of a last bit grows through the roundings of the layers that follow to what the
// format itself costs (half a percent of the logits after four layers): 1.4 % of the greedy bins of 448 rows came out
// differently.  Callers of that format keep the results they have.
constexpr int kAttnU = 6;   // cache rows a value stream requests at once

__device__ __forceinline__ void attn_unpack8(const uint4 v, float (&f)[8]) {
  const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    f[2 * i] = __uint_as_float(w[i] << 16);
    f[2 * i + 1] = __uint_as_float(w[i] & 0xFFFF0000u);
  }
}

// waves: 4 or 8 (workgroups of 256 or 512 threads)
inline size_t attn_fma_lds_bytes(int hd, int cap, int waves) {
  return sizeof(float) * ((size_t)kAttnQB * hd + (size_t)kAttnQB * cap + kAttnQB + (size_t)waves * kAttnQB * hd) +
         kAttnQB * 4 * sizeof(unsigned long long);   // tree mode: visibility bits of the block's queries
}

// THREADS: 256 or 512.  With few (episode, head) pairs - fewer workgroups than would fill the
// compute units twice - the larger workgroup hides more latency (M = 56: 31 -> 26 us per layer);
// with many pairs the smaller one is faster (M = 448: 131 against 167 us).
// TREE: tree mode compiled in (the linear kernel carries none of its registers).
// A workgroup serves one block of at most 8 queries of one (head, episode): blockIdx.z names the block.
// SPLIT = false: the episode has a single block and the workgroup also rotates and appends the new keys
// and values; SPLIT = true: several blocks per episode, the append ran as attn_append before.  With many
// queries per episode and few episodes the blocks are what fills the chip (76 tree tokens, one episode:
// 225 us per layer with one workgroup per head, 64 us with one per block).
template <int HD, int THREADS, bool TREE, bool SPLIT>
// The 256-thread single-block variant is held to 128 registers (four waves per SIMD: 108 -> 98 us per layer
// at 64 episodes); the same limit on the per-block variant measured slower (long prefixes: 72 -> 86 us).
__global__ __launch_bounds__(THREADS) __attribute__((amdgpu_waves_per_eu((THREADS == 256 && !SPLIT) ? 4 : 2))) void attn_verify_fma(AttnArgs a) {
  constexpr int kAttnThreads = THREADS, kAttnWaves = THREADS / 64;
  constexpr int HALF = HD / 2;
  constexpr int LPK = HD / 8;              // lanes that share one key row (16 bytes each)
  constexpr int G = kAttnThreads / LPK;    // key rows in flight per pass
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  float *qs = reinterpret_cast<float *>(smem);        // [QB][HD]
  float *sc = qs + kAttnQB * HD;                       // [QB][cap]
  float *inv_l = sc + (size_t)kAttnQB * a.cap;         // [QB]
  float *ored = inv_l + kAttnQB;                       // [waves][QB][HD]
  unsigned long long *amask = reinterpret_cast<unsigned long long *>(ored + (size_t)kAttnWaves * kAttnQB * HD);   // [QB][4]

  const int h = blockIdx.x, b = blockIdx.y;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int K = a.K, d = a.d, cap = a.cap;
  const int row0 = b * K;
  const int jb = SPLIT ? (int)(gridDim.z - 1 - blockIdx.z) * kAttnQB : 0, je = SPLIT ? min(K, jb + kAttnQB) : K;   // this workgroup's queries
  if (episode_sits_out(a.skip, a.prefix_len, b, K, cap)) {
    for (int idx = tid; idx < (je - jb) * HD; idx += kAttnThreads)
      attn_store(a, row0 + jb + idx / HD, h * HD + (idx % HD), 0.f);
    return;
  }
  int P = a.prefix_len[b];
  P = max(0, min(P, cap - K));  // never index past the cache, whatever the caller passed
  uint16_t *kc = a.k_cache + ((size_t)(b * a.H + h) * cap) * HD;
  uint16_t *vc = a.v_cache + ((size_t)(b * a.H + h) * cap) * HD;

  if (!SPLIT) {
    attn_append_rows<HD, TREE>(a, b, h, P, tid, kAttnThreads, 0, K);
    __syncthreads();  // the rotated fp32 keys are read back below by other waves of this workgroup
  }

  const int li = tid % LPK;   // which 8 channels of a row this lane covers
  const int g = tid / LPK;    // which key stream this lane belongs to
  {                       // one block of at most 8 queries per workgroup
    const int j0 = jb;
    const int nq = min(kAttnQB, K - j0);
    const int nkeys = P + j0 + nq;  // keys visible to the last query of the block
    for (int idx = tid; idx < kAttnQB * HALF; idx += kAttnThreads) {
      const int j = idx / HALF, i = idx - j * HALF;
      float r1 = 0.f, r2 = 0.f;
      if (j < nq) {
        const float *src = a.qkv + (size_t)(row0 + j0 + j) * 3 * d + h * HD;
        const float2 cs = a.rope[(size_t)(P + (TREE ? a.depth[row0 + j0 + j] : j0 + j)) * HALF + i];
        const float q1 = src[i], q2 = src[i + HALF];
        r1 = (q1 * cs.x - q2 * cs.y) * a.scale;
        r2 = (q2 * cs.x + q1 * cs.y) * a.scale;
      }
      qs[j * HD + i] = r1;
      qs[j * HD + i + HALF] = r2;
    }
    if (TREE && tid < kAttnQB * 4)
      amask[tid] = (tid >> 2) < nq ? a.anc[(size_t)(row0 + j0 + (tid >> 2)) * 4 + (tid & 3)] : 0ull;
    __syncthreads();
    float qf[kAttnQB][8];
#pragma unroll
    for (int j = 0; j < kAttnQB; ++j)
#pragma unroll
      for (int i = 0; i < 8; ++i) qf[j][i] = qs[j * HD + li * 8 + i];

    // is new row r - P visible to query j0 + li?  (tree mode: the bits were put in LDS with the queries)
    auto sees_new = [&](int r) __attribute__((always_inline)) {
      if (!TREE) return r <= P + j0 + li;
      const int t = r - P;
      return li < kAttnQB && ((amask[li * 4 + (t >> 6)] >> (t & 63)) & 1ull) != 0;
    };

    // ---- pass 1: scores ----
    auto score_key = [&](const float (&kf)[8], int r, bool vis) __attribute__((always_inline)) {
      float s[kAttnQB];
#pragma unroll
      for (int j = 0; j < kAttnQB; ++j) {
        float t = 0.f;
#pragma unroll
        for (int i = 0; i < 8; ++i) t = fmaf(qf[j][i], kf[i], t);
        s[j] = t;
      }
#pragma unroll
      for (int off = LPK / 2; off > 0; off >>= 1)
#pragma unroll
        for (int j = 0; j < kAttnQB; ++j) s[j] += __shfl_xor(s[j], off, kWave);
      float mine = s[0];
#pragma unroll
      for (int j = 1; j < kAttnQB; ++j) mine = (li == j) ? s[j] : mine;
      if (li < kAttnQB) sc[(size_t)li * cap + r] = vis ? mine : -INFINITY;
    };
    // prefix rows (bf16, from the cache) on the matrix cores: a tile of 16 keys is the A operand of
    // v_mfma_f32_16x16x32_bf16 straight from the cache (lane l: key l%16, 8 consecutive channels), the
    // block's queries are the B operand, each fp32 query as a bf16 head (columns 0-7) and a bf16 tail
    // (columns 8-15), kept in registers for the whole pass; lane l then holds the scores of keys
    // 4*(l/16)..+3 against column l%16, and head and tail columns are added with one exchange.  (With
    // plain FMAs every key cost 64 of them plus a 32-step butterfly over the 16 lanes that share a row.)
    {
      constexpr int KS = HD / 32;
      const int lr = lane & 15, lg = lane >> 4;
      typedef unsigned int attn_u32x4 __attribute__((ext_vector_type(4)));
      attn_u32x4 qb[KS];
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        uint32_t w[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const float x0 = qs[(lr & 7) * HD + ks * 32 + lg * 8 + 2 * i], x1 = qs[(lr & 7) * HD + ks * 32 + lg * 8 + 2 * i + 1];
          uint32_t h0, l0, h1, l1;
          split_bf16(x0, h0, l0);
          split_bf16(x1, h1, l1);
          w[i] = lr < 8 ? (h0 | (h1 << 16)) : (l0 | (l1 << 16));
        }
        qb[ks] = attn_u32x4{w[0], w[1], w[2], w[3]};
      }
      constexpr int TU = 2;                           // tiles a wave requests before it uses the first
      const int n_tiles = (P + 15) / 16;
      for (int t0 = wave; t0 < n_tiles; t0 += kAttnWaves * TU) {
        attn_u32x4 kf[TU][KS];
#pragma unroll
        for (int u = 0; u < TU; ++u) {
          const int r = min((t0 + u * kAttnWaves) * 16 + lr, P - 1);      // rows past the prefix repeat its last row
#pragma unroll
          for (int ks = 0; ks < KS; ++ks)
            kf[u][ks] = *reinterpret_cast<const attn_u32x4 *>(kc + (size_t)r * HD + ks * 32 + lg * 8);
        }
#pragma unroll
        for (int u = 0; u < TU; ++u) {
          const int t = t0 + u * kAttnWaves;
          if (t < n_tiles) {                          // uniform over the wave
            f32x4 acc = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int ks = 0; ks < KS; ++ks)
              acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, kf[u][ks]), __builtin_bit_cast(bf16x8, qb[ks]),
                                                            acc, 0, 0, 0);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              const float v = acc[i] + __shfl_xor(acc[i], 8, kWave);     // head column + tail column
              const int r = t * 16 + lg * 4 + i;
              if (lr < kAttnQB && r < P) sc[(size_t)lr * cap + r] = v;
            }
          }
        }
      }
    }
    // the block's own rows (fp32, rotated in place above)
    for (int r = P + g; r < nkeys; r += G) {
      const float *kp = a.qkv + (size_t)(row0 + r - P) * 3 * d + d + h * HD + li * 8;
      const float4 k0 = *reinterpret_cast<const float4 *>(kp), k1 = *reinterpret_cast<const float4 *>(kp + 4);
      const float kf[8] = {k0.x, k0.y, k0.z, k0.w, k1.x, k1.y, k1.z, k1.w};
      score_key(kf, r, sees_new(r));
    }
    __syncthreads();

    // ---- softmax per query: one wave per row, lanes stride over the keys ----
    for (int j = wave; j < nq; j += kAttnWaves) {
      float *row = sc + (size_t)j * cap;
      float mx = -INFINITY;
      for (int r = lane; r < nkeys; r += kWave) mx = fmaxf(mx, row[r]);
      mx = wave_max(mx);
      float sum = 0.f;
      for (int r = lane; r < nkeys; r += kWave) {
        const float p = expf(row[r] - mx);
        row[r] = p;
        sum += p;
      }
      sum = wave_sum(sum);
      if (lane == 0) inv_l[j] = 1.0f / sum;
    }
    __syncthreads();

    // ---- pass 2: weighted sum of the value rows ----
    float o[kAttnQB][8];
#pragma unroll
    for (int j = 0; j < kAttnQB; ++j)
#pragma unroll
      for (int i = 0; i < 8; ++i) o[j][i] = 0.f;
    auto add_value = [&](const float (&vf)[8], int r) __attribute__((always_inline)) {
#pragma unroll
      for (int j = 0; j < kAttnQB; ++j) {
        const float p = (j < nq) ? sc[(size_t)j * cap + r] : 0.f;
#pragma unroll
        for (int i = 0; i < 8; ++i) o[j][i] = fmaf(p, vf[i], o[j][i]);
      }
    };
    for (int r0 = g; r0 < P; r0 += G * kAttnU) {
      uint4 vv[kAttnU];
#pragma unroll
      for (int u = 0; u < kAttnU; ++u) {
        const int r = r0 + u * G;
        vv[u] = r < P ? *reinterpret_cast<const uint4 *>(vc + (size_t)r * HD + li * 8) : make_uint4(0, 0, 0, 0);
      }
#pragma unroll
      for (int u = 0; u < kAttnU; ++u) {
        const int r = r0 + u * G;
        if (r < P) {
          float vf[8];
          attn_unpack8(vv[u], vf);
          add_value(vf, r);
        }
      }
    }
    for (int r = P + g; r < nkeys; r += G) {
      const float *vp = a.qkv + (size_t)(row0 + r - P) * 3 * d + 2 * d + h * HD + li * 8;
      const float4 v0 = *reinterpret_cast<const float4 *>(vp), v1 = *reinterpret_cast<const float4 *>(vp + 4);
      const float vf[8] = {v0.x, v0.y, v0.z, v0.w, v1.x, v1.y, v1.z, v1.w};
      add_value(vf, r);
    }
#pragma unroll
    for (int off = LPK; off < kWave; off <<= 1)
#pragma unroll
      for (int j = 0; j < kAttnQB; ++j)
#pragma unroll
        for (int i = 0; i < 8; ++i) o[j][i] += __shfl_xor(o[j][i], off, kWave);
    if (lane < LPK) {
#pragma unroll
      for (int j = 0; j < kAttnQB; ++j)
#pragma unroll
        for (int i = 0; i < 8; ++i) ored[(size_t)(wave * kAttnQB + j) * HD + lane * 8 + i] = o[j][i];
    }
    __syncthreads();
    for (int idx = tid; idx < nq * HD; idx += kAttnThreads) {
      const int j = idx / HD, c = idx - j * HD;
      float t = 0.f;
#pragma unroll
      for (int w = 0; w < kAttnWaves; ++w) t += ored[(size_t)(w * kAttnQB + j) * HD + c];
      attn_store(a, row0 + j0 + j, h * HD + c, t * inv_l[j]);
    }
    __syncthreads();
  }
}

}  // namespace heisd
