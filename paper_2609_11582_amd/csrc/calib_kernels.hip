// Modality-aware value-rotation calibration (Sec. 2.3, Eq. 5): the attention weight of every
// calibration token, w_j = sum_i alpha_{i,j}^2 over the causal calibration queries i of every query
// head that reads the KV head, and the weighted second moment per modality,
// C_m = sum_{j in m} w_j v_j^T v_j. The eigendecomposition and R_m = H U_m^T run on the host
// (api.hip).
//
// Scores are dense contractions on the matrix cores: v_mfma_f32_32x32x16_f16 with A = 32 rows of the
// tile in LDS and B = 32 rows held in registers for the whole walk. Lane l holds A[l % 32][8 (l / 32)
// + e], B[8 (l / 32) + e][l % 32] and D[8 (i / 4) + 4 (l / 32) + i % 4][l % 32], i = 0 .. 15: for a
// row-major fp16 [token][128] operand, both A and B fragments of k-step ks are the 16 bytes at channel
// 16 ks + 8 (l / 32) of token l % 32. A lane thus owns one column (a query in the first pass, a key in
// the second) and half of the other side's rows, so the running maximum, the sums and the column
// weights stay in the lane; only the end of a walk crosses lanes.
//
//  k_calib_rowstats   (m_i, l_i) of every query row: base-2 running max and sum of 2^(s - m)
//                     over the causal keys (32 queries per wave, keys in tiles of 64);
//  k_calib_colweights per query head, the sum over its queries of alpha^2 for every key (32 keys per
//                     wave, every later query tile), alpha = 2^(s - m_i) / l_i;
//  k_calib_groupsum   w_j = the sum over the query heads of the group;
//  k_calib_covariance partial C_m of a run of 64-token chunks on the matrix cores (A = w v split into
//                     fp16 hi + lo parts, B = v), one partial per (run, modality);
//  k_calib_reduce     C_m = the sum of the partials, in a fixed order.
#include <algorithm>
#include <cfloat>
#include <cmath>

#include "launch.hpp"

namespace okvq {

typedef _Float16 c_half8 __attribute__((ext_vector_type(8)));
typedef float c_floatx4 __attribute__((ext_vector_type(4)));
typedef float c_floatx16 __attribute__((ext_vector_type(16)));

constexpr int kCalThreads = 256;  // 4 waves
constexpr int kCalTile = 64;      // rows of the tile staged in LDS: keys (rowstats) or queries (colweights)
constexpr int kCalWave = 32;      // queries (rowstats) or keys (colweights) held by a wave
constexpr int kCalGroup = 4 * kCalWave;  // and by a work-group
constexpr int kCovChunk = 64;     // tokens per staged covariance chunk

__device__ __forceinline__ c_half8 as_h8(uint4 u) { return __builtin_bit_cast(c_half8, u); }

// The eight k-step fragments of token row `row` (fp16 [128]) for this lane: channels 16 ks + 8
// (lane / 32) .. + 7. Rows at or beyond `valid` read as zero. neg: the row negated (a negative
// softmax scale is carried by the held operand, so that the scores' scale is non-negative).
__device__ __forceinline__ void load_held(const uint16_t* base, int row, int valid, int lane, bool neg, uint4 (&f)[8]) {
  const uint32_t flip = neg ? 0x80008000u : 0u;
  const uint4* p = reinterpret_cast<const uint4*>(base + (size_t)min(row, valid - 1) * kD) + (lane >> 5);
#pragma unroll
  for (int ks = 0; ks < 8; ++ks) {
    const uint4 v = p[2 * ks];
    f[ks] = row < valid ? make_uint4(v.x ^ flip, v.y ^ flip, v.z ^ flip, v.w ^ flip) : make_uint4(0, 0, 0, 0);
  }
}

// A tile of 64 token rows (fp16 [128], 16 chunks of 16 bytes) in LDS: chunk c of row r in slot c ^ (r %
// 16) of its 256 bytes, so that the lanes reading one chunk of 16 rows hit distinct banks. Filled by
// direct memory-to-LDS loads, four per wave (rows 16 wave .. + 15); rows at or beyond `valid` repeat
// the last one (their scores are masked or weighted by zero).
constexpr int kTileBytes = kCalTile * 2 * kD;
__device__ __forceinline__ void tile_issue(const uint16_t* base, int row0, int valid, int wave, int lane, uint32_t lds) {
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int r = 16 * wave + 4 * u + (lane >> 4);
    const uint4* p = reinterpret_cast<const uint4*>(base + (size_t)min(row0 + r, valid - 1) * kD);
    dma16(p + ((lane & 15) ^ (r & 15)), lds + (16 * wave + 4 * u) * 2 * kD);
  }
}
// this wave's direct loads have landed; after the work-group barrier that follows, every wave's have
__device__ __forceinline__ void tile_wait() { __asm__ volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// scores (unscaled) of the tile's two 32-row blocks against the held operand, as two independent
// chains of matrix products
__device__ __forceinline__ void score_tile(const uint8_t* t, int lane, const uint4 (&held)[8], c_floatx16 (&s)[2]) {
  const int r = lane & 31, x = (lane >> 5) ^ (r & 15);
#pragma unroll
  for (int i = 0; i < 16; ++i) s[0][i] = s[1][i] = 0.0f;
#pragma unroll
  for (int ks = 0; ks < 8; ++ks) {
    const uint8_t* p = t + r * 2 * kD + 16 * (x ^ (2 * ks));
    const uint4 a0 = *reinterpret_cast<const uint4*>(p), a1 = *reinterpret_cast<const uint4*>(p + 32 * 2 * kD);
    s[0] = __builtin_amdgcn_mfma_f32_32x32x16_f16(as_h8(a0), as_h8(held[ks]), s[0], 0, 0, 0);
    s[1] = __builtin_amdgcn_mfma_f32_32x32x16_f16(as_h8(a1), as_h8(held[ks]), s[1], 0, 0, 0);
  }
  // six fragments in flight ahead of the products (the scheduler alone keeps two: 99 -> 94 us for the
  // column weights of 4096 tokens, 28 heads)
  __builtin_amdgcn_sched_group_barrier(0x100, 6, 0);
#pragma unroll
  for (int i = 0; i < 5; ++i) {
    __builtin_amdgcn_sched_group_barrier(0x008, 2, 0);
    __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
  }
  __builtin_amdgcn_sched_group_barrier(0x008, 6, 0);
}
// row of score i of a block for this lane
__device__ __forceinline__ int score_row(int i, int lane) { return 8 * (i >> 2) + 4 * (lane >> 5) + (i & 3); }

// Work-group n of `total` in the order of a causal pass, longest walk first. Work-groups are dealt out
// to the 256 compute units in turn: the runs of 256 whose number has an odd count of one bits are
// reversed, so that a compute unit's walks add up to nearly the same (4096 tokens, 28 heads: 112 .. 120
// tiles instead of 102 .. 149).
__device__ __forceinline__ int walk_rank(int n, int total) {
  const int run = n >> 8;
  return ((__popc(run) & 1) && (run + 1) * 256 <= total) ? run * 256 + 255 - (n & 255) : n;
}

// 2^x on the hardware unit: results below 2^-126 flush to zero (they do not count in a sum of at
// least 1, or in a weight that other terms dominate)
__device__ __forceinline__ float hw_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// ---- pass 1: row statistics. One work-group per (query tile of 128, head, sequence), longest first;
// wave w holds queries 32 w .. 32 w + 31 of the tile as B operands and walks the causal key tiles of 64
// (staged in LDS, the next one loading during the current one's MFMAs). stats[(bz Hq + j) N + i] =
// (m_i, l_i): m in base-2 score units (scores times sm_scale log2 e), l_i = sum_{t <= i} 2^(s_it - m_i).
// A lane keeps its own running maximum and sum over its half of the keys; the two lanes of a query
// are joined at the end.
// Bound by issue: per score and SIMD a half v_max3, an fma, a quarter-rate v_exp_f32 and an add are 26
// cycles of a wave and the MFMAs 16 (a wave of 32 queries reads a key fragment from LDS once per 32
// products, half of what 16x16 blocks need). 4096 tokens, 28 heads: 265 -> 89 us (16x16 blocks, exp2f with
// its handling of subnormal results and a cross-lane maximum per tile before). ----
__global__ __launch_bounds__(kCalThreads, 4) void k_calib_rowstats(const uint16_t* __restrict__ q,
                                                                   const uint16_t* __restrict__ k, LenArgs lens, int b0,
                                                                   int nb, int N, int H, int Hq, float scale2,
                                                                   float2* __restrict__ stats) {
  __shared__ __attribute__((aligned(16))) uint8_t kt[2][kTileBytes];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int units = Hq * nb, total = (int)gridDim.x;
  const int rank = walk_rank((int)blockIdx.x, total);
  const int j = (rank % units) % Hq, bz = (rank % units) / Hq, b = b0 + bz;
  const int q0 = (total / units - 1 - rank / units) * kCalGroup;  // the last tile has the longest walk
  const int h = j / (Hq / H);
  const int L = min(max(lens.lens[bz], 0), N);
  if (q0 >= L) return;  // (uniform over the work-group)
  const int i0 = q0 + kCalWave * wave, qi = i0 + (lane & 31);
  const uint16_t* kbase = k + ((size_t)b * H + h) * N * kD;
  uint4 held[8];
  load_held(q + ((size_t)b * Hq + j) * N * kD, qi, L, lane, scale2 < 0.0f, held);
  const float scale = fabsf(scale2);
  float m = -__builtin_inff(), l = 0.0f;
  const int t_end = min(q0 + kCalGroup, L);  // keys up to the last query of the tile
  const uint32_t lds = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(uintptr_t)&kt[0][0]);
  tile_issue(kbase, 0, t_end, wave, lane, lds);
  int buf = 0;
  for (int t0 = 0; t0 < t_end; t0 += kCalTile, buf ^= 1) {
    tile_wait();
    __syncthreads();  // the tile is complete, and every wave is done with the other buffer
    if (t0 + kCalTile < t_end) tile_issue(kbase, t0 + kCalTile, t_end, wave, lane, lds + (buf ^ 1) * kTileBytes);
    if (t0 > i0 + kCalWave - 1) continue;  // every key is later than the wave's queries (wave-uniform)
    c_floatx16 s[2];
    score_tile(kt[buf], lane, held, s);
    if (t0 + kCalTile - 1 > i0) {  // keys later than a query do not count (wave-uniform)
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int i = 0; i < 16; ++i) s[kb][i] = (t0 + 32 * kb + score_row(i, lane) <= qi) ? s[kb][i] : -__builtin_inff();
    }
    float mx = s[0][0];
#pragma unroll
    for (int i = 1; i < 32; ++i) mx = fmaxf(mx, s[i >> 4][i & 15]);
    const float mn = fmaxf(m, mx * scale);
    const float ref = (mn == -__builtin_inff()) ? 0.0f : mn;  // nothing visible to this lane yet
    float p[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int i = 0; i < 32; ++i) p[i & 3] += hw_exp2(__builtin_fmaf(s[i >> 4][i & 15], scale, -ref));
    l = __builtin_fmaf(l, hw_exp2(m - ref), (p[0] + p[1]) + (p[2] + p[3]));
    m = mn;
  }
  // the query's two lanes: one of them may have seen no key (m = -inf, l = 0)
  const float mo = __shfl_xor(m, 32), lo = __shfl_xor(l, 32);
  const float mt = fmaxf(m, mo);
  l = l * hw_exp2(m - mt) + lo * hw_exp2(mo - mt);
  if (lane < 32 && qi < L) stats[((size_t)bz * Hq + j) * N + qi] = make_float2(mt, l);
}

// ---- pass 2: column weights of one query head. One work-group per (key tile of 128, head, sequence),
// longest first; wave w holds keys 32 w .. 32 w + 31 of the tile as B operands and walks the head's
// query tiles of 64 from the diagonal on (staged in LDS with their statistics as (2 m, 1 / l^2), so
// that alpha^2 = 2^(2 s - 2 m) / l^2 takes one exp2). wq[(bz Hq + j) N + t]: the head's sum over queries
// (zero beyond L); k_calib_groupsum adds the heads of each group. Bound by issue like pass 1 (two
// fmas and an exp2 per score): 206 -> 94 us at 4096 tokens, 28 heads. ----
__global__ __launch_bounds__(kCalThreads, 4) void k_calib_colweights(const uint16_t* __restrict__ q,
                                                                     const uint16_t* __restrict__ k, LenArgs lens,
                                                                     int b0, int nb, int N, int H, int Hq, float scale2,
                                                                     const float2* __restrict__ stats,
                                                                     float* __restrict__ wq) {
  __shared__ __attribute__((aligned(16))) uint8_t qt[2][kTileBytes];
  __shared__ __attribute__((aligned(16))) float2 st2[2][kCalTile];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int units = Hq * nb, total = (int)gridDim.x;
  const int rank = walk_rank((int)blockIdx.x, total);
  const int j = (rank % units) % Hq, bz = (rank % units) / Hq, b = b0 + bz;
  const int k0 = rank / units * kCalGroup;  // the first tile has the longest walk
  const int h = j / (Hq / H);
  const int L = min(max(lens.lens[bz], 0), N);
  const int t0 = k0 + kCalWave * wave, t = t0 + (lane & 31);  // the wave's keys, the lane's
  float acc[4] = {0.0f, 0.0f, 0.0f, 0.0f};
  if (k0 < L) {  // (uniform over the work-group)
    uint4 held[8];
    load_held(k + ((size_t)b * H + h) * N * kD, t, L, lane, scale2 < 0.0f, held);
    const float scale2x = 2.0f * fabsf(scale2);
    const int ntile = (L - k0 + kCalTile - 1) / kCalTile;  // query tiles from the diagonal on
    const uint16_t* qb = q + ((size_t)b * Hq + j) * N * kD;
    const float2* sb = stats + ((size_t)bz * Hq + j) * N;
    const uint32_t lds = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(uintptr_t)&qt[0][0]);
    auto issue = [&](int it, float2& sv) {
      const int qtile = k0 + kCalTile * it;
      sv = make_float2(0.f, 0.f);
      if (tid < kCalTile && qtile + tid < L) sv = sb[qtile + tid];
      tile_issue(qb, qtile, L, wave, lane, lds + (it & 1) * kTileBytes);
    };
    float2 sv;
    issue(0, sv);
    for (int it = 0, buf = 0; it < ntile; ++it, buf ^= 1) {
      // a query beyond the length gets (2 m, 1 / l^2) = (+inf, 0): its alpha^2 is 2^-inf * 0 = 0
      if (tid < kCalTile)
        st2[buf][tid] = (sv.y > 0.0f) ? make_float2(2.0f * sv.x, 1.0f / (sv.y * sv.y)) : make_float2(__builtin_inff(), 0.0f);
      tile_wait();
      __syncthreads();  // the tile is complete, and every wave is done with the other buffer
      if (it + 1 < ntile) issue(it + 1, sv);
      const int qtile = k0 + kCalTile * it;
      if (qtile + kCalTile - 1 < t0) continue;  // every query precedes the wave's keys (wave-uniform)
      c_floatx16 s[2];
      score_tile(qt[buf], lane, held, s);
      if (qtile < t0 + kCalWave - 1) {  // a query before the key does not count (wave-uniform)
#pragma unroll
        for (int i = 0; i < 32; ++i)
          s[i >> 4][i & 15] = (t <= qtile + 32 * (i >> 4) + score_row(i & 15, lane)) ? s[i >> 4][i & 15] : -__builtin_inff();
      }
#pragma unroll
      for (int qb2 = 0; qb2 < 2; ++qb2) {
#pragma unroll
        for (int i4 = 0; i4 < 4; ++i4) {
          const float4* sp = reinterpret_cast<const float4*>(&st2[buf][32 * qb2 + 8 * i4 + 4 * (lane >> 5)]);
          const float4 u0 = sp[0], u1 = sp[1];
          acc[0] = __builtin_fmaf(hw_exp2(__builtin_fmaf(s[qb2][4 * i4], scale2x, -u0.x)), u0.y, acc[0]);
          acc[1] = __builtin_fmaf(hw_exp2(__builtin_fmaf(s[qb2][4 * i4 + 1], scale2x, -u0.z)), u0.w, acc[1]);
          acc[2] = __builtin_fmaf(hw_exp2(__builtin_fmaf(s[qb2][4 * i4 + 2], scale2x, -u1.x)), u1.y, acc[2]);
          acc[3] = __builtin_fmaf(hw_exp2(__builtin_fmaf(s[qb2][4 * i4 + 3], scale2x, -u1.z)), u1.w, acc[3]);
        }
      }
    }
  }
  float sum = (acc[0] + acc[1]) + (acc[2] + acc[3]);
  sum += __shfl_xor(sum, 32);
  if (lane < 32 && t < N) wq[((size_t)bz * Hq + j) * N + t] = (t < L) ? sum : 0.0f;
}

// ---- w[(b H + h) N + t] = sum over the group's query heads, in head order. Grid (N / 256, H, nb) ----
__global__ __launch_bounds__(256) void k_calib_groupsum(const float* __restrict__ wq, int b0, int N, int H, int Hq,
                                                        float* __restrict__ w) {
  const int t = blockIdx.x * 256 + threadIdx.x, h = blockIdx.y, bz = blockIdx.z;
  if (t >= N) return;
  const int G = Hq / H;
  float s = 0.0f;
  for (int jj = 0; jj < G; ++jj) s += wq[((size_t)bz * Hq + h * G + jj) * N + t];
  w[((size_t)(b0 + bz) * H + h) * N + t] = s;
}

// ---- weighted covariance partials. Grid (runs of chunks, 2 H, sequences): a work-group takes
// run_chunks chunks of 64 tokens of one (sequence, KV head) and the output rows 64 half .. + 63, and writes
// partial[((bz H + h) nrun + run) 3 + m][c1][c2] = sum over the run's tokens t of modality m of w_t
// v_t[c1] v_t[c2]. A chunk is staged channel-major in LDS: v (fp16) and, for the work-group's rows, the hi
// / lo fp16 parts of w v; the next chunk's rows are loaded while it is used. Wave w accumulates the 16
// rows 16 w .. of the three modalities in registers over the whole run, so that the partials written
// here and read by the reduction are 1 / run_chunks of the chunks'. Bound by the partials' traffic: two
// chunks a run still give a work-group per compute unit at 4096 tokens and 4 heads, and 11.9 + 17.2 us
// for the two kernels became 11.7 + 5.8 us (four: 16.4 + 5.0 us). With fewer than 64 chunks in all the second
// chunk's chain is what the call takes, not the traffic: one a run (500 tokens, one head 11.7 -> 9.3 us a
// call, 4 heads 13.0 -> 11.8; at 64 chunks two a run take 14.6 us against 15.1) ----
constexpr int kCovShort = 64;
constexpr int kCovRows = kD / 2;  // output rows per work-group
__global__ __launch_bounds__(kCalThreads) void k_calib_covariance(const uint16_t* __restrict__ v,
                                                                  const uint8_t* __restrict__ modality,
                                                                  const float* __restrict__ w, LenArgs lens, int b0,
                                                                  int N, int H, int nrun, int run_chunks,
                                                                  float* __restrict__ partial) {
  __shared__ __attribute__((aligned(16))) _Float16 vt[kD][kCovChunk + 8];         // v[t][c] at [c][t]
  __shared__ __attribute__((aligned(16))) _Float16 whi[kCovRows][kCovChunk + 8];  // fp16(w v)
  __shared__ __attribute__((aligned(16))) _Float16 wlo[kCovRows][kCovChunk + 8];  // fp16(w v - hi)
  __shared__ __attribute__((aligned(8))) uint8_t mods[kCovChunk];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, tid = threadIdx.x;
  const int run = blockIdx.x, h = blockIdx.y >> 1, half = blockIdx.y & 1, bz = blockIdx.z, b = b0 + bz;
  const int L = min(max(lens.lens[bz], 0), N);
  const size_t seq = (size_t)b * H + h;
  const int col = lane & 15, g = lane >> 4;
  // staging: thread (token tt = tid / 4, channel quarter cq = tid % 4): 32 channels of one token
  const int tt = tid >> 2, cq = tid & 3;
  uint4 x[4];
  float wt;
  uint32_t md;
  auto load = [&](int chunk) {
    const int tok = chunk * kCovChunk + tt;
    const bool ok = tok < L;
    const uint4* src = reinterpret_cast<const uint4*>(v + (seq * N + (ok ? tok : 0)) * kD + 32 * cq);
#pragma unroll
    for (int u = 0; u < 4; ++u) x[u] = ok ? src[u] : make_uint4(0, 0, 0, 0);
    wt = ok ? w[seq * N + tok] : 0.0f;
    md = ok ? modality[(size_t)b * N + tok] : 3u;
  };
  c_floatx4 acc[3][8];
#pragma unroll
  for (int m = 0; m < 3; ++m)
#pragma unroll
    for (int cb = 0; cb < 8; ++cb) acc[m][cb] = c_floatx4{0.f, 0.f, 0.f, 0.f};
  const int c0 = run * run_chunks, c1 = min(c0 + run_chunks, (L + kCovChunk - 1) / kCovChunk);
  if (c0 < c1) load(c0);
  for (int chunk = c0; chunk < c1; ++chunk) {
    if (chunk > c0) __syncthreads();  // every wave is done with the previous chunk
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const c_half8 hv = as_h8(x[u]);
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const int c = 32 * cq + 8 * u + e;
        vt[c][tt] = hv[e];
        if ((cq >> 1) == half) {
          const float f = (float)hv[e] * wt;
          const _Float16 hi = (_Float16)f;
          whi[c & (kCovRows - 1)][tt] = hi;
          wlo[c & (kCovRows - 1)][tt] = (_Float16)(f - (float)hi);
        }
      }
    }
    if (cq == 0) mods[tt] = (uint8_t)md;
    __syncthreads();
    if (chunk + 1 < c1) load(chunk + 1);
#pragma unroll
    for (int ks = 0; ks < kCovChunk; ks += 32) {
      const uint2 mw = *reinterpret_cast<const uint2*>(&mods[ks + 8 * g]);  // tokens ks + 8 g .. + 7 of this lane's fragments
      const uint4 ah = *reinterpret_cast<const uint4*>(&whi[16 * wave + col][ks + 8 * g]);
      const uint4 al = *reinterpret_cast<const uint4*>(&wlo[16 * wave + col][ks + 8 * g]);
      uint4 bf[8];
#pragma unroll
      for (int cb = 0; cb < 8; ++cb) bf[cb] = *reinterpret_cast<const uint4*>(&vt[16 * cb + col][ks + 8 * g]);
#pragma unroll
      for (int m = 0; m < 3; ++m) {
        uint32_t mk[4];  // per-element fp16 masks (0xffff keeps the tokens of modality m)
#pragma unroll
        for (int p2 = 0; p2 < 4; ++p2) {
          const uint32_t mm = (p2 < 2 ? mw.x : mw.y) >> (16 * (p2 & 1));
          mk[p2] = ((mm & 0xffu) == (uint32_t)m ? 0x0000ffffu : 0u) | (((mm >> 8) & 0xffu) == (uint32_t)m ? 0xffff0000u : 0u);
        }
        if (!__any((mk[0] | mk[1] | mk[2] | mk[3]) != 0u)) continue;  // (wave-uniform)
        const uint4 amh = make_uint4(ah.x & mk[0], ah.y & mk[1], ah.z & mk[2], ah.w & mk[3]);
        const uint4 aml = make_uint4(al.x & mk[0], al.y & mk[1], al.z & mk[2], al.w & mk[3]);
#pragma unroll
        for (int cb = 0; cb < 8; ++cb) {
          acc[m][cb] = __builtin_amdgcn_mfma_f32_16x16x32_f16(as_h8(amh), as_h8(bf[cb]), acc[m][cb], 0, 0, 0);
          acc[m][cb] = __builtin_amdgcn_mfma_f32_16x16x32_f16(as_h8(aml), as_h8(bf[cb]), acc[m][cb], 0, 0, 0);
        }
      }
    }
  }
  // D[4 g + i][col] of block (rows 64 half + 16 wave .., column block cb)
  float* out = partial + ((((size_t)bz * H + h) * nrun + run) * 3 * kD + kCovRows * half + 16 * wave + 4 * g) * kD + col;
#pragma unroll
  for (int m = 0; m < 3; ++m)
#pragma unroll
    for (int cb = 0; cb < 8; ++cb)
#pragma unroll
      for (int i = 0; i < 4; ++i) out[((size_t)m * kD + i) * kD + 16 * cb] = acc[m][cb][i];
}

// ---- C_m[c1][c2] = the sum of the partials in a fixed order. A work-group of 256 threads takes 64
// groups of four consecutive elements; its wave r sums the partials p = r (mod 4), eight loads in
// flight, and the four sums are added in r order. Grid (3 kD kD / 256) ----
__global__ __launch_bounds__(256) void k_calib_reduce(const float* __restrict__ partial, int nparts,
                                                      float* __restrict__ cov) {
  __shared__ __attribute__((aligned(16))) float4 part[4][64];
  const int lane = threadIdx.x & 63, r = threadIdx.x >> 6;
  const size_t e4 = (size_t)blockIdx.x * 64 + lane;
  const float4* src = reinterpret_cast<const float4*>(partial) + e4;
  constexpr size_t kStride = (size_t)3 * kD * kD / 4;
  float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
  for (int p0 = r; p0 < nparts; p0 += 32) {
    float4 x[8];
#pragma unroll
    for (int u = 0; u < 8; ++u)
      x[u] = (p0 + 4 * u < nparts) ? src[(size_t)(p0 + 4 * u) * kStride] : make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
    for (int u = 0; u < 8; ++u) s = make_float4(s.x + x[u].x, s.y + x[u].y, s.z + x[u].z, s.w + x[u].w);
  }
  part[r][lane] = s;
  __syncthreads();
  if (r != 0) return;
  float4 t = part[0][lane];
#pragma unroll
  for (int u = 1; u < 4; ++u) {
    const float4 y = part[u][lane];
    t = make_float4(t.x + y.x, t.y + y.y, t.z + y.z, t.w + y.w);
  }
  reinterpret_cast<float4*>(cov)[e4] = t;
}

size_t calib_workspace_bytes(int B, int H, int Hq, int N) {
  // row statistics (float2) and the per-head column sums (float) of up to 256 sequences
  const size_t stats = (size_t)std::min(B, kMaxLenArgs) * Hq * N * (sizeof(float2) + sizeof(float));
  const size_t nchunk = (N + kCovChunk - 1) / kCovChunk;  // (at least the runs of chunks the launch writes)
  const size_t parts = (size_t)B * H * nchunk * 3 * kD * kD * sizeof(float);
  return std::max(stats, parts);
}

hipError_t launch_calib_weights(const uint16_t* q, const uint16_t* k, const LenArgs& lens, int b0, int nb, int N,
                                int H, int Hq, float sm_scale, float* w, void* ws, hipStream_t s) {
  // Masked scores are -inf before the scale, so the scale may not be zero (-inf 0 is NaN). The least normal number
  // stands for everything below it, with the same result: a score is less than 2^39 (128 products of fp16 values),
  // so that it scales to less than 2^-87, whose power of two rounds to 1.
  float scale2 = sm_scale * 1.4426950408889634f;
  if (std::fabs(scale2) < FLT_MIN) scale2 = FLT_MIN;
  float2* stats = static_cast<float2*>(ws);
  const long groups = (long)((N + kCalGroup - 1) / kCalGroup) * Hq * nb;
  if (groups > INT32_MAX) return hipErrorInvalidValue;
  const dim3 gq((unsigned)groups);
  hipLaunchKernelGGL(k_calib_rowstats, gq, dim3(kCalThreads), 0, s, q, k, lens, b0, nb, N, H, Hq, scale2, stats);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  float* wq = reinterpret_cast<float*>(stats + (size_t)nb * Hq * N);
  hipLaunchKernelGGL(k_calib_colweights, gq, dim3(kCalThreads), 0, s, q, k, lens, b0, nb, N, H, Hq, scale2,
                     static_cast<const float2*>(stats), wq);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  hipLaunchKernelGGL(k_calib_groupsum, dim3((N + 255) / 256, H, nb), dim3(256), 0, s, static_cast<const float*>(wq), b0,
                     N, H, Hq, w);
  return hipGetLastError();
}

int calib_covariance_run(int B, int H, int N) {
  return (int64_t)B * H * ((N + kCovChunk - 1) / kCovChunk) < kCovShort ? 1 : 2;
}
int calib_covariance_runs(int run_chunks, int N) { return (N + run_chunks * kCovChunk - 1) / (run_chunks * kCovChunk); }

hipError_t launch_calib_covariance(const uint16_t* v, const uint8_t* modality, const float* w, const LenArgs& lens,
                                   int b0, int nb, int N, int H, int run_chunks, float* partial, int part0, float* cov,
                                   bool reduce, int nparts_total, hipStream_t s) {
  const int nrun = calib_covariance_runs(run_chunks, N);
  hipLaunchKernelGGL(k_calib_covariance, dim3(nrun, 2 * H, nb), dim3(kCalThreads), 0, s, v, modality, w, lens, b0, N, H,
                     nrun, run_chunks, partial + (size_t)part0 * 3 * kD * kD);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || !reduce) return e;
  hipLaunchKernelGGL(k_calib_reduce, dim3(3 * kD * kD / 256), dim3(256), 0, s, static_cast<const float*>(partial),
                     nparts_total, cov);
  return hipGetLastError();
}

}  // namespace okvq
