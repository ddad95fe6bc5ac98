// Exact-order value codec of the bit-width ladder: b-bit values, b = 2, 3, 4 (the K3/V2 row of Tab. 3 and the
// K2V2 / K3V3 / K4V4 columns of Tab. 5), in the token-major bit-stream layout: a token's 128 codes form a
// little-endian bit stream, channel c at bits [b c, b c + b) of the token's 16 b bytes. (Keys and matrix-core
// values: codec_block.hip.)
//
// One work-group of 128 threads, thread = output channel, per 32-token window: the exact-mode order of the
// 2-bit codec -- y_c = sum_j fl(R_cj v_j) left to right in fp32, n16 by the halving tree -- and code = #{k :
// y_c > fl(n16 tau_k)} against the 2^b - 1 thresholds. A thread holds its row of R_m in registers for each
// modality present in the window (R is read once per window, not once per token); then a thread per (token,
// 32 channels) packs b dwords.
#include "launch.hpp"

namespace okvq {
namespace {

// OR the 32 codes of channels 32 part .. 32 part + 31 (one per byte of `codes`) into the b dwords
// they occupy: bits b (c - 32 part) of the run starting at dword b part.
template <int kBits>
__device__ __forceinline__ void pack32(const uint32_t (&cw)[8], uint32_t (&w)[kBits]) {
#pragma unroll
  for (int i = 0; i < kBits; ++i) w[i] = 0u;
#pragma unroll
  for (int c = 0; c < 32; ++c) {
    const uint32_t v = (cw[c >> 2] >> (8 * (c & 3))) & 0xffu;
    const int bit = kBits * c, d = bit >> 5, sh = bit & 31;
    w[d] |= v << sh;
    if (sh + kBits > 32) w[d + 1] |= v >> (32 - sh);
  }
}

template <int kBits>
__device__ __forceinline__ void store_run(uint8_t* row, int part, const uint32_t (&w)[kBits]) {
  uint32_t* p = reinterpret_cast<uint32_t*>(row) + kBits * part;
#pragma unroll
  for (int i = 0; i < kBits; ++i) p[i] = w[i];
}

__device__ __forceinline__ float tree_norm_lds(const float* xs) {  // xs: 128 floats (LDS)
  float tt[64];
#pragma unroll
  for (int i = 0; i < 64; ++i) tt[i] = xs[i] * xs[i] + xs[i + 64] * xs[i + 64];
#pragma unroll
  for (int n = 32; n >= 1; n >>= 1) {
#pragma unroll
    for (int i = 0; i < n; ++i) tt[i] = tt[i] + tt[i + n];
  }
  return sqrt_rn(tt[0]);
}

// The value tokens [begin, len) of sequence b: stateless [0, lens), append from the device lengths.
__device__ __forceinline__ void value_span(const LadderValueArgs& a, int bz, int b, int& begin, int& len) {
  begin = 0;
  len = a.lens.lens[bz];
  if (a.begin_dev) {
    begin = min(max(a.begin_dev[b], 0), a.cap);
    len = min(begin + min(max(a.count_dev[b], 0), a.n_rows), a.cap);
  }
}

template <int kBits>
__global__ __launch_bounds__(128) void k_ladder_values(LadderValueArgs a) {
  constexpr int kTop = (1 << kBits) - 1;
  constexpr int kRowBytes = 16 * kBits;
  __shared__ __attribute__((aligned(16))) float xs[kW][kD];
  __shared__ float nrm[kW];
  __shared__ int mods[kW];
  __shared__ __attribute__((aligned(16))) uint8_t ct[kW][kD];
  const int h = blockIdx.y, bz = blockIdx.z, b = a.b0 + bz;
  int begin, len;
  value_span(a, bz, b, begin, len);
  const int t0 = begin + kW * blockIdx.x;
  if (t0 >= len) return;
  const int c = threadIdx.x;
  const size_t seq = (size_t)b * a.H + h;
  for (int t = 0; t < kW; ++t) {
    const int tok = t0 + t;
    xs[t][c] = (tok < len) ? h2f(a.v[(seq * a.n_rows + (tok - begin)) * kD + c]) : 0.0f;
  }
  if (c < kW) {
    const int tok = t0 + c;
    mods[c] = (tok < len) ? (int)a.modality[(size_t)b * a.n_rows + (tok - begin)] : -1;
    if (tok < len && a.mod_out && h == 0) a.mod_out[(size_t)b * a.cap + tok] = (uint8_t)mods[c];
  }
  __syncthreads();
  if (c < kW) {
    const int tok = t0 + c;
    const uint32_t n16 = (tok < len) ? norm_to_f16(tree_norm_lds(xs[c])) : 0u;
    nrm[c] = h2f(n16);
    if (tok < len) a.v_norm[seq * a.cap + tok] = (uint16_t)n16;
  }
  __syncthreads();
  // codes default to 0 (padded or out-of-contract tokens); then, per modality present in the window,
  // this thread's row c of R_m in registers against every token of that modality
  for (int t = 0; t < kW; ++t) ct[t][c] = 0;
  for (int m = 0; m < 3; ++m) {
    bool any = false;
    for (int t = 0; t < kW; ++t) any |= mods[t] == m;
    if (!any) continue;  // uniform over the work-group
    float rr[kD];
    const float4* rp = reinterpret_cast<const float4*>(a.rot + ((size_t)m * kD + c) * kD);
#pragma unroll
    for (int k4 = 0; k4 < kD / 4; ++k4) {
      const float4 f = rp[k4];
      rr[4 * k4] = f.x;
      rr[4 * k4 + 1] = f.y;
      rr[4 * k4 + 2] = f.z;
      rr[4 * k4 + 3] = f.w;
    }
    for (int t = 0; t < kW; ++t) {
      if (mods[t] != m) continue;
      const float4* xr = reinterpret_cast<const float4*>(xs[t]);
      float acc = 0.0f;
#pragma unroll
      for (int k4 = 0; k4 < kD / 4; ++k4) {  // left to right, no contraction: the exact order
        const float4 x4 = xr[k4];
        acc = acc + rr[4 * k4] * x4.x;
        acc = acc + rr[4 * k4 + 1] * x4.y;
        acc = acc + rr[4 * k4 + 2] * x4.z;
        acc = acc + rr[4 * k4 + 3] * x4.w;
      }
      const float nv = nrm[t];
      uint32_t code = 0;
#pragma unroll
      for (int k = 0; k < kTop; ++k) code += (uint32_t)(acc > nv * a.tau[k]);
      ct[t][c] = (uint8_t)code;
    }
  }
  __syncthreads();
  // packing: thread = (token c / 4, channels 32 (c % 4) .. +31)
  const int t = c >> 2, part = c & 3, tok = t0 + t;
  if (tok >= len) return;
  uint32_t cw[8];
  const uint4* src = reinterpret_cast<const uint4*>(&ct[t][32 * part]);
  const uint4 u0 = src[0], u1 = src[1];
  cw[0] = u0.x; cw[1] = u0.y; cw[2] = u0.z; cw[3] = u0.w;
  cw[4] = u1.x; cw[5] = u1.y; cw[6] = u1.z; cw[7] = u1.w;
  uint32_t w[kBits];
  pack32<kBits>(cw, w);
  store_run<kBits>(a.v_codes + (seq * a.cap + tok) * kRowBytes, part, w);
}

}  // namespace

hipError_t launch_ladder_values(const LadderValueArgs& a, int bits, int nb, int max_len, hipStream_t s) {
  if (nb <= 0 || max_len <= 0) return hipSuccess;
  const dim3 grid((max_len + kW - 1) / kW, a.H, nb);
  switch (bits) {
    case 2: hipLaunchKernelGGL(k_ladder_values<2>, grid, dim3(128), 0, s, a); break;
    case 3: hipLaunchKernelGGL(k_ladder_values<3>, grid, dim3(128), 0, s, a); break;
    case 4: hipLaunchKernelGGL(k_ladder_values<4>, grid, dim3(128), 0, s, a); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace okvq
