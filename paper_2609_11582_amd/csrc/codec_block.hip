// Block codec: keys and MFMA-mode values of an append (or of a stateless call) in one launch of many
// small work-groups, for the 2-bit layout (every key metadata format) and the bit-width ladder (Sec. 2.1
// Eq. 2 and Sec. 2.3 Eq. 4 for keys; Sec. 2.3 Eq. 6 with the codebook of Eq. 3 for values). The results
// are the bytes of the tile codec (codec_fused.hip) and of the ladder's exact-order definitions: the same
// operations in the same order, spread so that four waves share a SIMD instead of two.
//
// A work-group of 256 threads has one role:
//  * keys, units of 64 tokens (two 32-token windows): thread (t, q) holds the 32 channels 32 u + 8 q + e
//    (u, q < 4, e < 8) of token t, so that a token spans a DPP quad and a load instruction reads 64
//    contiguous bytes of a row. The norm tree's levels 64, 32 and 4 .. 1 and the butterflies h = 1, 2, 4,
//    32, 64 stay in the lane; the levels and stages 16 and 8 cross the quad. The directions go to an LDS
//    tile, thread (window, channel) reduces the window's minimum and maximum (exact in any order) and
//    forms the metadata, and every thread codes its 32 channels;
//  * values, units of 128 tokens: the rows go straight to LDS as MFMA operands; wave v forms the fp16
//    norms of 32 tokens, then the output channels 32 v .. 32 v + 31 of all 128 tokens with its slice of
//    R_m (fp16 hi + lo) in registers, one modality at a time. The 2-bit layout takes rows = tokens (a
//    lane ends with four consecutive tokens of one channel, one byte of its layout), the ladder rows =
//    channels (a lane ends with four consecutive channels of one token, contiguous bits of its stream).
// One work-group per unit: roles alternate in runs of 256 work-groups, one per compute unit, so that a
// compute unit holds both and the value role's loads and matrix products overlap the key role's VALU work.
//
// Older rows of the open window come from the fp16 key stage; the work-group of a sequence's first key
// unit, the only one that reads it, rewrites it after a barrier that follows its reads. The lengths
// advance in a launch of their own: counting finished work-groups on one word costs 11.5 ns each, one
// after another (8 us of the 39 us of a 32768-token, 4-head prefill with 1024 work-groups), the launch
// 1.3-1.6 us.
//
// Stateless 2-bit values have no prepared fragments of R_m, only the fp32 matrix, which every work-group converts:
// large calls take wider units (k_values_wide below).
//
// Bound by VALU issue (keys about 20 operations a channel, values about 8) at four waves per SIMD. 32768
// tokens, 4 KV heads: 38.7 -> 29.1 us a call for the 2-bit layout (the tile codec: two waves per SIMD), 73 ->
// 32 us at 3 bits (separate key and value kernels, which converted R_m in every work-group).
#include <hip/hip_ext.h>

#include <algorithm>

#include "lane_quant.hpp"
#include "launch.hpp"

namespace okvq {
namespace {

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef float floatx4 __attribute__((ext_vector_type(4)));

constexpr int kThreads = 256;
constexpr int kKeyUnit = 64;    // tokens per key unit
constexpr int kValUnit = 128;   // most tokens per value unit
constexpr uint32_t kRun = 256;      // work-groups per run of one role (compute units)

__device__ __forceinline__ half8 as_half8(uint4 u) { return __builtin_bit_cast(half8, u); }

struct KeyShared {
  float z[kKeyUnit][kD];     // directions: the 16-byte chunk c / 4 of token t in slot (c / 4) ^ swz(t)
  float2 stat[2][kD];        // per window and channel: (minimum, 1 / step) as the codes use them
};
struct ValueShared {
  uint4 rows[kValUnit / 16][4][64];  // the value rows as MFMA operands: [row block][k-block][lane]
  float nrm[kValUnit];       // 2-bit layout: fl(1 / T) of the value decision; ladder: fp16 norm as fp32
  uint32_t tmod[kValUnit / 16][16];  // per token: the rotation of its code (3: none)
  uint8_t ktab[3][kValUnit / 4];     // 2-bit layout: per modality and token quad, 2-bit masks of the coded tokens
  uint32_t present[4];       // per wave: bit 8 m + row block where it holds a token of modality m
};
union BlockShared {
  KeyShared k;
  ValueShared v;
};

// slot permutation of a token's chunks in the direction tile: the 16 lanes (4 tokens x 4 quad lanes) of a
// write hit distinct banks, and a column of one row is read by consecutive lanes either way
__device__ __forceinline__ int swz(int t) { return (t & 1) | ((t & 2) << 2); }

template <int kPerm>
__device__ __forceinline__ uint32_t quad_perm(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, kPerm, 0xf, 0xf, true);
}
constexpr int kXor1 = 0xB1, kXor2 = 0x4E, kNext = 0x39;  // lane q <- q ^ 1, q ^ 2, (q + 1) mod 4 of its quad

// Butterfly stage across lanes q and q ^ 1 (or q ^ 2) of a quad as own + s partner (one rounding): a + b in
// the lower lane and b - a in the upper one, the stage's a - b negated. Both lanes of a later stage's pair
// carry the same sign, so the signs multiply out and are undone by the exact sign of the final scale. One
// fmac with a DPP operand per channel (the compiler forms a move and an fma); the s_nop covers the two wait
// states between a VALU write and a DPP read of the register.
#define OKVQ_QUAD_FMAC(perm)                                                                                   \
  __asm__("s_nop 1\n\t"                                                                                        \
          "v_fmac_f32_dpp %0, %0, %8 " perm "\n\t"                                                             \
          "v_fmac_f32_dpp %1, %1, %8 " perm "\n\t"                                                             \
          "v_fmac_f32_dpp %2, %2, %8 " perm "\n\t"                                                             \
          "v_fmac_f32_dpp %3, %3, %8 " perm "\n\t"                                                             \
          "v_fmac_f32_dpp %4, %4, %8 " perm "\n\t"                                                             \
          "v_fmac_f32_dpp %5, %5, %8 " perm "\n\t"                                                             \
          "v_fmac_f32_dpp %6, %6, %8 " perm "\n\t"                                                             \
          "v_fmac_f32_dpp %7, %7, %8 " perm                                                                    \
          : "+v"(x[i]), "+v"(x[i + 1]), "+v"(x[i + 2]), "+v"(x[i + 3]), "+v"(x[i + 4]), "+v"(x[i + 5]),         \
            "+v"(x[i + 6]), "+v"(x[i + 7])                                                                     \
          : "v"(s))
template <int kMask>
__device__ __forceinline__ void signed_stage(float (&x)[32], float s) {
  static_assert(kMask == 1 || kMask == 2, "a lane of the quad");
#pragma unroll
  for (int i = 0; i < 32; i += 8) {
    if constexpr (kMask == 1)
      OKVQ_QUAD_FMAC("quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf");
    else
      OKVQ_QUAD_FMAC("quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf");
  }
}
#undef OKVQ_QUAD_FMAC

// In-lane butterfly stage over index distance d of x[8 u + e]
template <int kDist>
__device__ __forceinline__ void lane_stage(float (&x)[32]) {
#pragma unroll
  for (int i = 0; i < 32; ++i) {
    if ((i & kDist) == 0) {
      const float a = x[i], b = x[i + kDist];
      x[i] = a + b;
      x[i + kDist] = a - b;
    }
  }
}

// Direction and fp16 norm (returned) of the quad's token in the key codec's bit-exact order. raw[4 u + d]:
// channels 32 u + 8 q + 2 d, + 1; x[8 u + e]: channel 32 u + 8 q + e; sg[2 u + j]: the int8 signs of channels
// 32 u + 8 q + 4 j .. + 3, whose top bits flip the fp16 sign bits.
__device__ __forceinline__ uint32_t quad_direction(const uint32_t (&raw)[16], const uint32_t (&sg)[8], int q,
                                                   float (&x)[32]) {
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    const uint32_t r = raw[i] ^ (__builtin_amdgcn_perm(0u, sg[i >> 1], (i & 1) ? 0x030c020cu : 0x010c000cu) & 0x80008000u);
    x[2 * i] = h2f(r & 0xffffu);
    x[2 * i + 1] = h2f(r >> 16);
  }
  float t[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) {  // levels 64 and 32 (squares of fp16 values are exact)
    const float a = __builtin_fmaf(x[e], x[e], x[16 + e] * x[16 + e]);
    const float b = __builtin_fmaf(x[8 + e], x[8 + e], x[24 + e] * x[24 + e]);
    t[e] = a + b;
  }
#pragma unroll
  for (int e = 0; e < 8; ++e) t[e] = t[e] + xchg<2>(t[e]);  // level 16
#pragma unroll
  for (int e = 0; e < 8; ++e) t[e] = t[e] + xchg<1>(t[e]);  // level 8
#pragma unroll
  for (int n = 4; n >= 1; n >>= 1) {
#pragma unroll
    for (int e = 0; e < n; ++e) t[e] = t[e] + t[e + n];
  }
  const uint32_t n16 = norm_to_f16(sqrt_rn(t[0]));
  lane_stage<1>(x);
  lane_stage<2>(x);
  lane_stage<4>(x);
  const float s1 = (q & 1) ? -1.0f : 1.0f, s2 = (q & 2) ? -1.0f : 1.0f;
  signed_stage<1>(x, s1);  // h = 8
  signed_stage<2>(x, s2);  // h = 16
  lane_stage<8>(x);        // h = 32
  lane_stage<16>(x);       // h = 64
  // a zero row's butterflies are +-0: the factor 0 gives z = +-0, which the statistics (+0
  // canonicalization) and the codes treat like z = 0
  const float cinv = (n16 == 0) ? 0.0f : s1 * s2 * div_rn(kKappa, h2f(n16));
#pragma unroll
  for (int i = 0; i < 32; ++i) x[i] = x[i] * cinv;
  return n16;
}

// Code of x against the symmetric thresholds -t[n - 1] .. -t[0], 0, t[0] .. t[n - 1] (t ascending): #{k : x >
// tau_k}, a value on a threshold taking the lower code. For x <= 0 the count of magnitudes t <= |x| is that
// of t below |x|'s next float.
template <int kBits>
__device__ __forceinline__ uint32_t symmetric_code(float x, const float* t) {
  constexpr int n = (1 << (kBits - 1)) - 1;
  const bool neg = !(x > 0.0f);
  const float a = __builtin_bit_cast(float, (__builtin_bit_cast(uint32_t, x) & 0x7fffffffu) + (neg ? 1u : 0u));
  uint32_t c = 0;
#pragma unroll
  for (int k = 0; k < n; ++k) c += (uint32_t)(a > t[k]);
  return c ^ (neg ? (uint32_t)n : (uint32_t)(n + 1));
}

// ------------------------------------------------------------------------------------------------
// Keys
// ------------------------------------------------------------------------------------------------
struct Unit {
  int b, h, tok0, begin, len, first, x;
  size_t seq;
};

// Unit u (x fastest) of `tokens` tokens of the role with nx units per (sequence, KV head): stateless [0,
// lens), append from the device lengths (clamped into the buffers).
__device__ __forceinline__ Unit unit_at(const BlockArgs& a, uint32_t u, uint32_t nx, int tokens) {
  Unit c;
  const uint32_t r = u / nx, bz = r / (uint32_t)a.H;
  c.x = (int)(u - r * nx);
  c.h = (int)(r - bz * (uint32_t)a.H);
  c.b = a.b0 + (int)bz;
  c.seq = (size_t)c.b * a.H + c.h;
  c.begin = 0;
  if (a.begin_dev) {
    c.begin = min(max(a.begin_dev[c.b], 0), a.cap);
    c.len = min(c.begin + min(max(a.count_dev[c.b], 0), a.n_rows), a.cap);
  } else {
    c.len = a.lens.lens[bz];
  }
  c.first = c.begin / kW * kW;
  c.tok0 = c.first + tokens * c.x;
  return c;
}

// Metadata of one channel of a window from its minimum and maximum (thread = channel c; the 32 lanes of an
// MXFP4 block are consecutive): written to the cache, and (minimum, 1 / step) as the codes use them returned.
template <int kMeta>
__device__ __forceinline__ float2 key_metadata(const BlockArgs& a, size_t win, int c, float lo, float hi, float top,
                                               bool live) {
  const float l = lo + 0.0f, u = hi + 0.0f;  // canonical +0
  const float step = div_rn(u - l, top);
  if constexpr (kMeta == kMetaMx) return mx_metadata(a.k_mx + win * kMxRecord, c, l, step, live);
  const uint32_t m16 = f2h(l), s16 = f2h(step);
  if (live) {
    a.k_min[win * kD + c] = (uint16_t)m16;
    a.k_step[win * kD + c] = (uint16_t)s16;
  }
  return make_float2(h2f(m16), (s16 == 0) ? 0.0f : div_rn(1.0f, h2f(s16)));
}

// The quad's b-bit fields (8 channels, 8 b bits per lane and u) as dwords of the token's bit stream, stored by
// the lanes that hold one: 2 bits -- lanes 0, 2; 3 bits -- lanes 0 .. 2; 4 bits -- every lane.
template <int kBits>
__device__ __forceinline__ void store_stream(uint32_t* row, int u, int q, uint32_t f, bool ok) {
  if constexpr (kBits == 4) {
    if (ok) row[4 * u + q] = f;
  } else if constexpr (kBits == 3) {
    const uint32_t nx = quad_perm<kNext>(f);
    const uint32_t w = (f >> (8 * q)) | (nx << ((24 - 8 * q) & 31));
    if (ok && q < 3) row[3 * u + q] = w;
  } else {
    const uint32_t w = f | (quad_perm<kXor1>(f) << 16);
    if (ok && !(q & 1)) row[2 * u + (q >> 1)] = w;
  }
}

// The ladder's codes of the lane's 8 channels of group u as a bit field: method keys (st: the window's
// (minimum, 1 / step) of those channels) or TurboQuant keys (st null).
template <int kBits, int kMeta>
__device__ __forceinline__ uint32_t ladder_field(const BlockArgs& a, const float* x, const float2* st) {
  uint32_t f = 0;
  if constexpr (kMeta == kMetaTq) {
#pragma unroll
    for (int e = 0; e < 8; ++e) f |= symmetric_code<kBits>(x[e], a.ktau) << (kBits * e);
  } else {
    constexpr float top = (float)((1 << kBits) - 1);
#pragma unroll
    for (int half = 0; half < 2; ++half) {  // four codes summed exactly in fp32, then one conversion
      float s = 0.0f;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float2 m = st[4 * half + e];
        const float t = (x[4 * half + e] - m.x) * m.y;
        s = __builtin_fmaf(__builtin_rintf(__builtin_amdgcn_fmed3f(t, 0.0f, top)), (float)(1 << (kBits * e)), s);
      }
      f |= (uint32_t)s << (4 * kBits * half);
    }
  }
  return f;
}

template <int kBits, int kMeta>
__device__ __forceinline__ void ladder_key_codes(const BlockArgs& a, const Unit& c, int tok, int q, bool valid, bool slot,
                                                 const float (&x)[32], const float2* stat) {
  uint32_t* row = reinterpret_cast<uint32_t*>(a.k_codes + (c.seq * a.cap + tok) * (16 * kBits));
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    __builtin_amdgcn_sched_barrier(0);  // one group's statistics in registers at a time
    const uint32_t f = ladder_field<kBits, kMeta>(a, &x[8 * u], stat + 32 * u + 8 * q);
    store_stream<kBits>(row, u, q, valid ? f : 0u, slot);
  }
}

template <int kMeta, bool kLadder>
__device__ __forceinline__ void key_unit(const BlockArgs& a, KeyShared& sh, const Unit& c) {
  constexpr bool kTq = kMeta == kMetaTq;
  constexpr bool kStaged = !(kLadder && kTq);  // a key stage holds the open window's raw rows
  const int tid = threadIdx.x, t = tid >> 2, q = tid & 3;
  const int tok = c.tok0 + t;
  const bool valid = tok < c.len, fresh = valid && tok >= c.begin;
  // the token's row: from the stage below begin, else the new row; lanes past the length read a clamped row
  // whose codes are never used
  const uint16_t* p = a.k + (c.seq * a.n_rows + (size_t)min(max(tok - c.begin, 0), c.len - c.begin - 1)) * kD;
  if (kStaged && tok < c.begin) p = a.stage + (c.seq * kW + (tok - c.first)) * kD;
  uint32_t raw[16];
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const uint4 v = reinterpret_cast<const uint4*>(p)[4 * u + q];
    raw[4 * u] = v.x;
    raw[4 * u + 1] = v.y;
    raw[4 * u + 2] = v.z;
    raw[4 * u + 3] = v.w;
  }
  uint32_t sg[8];
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const uint2 w = *reinterpret_cast<const uint2*>(a.signs + 32 * u + 8 * q);
    sg[2 * u] = w.x;
    sg[2 * u + 1] = w.y;
  }
  float x[32];
  const uint32_t n16 = quad_direction(raw, sg, q, x);
  const int npad = (c.len + kW - 1) / kW * kW;
  const bool slot = tok < npad && (kStaged || tok >= c.begin);  // slots written: every window with a valid token
  auto store_raw = [&](uint16_t* row) {
    uint4* d = reinterpret_cast<uint4*>(row);
#pragma unroll
    for (int i = 0; i < 4; ++i) d[4 * i + q] = make_uint4(raw[4 * i], raw[4 * i + 1], raw[4 * i + 2], raw[4 * i + 3]);
  };
  if (a.k_res && fresh && tok >= c.len - kResidual)  // the residual ring: raw rows of the last 128 tokens
    store_raw(a.k_res + (c.seq * kResidual + (tok & (kResidual - 1))) * kD);
  // the open window's raw rows: slot t of the stage; a window this unit starts with keeps the rows below
  // begin, a later one's rows are read again after the barrier below
  const int open = c.len / kW * kW;
  const bool restage = kStaged && a.stage && c.x == 0 && open < c.len;  // uniform
  if (restage && open == c.first && t < kW && fresh) store_raw(a.stage + (c.seq * kW + t) * kD);
  if (q == 0 && slot) a.k_norm[c.seq * a.cap + tok] = valid ? (uint16_t)n16 : (uint16_t)0;

  if constexpr (!kTq) {
    // ---- window statistics: thread (window, channel) over the window's valid tokens ----
    const int sw = swz(t);
#pragma unroll
    for (int i = 0; i < 8; ++i)
      *reinterpret_cast<float4*>(&sh.z[t][4 * ((8 * (i >> 1) + 2 * q + (i & 1)) ^ sw)]) =
          make_float4(x[4 * i], x[4 * i + 1], x[4 * i + 2], x[4 * i + 3]);
    __syncthreads();  // (every stage read of the unit has landed, too)
    const int w = tid >> 7, ch = tid & (kD - 1);
    const int nv = min(max(c.len - (c.tok0 + kW * w), 0), kW);  // wave-uniform
    float lo[4], hi[4];  // independent chains
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      lo[i] = __builtin_inff();
      hi[i] = -__builtin_inff();
    }
    const float* zc = &sh.z[kW * w][ch & 3];
    const int c4 = ch >> 2;
    if (nv == kW) {
#pragma unroll
      for (int i = 0; i < kW; ++i) {
        if (i == kW / 2) __builtin_amdgcn_sched_barrier(0);  // half of the rows in flight at a time
        const float v = zc[i * kD + 4 * (c4 ^ swz(i))];
        lo[i & 3] = fminf(lo[i & 3], v);
        hi[i & 3] = fmaxf(hi[i & 3], v);
      }
    } else {
      for (int i = 0; i < nv; ++i) {
        const float v = zc[i * kD + 4 * (c4 ^ swz(i))];
        lo[0] = fminf(lo[0], v);
        hi[0] = fmaxf(hi[0], v);
      }
    }
    const float l = fminf(fminf(lo[0], lo[1]), fminf(lo[2], lo[3]));
    const float h = fmaxf(fmaxf(hi[0], hi[1]), fmaxf(hi[2], hi[3]));
    const bool has = nv > 0;
    const size_t win = c.seq * (a.cap / kW) + (c.tok0 / kW + w);
    const float top = kLadder ? (float)((1 << a.key_bits) - 1) : 3.0f;
    sh.stat[w][ch] = key_metadata<kMeta>(a, win, ch, has ? l : 0.0f, has ? h : 0.0f, top, has);
    __syncthreads();
  } else if (restage && open != c.first) {
    __syncthreads();  // every stage read of the unit has landed
  }
  if (restage && open != c.first && t < kW && open + t < c.len) {
    const uint4* s = reinterpret_cast<const uint4*>(a.k + (c.seq * a.n_rows + (open + t - c.begin)) * kD);
    uint4* d = reinterpret_cast<uint4*>(a.stage + (c.seq * kW + t) * kD);
#pragma unroll
    for (int i = 0; i < 4; ++i) d[4 * i + q] = s[4 * i + q];
  }
  // ---- codes ----
  const float2* stat = &sh.stat[t >> 5][0];
  if constexpr (kLadder) {
    if (a.key_bits == 2)
      ladder_key_codes<2, kMeta>(a, c, tok, q, valid, slot, x, stat);
    else if (a.key_bits == 3)
      ladder_key_codes<3, kMeta>(a, c, tok, q, valid, slot, x, stat);
    else
      ladder_key_codes<4, kMeta>(a, c, tok, q, valid, slot, x, stat);
  } else {
    // word 2 u + q / 2 of the token: channels 32 u + 16 (q / 2) .. + 15, even ones in the low half;
    // this lane fills bits 8 (q & 1) .. + 7 of both halves. t = fl(fl(z - m) fl(1 / step)) is clamped
    // and rounded to an integer (ties to even) by adding 2^23, which leaves the code in the low bits
    uint32_t* row = reinterpret_cast<uint32_t*>(a.k_codes + (c.seq * a.cap + tok) * 32);
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      __builtin_amdgcn_sched_barrier(0);  // one group's statistics in registers at a time
      uint32_t lo = 0, hi = 0;
#pragma unroll
      for (int d = 0; d < 4; ++d) {
        const float z0 = x[8 * u + 2 * d], z1 = x[8 * u + 2 * d + 1];
        uint32_t c0, c1;
        if constexpr (kTq) {
          c0 = (uint32_t)(z0 > a.th.t0) + (uint32_t)(z0 > a.th.t1) + (uint32_t)(z0 > a.th.t2);
          c1 = (uint32_t)(z1 > a.th.t0) + (uint32_t)(z1 > a.th.t1) + (uint32_t)(z1 > a.th.t2);
        } else {
          const float4 s = *reinterpret_cast<const float4*>(&stat[32 * u + 8 * q + 2 * d]);
          constexpr float kRound = 8388608.0f;  // 2^23
          c0 = __builtin_bit_cast(uint32_t, __builtin_amdgcn_fmed3f((z0 - s.x) * s.y, 0.0f, 3.0f) + kRound);
          c1 = __builtin_bit_cast(uint32_t, __builtin_amdgcn_fmed3f((z1 - s.z) * s.w, 0.0f, 3.0f) + kRound);
        }
        lo |= c0 << (2 * d);
        hi |= c1 << (2 * d);
      }
      uint32_t w = __builtin_amdgcn_perm(hi, lo, 0x0c040c00u) << (8 * (q & 1));  // low bytes of lo and hi
      w |= quad_perm<kXor1>(w);
      if (slot && !(q & 1)) row[2 * u + (q >> 1)] = valid ? w : 0u;
    }
  }
}

// ------------------------------------------------------------------------------------------------
// Values
// ------------------------------------------------------------------------------------------------
// The wave's slice of R_m as MFMA operands: bf[i][kk][part] for output block kNb v + i, k-block kk, part 0 =
// fp16(R) and 1 = fp16(R - fp16(R)); from the prepared fragments, or converted from the fp32 matrix.
template <int kNb>
__device__ __forceinline__ void load_rot_slice(const BlockArgs& a, int m, int v, int lane, uint4 (&bf)[kNb][4][2]) {
  if (kNb > 1 && a.rotfrag) {  // (one block a wave: only without fragments)
    const char* base = reinterpret_cast<const char*>(a.rotfrag) + (size_t)(m * 8 + kNb * v) * 8 * 1024;
    const uint32_t off = 16u * (uint32_t)lane;
#pragma unroll
    for (int i = 0; i < kNb; ++i)
#pragma unroll
      for (int kk = 0; kk < 4; ++kk)
#pragma unroll
        for (int part = 0; part < 2; ++part)
          bf[i][kk][part] = *reinterpret_cast<const uint4*>(base + ((i * 4 + kk) * 2 + part) * 1024 + off);
    return;
  }
  const int r = lane & 15, g = lane >> 4;
#pragma unroll
  for (int i = 0; i < kNb; ++i)
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
      const float4* p = reinterpret_cast<const float4*>(a.rot + ((size_t)(m * kD + 16 * (kNb * v + i) + r)) * kD + 32 * kk + 8 * g);
      const float4 f0 = p[0], f1 = p[1];
      const float fv[8] = {f0.x, f0.y, f0.z, f0.w, f1.x, f1.y, f1.z, f1.w};
      half8 hv, lv;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        hv[e] = (_Float16)fv[e];
        lv[e] = (_Float16)(fv[e] - (float)hv[e]);
      }
      bf[i][kk][0] = __builtin_bit_cast(uint4, hv);
      bf[i][kk][1] = __builtin_bit_cast(uint4, lv);
    }
}

__device__ __forceinline__ int floor_i32(float x) {  // one instruction (v_cvt_flr_i32_f32)
  int r;
  __asm__("v_cvt_flr_i32_f32 %0, %1" : "=v"(r) : "v"(x));
  return r;
}

// VALU row swaps (lanes 32-63 of a with lanes 0-31 of b; odd 16-lane rows of a with even rows of b). From
// inline assembly: the compiler takes the builtin's two results for the same value where they are added.
// s_nop: the wait states between a VALU write and the swap.
__device__ __forceinline__ void swap_halves(float (&a)[8], float (&b)[8]) {
#pragma unroll
  for (int i = 0; i < 8; i += 4)
    __asm__("s_nop 1\n\t"
            "v_permlane32_swap_b32 %0, %4\n\t"
            "v_permlane32_swap_b32 %1, %5\n\t"
            "v_permlane32_swap_b32 %2, %6\n\t"
            "v_permlane32_swap_b32 %3, %7\n\t"
            "s_nop 1"
            : "+v"(a[i]), "+v"(a[i + 1]), "+v"(a[i + 2]), "+v"(a[i + 3]), "+v"(b[i]), "+v"(b[i + 1]), "+v"(b[i + 2]),
              "+v"(b[i + 3]));
}
__device__ __forceinline__ void swap_rows(float (&a)[8], float (&b)[8]) {
#pragma unroll
  for (int i = 0; i < 8; i += 4)
    __asm__("s_nop 1\n\t"
            "v_permlane16_swap_b32 %0, %4\n\t"
            "v_permlane16_swap_b32 %1, %5\n\t"
            "v_permlane16_swap_b32 %2, %6\n\t"
            "v_permlane16_swap_b32 %3, %7\n\t"
            "s_nop 1"
            : "+v"(a[i]), "+v"(a[i + 1]), "+v"(a[i + 2]), "+v"(a[i + 3]), "+v"(b[i]), "+v"(b[i + 1]), "+v"(b[i + 2]),
              "+v"(b[i + 3]));
}
// the value of lane l ^ 16 (l ^ 32)
__device__ __forceinline__ uint32_t xor16(uint32_t v, int g) {
  uint32_t a = v, b = v;
  __asm__("s_nop 1\n\tv_permlane16_swap_b32 %0, %1\n\ts_nop 1" : "+v"(a), "+v"(b));
  return (g & 1) ? a : b;
}
__device__ __forceinline__ uint32_t xor32(uint32_t v, int g) {
  uint32_t a = v, b = v;
  __asm__("s_nop 1\n\tv_permlane32_swap_b32 %0, %1\n\ts_nop 1" : "+v"(a), "+v"(b));
  return (g & 2) ? a : b;
}

// Sum of squares of the rows of two row blocks in LDS (lane l: row l % 16 of block l / 32) by the halving tree: levels
// 64 and 32 in the lane, 16 and 8 across lane groups (the first by a row swap that leaves block 0 in lanes 0-31
// and block 1 in lanes 32-63)
__device__ __forceinline__ float row_squares(const uint4 (&rows0)[4][64], const uint4 (&rows1)[4][64], int lane) {
  float p[2][8];
#pragma unroll
  for (int rb = 0; rb < 2; ++rb) {
    half8 xv[4];
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) xv[kk] = as_half8((rb ? rows1 : rows0)[kk][lane]);
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      // squares of fp16 values are exact; as fma (mixed precision) they need no conversion of their own
      const float f0 = (float)xv[0][e], f1 = (float)xv[1][e], f2 = (float)xv[2][e], f3 = (float)xv[3][e];
      const float l0 = __builtin_fmaf(f0, f0, __builtin_fmaf(f2, f2, 0.0f));
      const float l1 = __builtin_fmaf(f1, f1, __builtin_fmaf(f3, f3, 0.0f));
      p[rb][e] = l0 + l1;
    }
  }
  float s[8], z[8];
  swap_halves(p[0], p[1]);
#pragma unroll
  for (int e = 0; e < 8; ++e) z[e] = s[e] = p[0][e] + p[1][e];
  swap_rows(s, z);
#pragma unroll
  for (int e = 0; e < 8; ++e) s[e] = s[e] + z[e];
#pragma unroll
  for (int n = 4; n >= 1; n >>= 1) {
#pragma unroll
    for (int e = 0; e < n; ++e) s[e] = s[e] + s[e + n];
  }
  return s[0];
}

// Codes of the lane's four channels 16 nb + 4 g .. + 3 of its token as a 4 b-bit field
template <int kBits>
__device__ __forceinline__ uint32_t value_field(floatx4 y, const float (&t)[7]) {
  uint32_t f = 0;
#pragma unroll
  for (int i = 0; i < 4; ++i) f |= symmetric_code<kBits>(y[i], t) << (kBits * i);
  return f;
}

// Ladder codes of a row block: p0, p1 = the fields of output blocks 2 v and 2 v + 1 (channels 32 v + 4 g ..
// and 32 v + 16 + 4 g ..), put together across the token's four lane groups into the b dwords of channels
// 32 v .. 32 v + 31 of its bit stream.
template <int kBits>
__device__ __forceinline__ void store_value_stream(uint32_t* dst, int lane, uint32_t p0, uint32_t p1, bool ok) {
  const int g = lane >> 4;
  // lane groups 0, 2 join the first block's fields of groups g, g + 1; groups 1, 3 the second block's
  const uint32_t got = xor16((g & 1) ? p0 : p1, g);
  const uint32_t w = (g & 1) ? (got | (p1 << (4 * kBits))) : (p0 | (got << (4 * kBits)));
  // bits 8 b s .. + 8 b - 1 of the run, s = 0, 2, 1, 3 for g = 0 .. 3
  if constexpr (kBits == 4) {
    if (ok) dst[2 * (g & 1) + (g >> 1)] = w;
  } else if constexpr (kBits == 2) {
    const uint32_t up = xor32(w, g);
    if (ok && g < 2) dst[g] = w | (up << 16);
  } else {
    const int s = 2 * (g & 1) + (g >> 1);  // dword s takes the fields s and s + 1
    const int next = (lane & 15) + 16 * (g == 0 ? 2 : g == 2 ? 1 : 3);
    const uint32_t nx = (uint32_t)__shfl((int)w, next);
    if (ok && s < 3) dst[s] = (w >> (8 * s)) | (nx << (24 - 8 * s));
  }
}

template <int kBits, int kRb>
__device__ __forceinline__ void ladder_values(const BlockArgs& a, const Unit& c, ValueShared& sv, int v, int lane, int m,
                                              uint32_t rbs, const uint4 (&bf)[2][4][2], uint32_t (&p)[8]) {
  constexpr int n = (1 << (kBits - 1)) - 1;
#pragma unroll
  for (int rb = 0; rb < kRb; ++rb) {
    if (!((rbs >> rb) & 1u)) continue;  // uniform
    floatx4 y0 = {0.f, 0.f, 0.f, 0.f}, y1 = y0;
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
      const half8 x = as_half8(sv.rows[rb][kk][lane]);
#pragma unroll
      for (int part = 0; part < 2; ++part) {
        y0 = __builtin_amdgcn_mfma_f32_16x16x32_f16(as_half8(bf[0][kk][part]), x, y0, 0, 0, 0);
        y1 = __builtin_amdgcn_mfma_f32_16x16x32_f16(as_half8(bf[1][kk][part]), x, y1, 0, 0, 0);
      }
    }
    const float nv = sv.nrm[16 * rb + (lane & 15)];
    float t[7];
#pragma unroll
    for (int k = 0; k < 7; ++k) t[k] = k < n ? nv * a.vtau[k] : 0.0f;
    const bool mine = sv.tmod[rb][lane & 15] == (uint32_t)m;
    p[rb] = mine ? value_field<kBits>(y0, t) | (value_field<kBits>(y1, t) << 16) : p[rb];
  }
}

template <int kBits, int kRb>
__device__ __forceinline__ void ladder_store(const BlockArgs& a, const Unit& c, int v, int lane, const uint32_t (&p)[8]) {
#pragma unroll
  for (int rb = 0; rb < kRb; ++rb) {
    const int tok = c.tok0 + 16 * rb + (lane & 15);
    if (c.tok0 + 16 * rb >= c.len) break;  // uniform
    store_value_stream<kBits>(reinterpret_cast<uint32_t*>(a.v_codes + (c.seq * a.cap + tok) * (16 * kBits)) + kBits * v, lane,
                              p[rb] & 0xffffu, p[rb] >> 16, tok >= c.begin && tok < c.len);
  }
}

// kUnit: 128 tokens, or 64 (half the serial chain, twice the reads of R_m). The first kUnit / 32 waves load 32
// rows each and form their norms.
template <bool kLadder, int kUnit>
__device__ __forceinline__ void value_unit(const BlockArgs& a, ValueShared& sv, const Unit& c) {
  constexpr int kRb = kUnit / 16, kRowWaves = kUnit / 32;
  const int tid = threadIdx.x, lane = tid & 63, r = lane & 15, g = lane >> 4;
  const int v = __builtin_amdgcn_readfirstlane(tid >> 6);
  const uint32_t lds = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(uintptr_t)&sv.rows[2 * v][0][0]);
  const int wtok0 = c.tok0 + 32 * v;
  const bool rows = v < kRowWaves;  // wave-uniform
  if (rows) {
#pragma unroll
    for (int rb = 0; rb < 2; ++rb) {  // rows outside the new tokens repeat the nearest one (never coded)
      const int row = min(max(wtok0 + 16 * rb + r - c.begin, 0), c.len - c.begin - 1);
      const uint4* p = reinterpret_cast<const uint4*>(a.v + (c.seq * a.n_rows + row) * kD) + g;
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) dma16(p + 4 * kk, lds + (rb * 4 + kk) * 1024);
    }
  }
  // lane l: token 16 (l / 32) + l % 16 of the wave's 32
  const int mytok = wtok0 + 16 * (lane >> 5) + r;
  const bool fresh = mytok >= c.begin && mytok < c.len;
  const uint32_t mymod = a.modality[(size_t)c.b * a.n_rows + min(max(mytok - c.begin, 0), c.len - c.begin - 1)];
  // the first modality's slice (video, the most frequent; R_0 with the global rotation), in flight with the rows
  const int first_m = a.global_rot ? 0 : 1;
  uint4 bf[2][4][2];
  load_rot_slice(a, first_m, v, lane, bf);
  if (rows) {
    __asm__ volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the wave's rows have landed

    const float sq = row_squares(sv.rows[2 * v], sv.rows[2 * v + 1], lane);
    const uint32_t n16 = fresh ? norm_to_f16(sqrt_rn(sq)) : 0u;
    // 3: no code; with the global rotation every coded token takes R_0. (The ladder codes a zero row too:
    // its code is that of y = 0 against zero thresholds.)
    const uint32_t mt = (fresh && mymod <= 2u && (kLadder || n16 != 0)) ? (a.global_rot ? 0u : mymod) : 3u;
    const int wt = 32 * v + 16 * (lane >> 5) + r;  // token of the unit
    if ((g & 1) == 0) {
      sv.nrm[wt] = kLadder ? h2f(n16) : (n16 != 0) ? __builtin_amdgcn_rcpf(h2f(n16) * a.th.t2) : 0.0f;
      if constexpr (kLadder) sv.tmod[2 * v + (lane >> 5)][r] = mt;
      const int wend = kLadder ? c.len : (c.len + kW - 1) / kW * kW;
      if (mytok >= c.begin && mytok < wend) a.v_norm[c.seq * a.cap + mytok] = (uint16_t)n16;
      if (fresh && a.mod_out && c.h == 0) a.mod_out[(size_t)c.b * a.cap + mytok] = (uint8_t)mymod;
      if (a.v_res && fresh && mytok >= c.len - kResidual) {  // the residual ring: raw rows of the last 128 tokens
        uint4* d = reinterpret_cast<uint4*>(a.v_res + (c.seq * kResidual + (mytok & (kResidual - 1))) * kD);
#pragma unroll
        for (int kk = 0; kk < 4; ++kk)
#pragma unroll
          for (int gg = 0; gg < 4; ++gg) d[4 * kk + gg] = sv.rows[2 * v + (lane >> 5)][kk][16 * gg + r];
      }
    }
    uint32_t pres = 0;
#pragma unroll
    for (int m = 0; m < 3; ++m) {
      const uint64_t mb = __ballot(mt == (uint32_t)m);
      if (mb & 0xffffull) pres |= 1u << (8 * m + 2 * v);
      if (mb >> 32) pres |= 2u << (8 * m + 2 * v);
      if constexpr (!kLadder) {
        if (lane < 8) {  // quad `lane` of the wave: its tokens' bits -> bits 2 i, 2 i + 1
          const uint32_t b4 = (uint32_t)(mb >> (32 * (lane >> 2) + 4 * (lane & 3))) & 15u;
          const uint32_t spread = (b4 & 1u) | ((b4 & 2u) << 1) | ((b4 & 4u) << 2) | ((b4 & 8u) << 3);
          sv.ktab[m][8 * v + lane] = (uint8_t)(spread * 3u);
        }
      }
    }
    if (lane == 0) sv.present[v] = pres;
  } else if (lane == 0) {
    sv.present[v] = 0u;
  }
  __syncthreads();  // rows and tables complete

  const uint4 pw = *reinterpret_cast<const uint4*>(&sv.present[0]);
  const uint32_t present = __builtin_amdgcn_readfirstlane(pw.x | pw.y | pw.z | pw.w);
  uint32_t vb[4] = {0u, 0u, 0u, 0u};  // 2-bit layout: window w, bits 0-15 row block 2 w, 16-31 row block 2 w + 1
  uint32_t pk[8];                     // ladder: the row blocks' fields, the second output block's 16 bits up
  if constexpr (kLadder) {
#pragma unroll
    for (int i = 0; i < 8; ++i) pk[i] = 0u;
  }
#pragma unroll 1
  for (int mi = 0, m = first_m; mi < 3; ++mi, m = (m == 2) ? 0 : m + 1) {
    const uint32_t rbs = (present >> (8 * m)) & 0xffu;
    if (rbs == 0) continue;
    if (m != first_m) load_rot_slice(a, m, v, lane, bf);
    if constexpr (kLadder) {
      if (a.value_bits == 2)
        ladder_values<2, kRb>(a, c, sv, v, lane, m, rbs, bf, pk);
      else if (a.value_bits == 3)
        ladder_values<3, kRb>(a, c, sv, v, lane, m, rbs, bf, pk);
      else
        ladder_values<4, kRb>(a, c, sv, v, lane, m, rbs, bf, pk);
    } else {
#pragma unroll
      for (int w = 0; w < kRb / 2; ++w) {
        if (!((rbs >> (2 * w)) & 3u)) continue;  // uniform
        floatx4 y[2][2];
#pragma unroll
        for (int i = 0; i < 2; ++i) y[i][0] = y[i][1] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) {
          const half8 x0 = as_half8(sv.rows[2 * w][kk][lane]), x1 = as_half8(sv.rows[2 * w + 1][kk][lane]);
#pragma unroll
          for (int part = 0; part < 2; ++part) {
            y[0][0] = __builtin_amdgcn_mfma_f32_16x16x32_f16(x0, as_half8(bf[0][kk][part]), y[0][0], 0, 0, 0);
            y[0][1] = __builtin_amdgcn_mfma_f32_16x16x32_f16(x0, as_half8(bf[1][kk][part]), y[0][1], 0, 0, 0);
            y[1][0] = __builtin_amdgcn_mfma_f32_16x16x32_f16(x1, as_half8(bf[0][kk][part]), y[1][0], 0, 0, 0);
            y[1][1] = __builtin_amdgcn_mfma_f32_16x16x32_f16(x1, as_half8(bf[1][kk][part]), y[1][1], 0, 0, 0);
          }
        }
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          // code = clamp(floor(y / T) + 2, 0, 3) with y / T taken as y fl(1 / T) (the tile codec's decision)
          const float4 it = *reinterpret_cast<const float4*>(&sv.nrm[16 * (2 * w + i) + 4 * g]);
          const float iv[4] = {it.x, it.y, it.z, it.w};
          uint32_t s0 = 0, s1 = 0;
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            s0 += (uint32_t)min(max(floor_i32(y[i][0][k] * iv[k]), -2), 1) << (2 * k);
            s1 += (uint32_t)min(max(floor_i32(y[i][1][k] * iv[k]), -2), 1) << (2 * k);
          }
          const uint32_t bytes = ((s0 + 0xAAu) & 0xFFu) | (((s1 + 0xAAu) & 0xFFu) << 8);  // + 2 per token
          vb[w] |= (bytes & ((uint32_t)sv.ktab[m][4 * (2 * w + i) + g] * 0x0101u)) << (16 * i);
        }
      }
    }
  }
  if constexpr (kLadder) {
    if (a.value_bits == 2)
      ladder_store<2, kRb>(a, c, v, lane, pk);
    else if (a.value_bits == 3)
      ladder_store<3, kRb>(a, c, v, lane, pk);
    else
      ladder_store<4, kRb>(a, c, v, lane, pk);
  } else {
    const int ncw = a.cap / kW;
#pragma unroll
    for (int w = 0; w < kRb / 2; ++w) {
      const int ws = c.tok0 + kW * w;
      if (ws >= c.len) break;
      uint16_t* dst = reinterpret_cast<uint16_t*>(a.v_codes + (c.seq * ncw + ws / kW) * 1024 + 16 * lane + 2 * v);
      uint32_t w0 = vb[w] & 0xffffu, w1 = vb[w] >> 16;
      if (ws < c.begin) {  // the window holds older tokens: keep their code bits
        const int old0 = min(max(c.begin - (ws + 4 * g), 0), 4);       // tokens 4g .. 4g+3
        const int old1 = min(max(c.begin - (ws + 16 + 4 * g), 0), 4);  // tokens 16+4g ..
        const uint32_t k0 = ((1u << (2 * old0)) - 1u) * 0x0101u;
        const uint32_t k1 = ((1u << (2 * old1)) - 1u) * 0x0101u;
        w0 = ((uint32_t)dst[0] & k0) | (w0 & ~k0);
        w1 = ((uint32_t)dst[4] & k1) | (w1 & ~k1);
      }
      dst[0] = (uint16_t)w0;
      dst[4] = (uint16_t)w1;
    }
  }
}

// ------------------------------------------------------------------------------------------------
// Stateless 2-bit values from the fp32 matrix: units of 256 tokens on eight waves, one output block of 16 channels
// each, so that every slice of R_m is converted once for 256 tokens, at the same four waves per SIMD. A lane's code
// bytes (one per window and row block) meet in LDS, where the rows were, and leave 16 bytes a lane. Bound by the
// conversion (8.4 of 25.5 us in units of 128 tokens, where prepared fragments would take 17.1) and the matrix
// products: 32768 tokens of 4 heads 25.5 -> 20.6 us, 131072 tokens 82.7 -> 66.7.
constexpr int kWideUnit = 256, kWideWaves = 8;
struct WideShared {
  uint4 rows[kWideUnit / 16][4][64];
  float nrm[kWideUnit];
  uint8_t ktab[3][kWideUnit / 4];
  uint32_t present[3][kWideWaves];
};

__global__ __launch_bounds__(64 * kWideWaves, 4) void k_values_wide(BlockArgs a) {
  __shared__ __attribute__((aligned(16))) WideShared sv;
  const Unit c = unit_at(a, blockIdx.x, a.val_nx, kWideUnit);
  if (c.tok0 >= c.len) return;  // uniform
  const int tid = threadIdx.x, lane = tid & 63, r = lane & 15, g = lane >> 4;
  const int v = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wtok0 = c.tok0 + 32 * v;
  const uint32_t lds = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(uintptr_t)&sv.rows[2 * v][0][0]);
#pragma unroll
  for (int rb = 0; rb < 2; ++rb) {  // rows past the end repeat the last one (never coded)
    const uint4* p = reinterpret_cast<const uint4*>(a.v + (c.seq * a.n_rows + min(wtok0 + 16 * rb + r, c.len - 1)) * kD) + g;
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) dma16(p + 4 * kk, lds + (rb * 4 + kk) * 1024);
  }
  const int mytok = wtok0 + 16 * (lane >> 5) + r;  // lane l: token 16 (l / 32) + l % 16 of the wave's 32
  const bool fresh = mytok < c.len;
  const uint32_t mymod = a.modality[(size_t)c.b * a.n_rows + min(mytok, c.len - 1)];
  const int first_m = a.global_rot ? 0 : 1;
  uint4 bf[1][4][2];
  load_rot_slice(a, first_m, v, lane, bf);
  __asm__ volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the wave's rows have landed
  const float sq = row_squares(sv.rows[2 * v], sv.rows[2 * v + 1], lane);
  const uint32_t n16 = fresh ? norm_to_f16(sqrt_rn(sq)) : 0u;
  const uint32_t mt = (fresh && mymod <= 2u && n16 != 0) ? (a.global_rot ? 0u : mymod) : 3u;
  if ((g & 1) == 0) {
    sv.nrm[32 * v + 16 * (lane >> 5) + r] = (n16 != 0) ? __builtin_amdgcn_rcpf(h2f(n16) * a.th.t2) : 0.0f;
    if (mytok < (c.len + kW - 1) / kW * kW) a.v_norm[c.seq * a.cap + mytok] = (uint16_t)n16;
  }
#pragma unroll
  for (int m = 0; m < 3; ++m) {
    const uint64_t mb = __ballot(mt == (uint32_t)m);
    if (lane < 8) {  // quad `lane` of the wave: its tokens' bits -> bits 2 i, 2 i + 1
      const uint32_t b4 = (uint32_t)(mb >> (32 * (lane >> 2) + 4 * (lane & 3))) & 15u;
      const uint32_t spread = (b4 & 1u) | ((b4 & 2u) << 1) | ((b4 & 4u) << 2) | ((b4 & 8u) << 3);
      sv.ktab[m][8 * v + lane] = (uint8_t)(spread * 3u);
    }
    if (lane == 0) sv.present[m][v] = ((mb & 0xffffull) ? 1u << (2 * v) : 0u) | ((mb >> 32) ? 2u << (2 * v) : 0u);
  }
  __syncthreads();  // rows and tables complete
  uint32_t vb[kWideUnit / 64] = {0u, 0u, 0u, 0u};  // byte i of word q: row block 4 q + i
#pragma unroll 1
  for (int mi = 0, m = first_m; mi < 3; ++mi, m = (m == 2) ? 0 : m + 1) {
    const uint4 p0 = *reinterpret_cast<const uint4*>(&sv.present[m][0]), p1 = *reinterpret_cast<const uint4*>(&sv.present[m][4]);
    const uint32_t rbs = __builtin_amdgcn_readfirstlane(p0.x | p0.y | p0.z | p0.w | p1.x | p1.y | p1.z | p1.w);
    if (rbs == 0) continue;
    if (m != first_m) load_rot_slice(a, m, v, lane, bf);
#pragma unroll
    for (int w = 0; w < kWideUnit / kW; ++w) {
      if (!((rbs >> (2 * w)) & 3u)) continue;  // uniform
      floatx4 y[2] = {floatx4{0.f, 0.f, 0.f, 0.f}, floatx4{0.f, 0.f, 0.f, 0.f}};
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) {
        const half8 x0 = as_half8(sv.rows[2 * w][kk][lane]), x1 = as_half8(sv.rows[2 * w + 1][kk][lane]);
#pragma unroll
        for (int part = 0; part < 2; ++part) {
          y[0] = __builtin_amdgcn_mfma_f32_16x16x32_f16(x0, as_half8(bf[0][kk][part]), y[0], 0, 0, 0);
          y[1] = __builtin_amdgcn_mfma_f32_16x16x32_f16(x1, as_half8(bf[0][kk][part]), y[1], 0, 0, 0);
        }
      }
#pragma unroll
      for (int i = 0; i < 2; ++i) {  // the same decision as above
        const float4 it = *reinterpret_cast<const float4*>(&sv.nrm[16 * (2 * w + i) + 4 * g]);
        const float iv[4] = {it.x, it.y, it.z, it.w};
        uint32_t s0 = 0;
#pragma unroll
        for (int k = 0; k < 4; ++k) s0 += (uint32_t)min(max(floor_i32(y[i][k] * iv[k]), -2), 1) << (2 * k);
        vb[w / 2] |= ((s0 + 0xAAu) & (uint32_t)sv.ktab[m][4 * (2 * w + i) + g]) << (8 * (2 * (w & 1) + i));
      }
    }
  }
  __syncthreads();  // every wave is done with the rows
  uint8_t* tile = reinterpret_cast<uint8_t*>(&sv.rows[0][0][0]);  // the unit's code bytes: [window][1024]
#pragma unroll
  for (int rb = 0; rb < kWideUnit / 16; ++rb)
    tile[1024 * (rb >> 1) + 16 * lane + 8 * (rb & 1) + v] = (uint8_t)(vb[rb >> 2] >> (8 * (rb & 3)));
  __syncthreads();
  if (wtok0 < c.len)  // wave v: window v
    *reinterpret_cast<uint4*>(a.v_codes + (c.seq * (a.cap / kW) + wtok0 / kW) * 1024 + 16 * lane) =
        *reinterpret_cast<const uint4*>(tile + 1024 * v + 16 * lane);
}

// ------------------------------------------------------------------------------------------------
// Work-groups n < 2 paired alternate between the roles in runs of kRun; the rest of the key units (half as
// long as the value units: they fill the end) and then the rest of the value units follow.
template <int kMeta, bool kLadder, int kUnit>
__global__ __launch_bounds__(kThreads, 4) void k_codec_block(BlockArgs a) {
  __shared__ __attribute__((aligned(16))) BlockShared sh;
  const uint32_t n = blockIdx.x, paired = a.paired, key_units = a.key_units;
  bool key;
  uint32_t u;
  if (n < 2 * paired) {
    key = ((n / kRun) & 1) == 0;
    u = n / (2 * kRun) * kRun + n % kRun;
  } else {
    key = n < paired + key_units;
    u = key ? n - paired : n - key_units;
  }
  const Unit c = unit_at(a, u, key ? a.key_nx : a.val_nx, key ? kKeyUnit : kUnit);
  if (c.len <= c.begin || c.tok0 >= c.len) return;  // uniform
  if (key)
    key_unit<kMeta, kLadder>(a, sh.k, c);
  else
    value_unit<kLadder, kUnit>(a, sh.v, c);
}

template <int kUnit>
auto pick(int key_meta, bool ladder) -> void (*)(BlockArgs) {
  if (ladder) return key_meta == kMetaTq ? k_codec_block<kMetaTq, true, kUnit> : k_codec_block<kMetaFp16, true, kUnit>;
  return key_meta == kMetaMx   ? k_codec_block<kMetaMx, false, kUnit>
         : key_meta == kMetaTq ? k_codec_block<kMetaTq, false, kUnit>
                               : k_codec_block<kMetaFp16, false, kUnit>;
}

}  // namespace

// A launch holds fewer than 2^32 threads: beyond, the sequences in two halves (the events around both)
static hipError_t launch_halves(const BlockArgs& args, int key_meta, bool keys, bool values, int span, hipStream_t s,
                                hipEvent_t const* events) {
  if (args.nb < 2) return hipErrorInvalidValue;
  hipEvent_t ev[2][2] = {{events ? events[0] : nullptr, nullptr}, {nullptr, events ? events[1] : nullptr}};
  BlockArgs a = args;
  a.nb = args.nb / 2;
  const hipError_t e = launch_codec_block(a, key_meta, keys, values, span, s, events ? ev[0] : nullptr);
  if (e != hipSuccess) return e;
  a.b0 = args.b0 + args.nb / 2;
  a.nb = args.nb - args.nb / 2;
  for (int i = 0; i < a.nb; ++i) a.lens.lens[i] = args.lens.lens[args.nb / 2 + i];
  return launch_codec_block(a, key_meta, keys, values, span, s, events ? ev[1] : nullptr);
}

hipError_t launch_codec_block(const BlockArgs& args, int key_meta, bool keys, bool values, int span, hipStream_t s,
                              hipEvent_t const* events) {
  if (args.nb <= 0 || span <= 0 || (!keys && !values)) return hipSuccess;
  BlockArgs a = args;
  const int64_t per = (int64_t)a.H * a.nb;
  // Stateless 2-bit values: wide units from 129 on. Up to 128 the 64-token units are at most two per compute unit,
  // one round, and have the shorter chain (4 heads: 2048 tokens 9.1 us against 12.5, 8192 tokens 12.5 against 12.9);
  // beyond, every round of theirs converts R_m again (9216 tokens 16.2 against 13.0, 65536 tokens 46.3 against 35.7).
  const int64_t wide = per * ((span + kWideUnit - 1) / kWideUnit);
  if (!keys && a.key_bits == 0 && !a.rotfrag && wide > 128) {
    if (wide * 64 * kWideWaves > UINT32_MAX) return launch_halves(args, key_meta, keys, values, span, s, events);
    a.val_nx = (span + kWideUnit - 1) / kWideUnit;
    hipLaunchKernelGGL(k_values_wide, dim3((uint32_t)wide), dim3(64 * kWideWaves), 0, s, a);
    return hipGetLastError();
  }
  a.key_nx = std::max((span + kKeyUnit - 1) / kKeyUnit, 1);
  // Half-size value units where whole ones would leave compute units with fewer than two: a unit's serial
  // chain is what such a launch takes (four 512-token chunks of 8 sequence heads, with their decode steps:
  // 127.5 -> 121.2 us), while a full chip pays for the second read of R_m (32768 tokens, 4 heads: 29.9 against
  // 32.4 us).
  const bool half_units = per * ((span + kValUnit - 1) / kValUnit) < 512;
  const int val_unit = half_units ? kValUnit / 2 : kValUnit;
  a.val_nx = std::max((span + val_unit - 1) / val_unit, 1);
  const int64_t ku = keys ? per * a.key_nx : 0, vu = values ? per * a.val_nx : 0;
  if ((ku + vu) * kThreads > UINT32_MAX) return launch_halves(args, key_meta, keys, values, span, s, events);
  a.key_units = (uint32_t)ku;
  a.paired = (uint32_t)(std::min(ku, vu) / kRun * kRun);
  const bool ladder = a.key_bits != 0;
  void (*fn)(BlockArgs) = half_units ? pick<kValUnit / 2>(key_meta, ladder) : pick<kValUnit>(key_meta, ladder);
  const dim3 grid((uint32_t)(ku + vu));
  if (events)
    hipExtLaunchKernelGGL(fn, grid, dim3(kThreads), 0, s, events[0], events[1], 0, a);
  else
    hipLaunchKernelGGL(fn, grid, dim3(kThreads), 0, s, a);
  return hipGetLastError();
}

}  // namespace okvq
