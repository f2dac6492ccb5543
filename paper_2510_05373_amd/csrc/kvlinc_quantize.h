// Device functions of the append path that work on rows and on one group of 128 tokens: the Hadamard rotation of new
// values, Eq. 1 at 2 or 4 bits, and the packing of a group record (Sec. 3.1, Obs. 3; Sec. 2, Eq. 1).  Included by the
// append kernels only; compiled with floating-point contraction off (one binary32 rounding per written operation: the
// rotation and the quantizer are bit-exact contracts).
//
// Work is laid out for registers: a row of 128 channels sits in 4 lanes (rotation, value quantizer) or 16 lanes (key
// quantizer), minima and maxima run on binary16 pairs, and a 2-bit code is the number of binary16 thresholds an element
// lies above, so that two elements take one packed subtraction per threshold and no conversion.
#pragma once

#include <hip/hip_runtime.h>

#include "kvlinc_internal.h"
#include "kvlinc_mfma.h"

#pragma clang fp contract(off)

namespace kvlinc {
namespace {

typedef _Float16 half8_t __attribute__((ext_vector_type(8)));

constexpr int kRowH = 136;         // halfs per LDS row of a 128-wide fp16 tile (rows stay 16-byte aligned)
constexpr int kPlaneWords = 1024;  // a 128 x 128 tile of 2-bit codes; 4-bit codes take two such planes per tile

__device__ __forceinline__ bool nonfinite_pair(uint32_t w) { return ((w & 0x7C00u) == 0x7C00u) || ((w & 0x7C000000u) == 0x7C000000u); }

// Barrier for data exchanged through LDS: unlike __syncthreads it leaves global loads in flight.
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

__device__ __forceinline__ half2_t h2_min(half2_t a, half2_t b) { return __builtin_elementwise_minimum(a, b); }  // (NaN propagates)
__device__ __forceinline__ half2_t h2_max(half2_t a, half2_t b) { return __builtin_elementwise_maximum(a, b); }
template <int CTRL>
__device__ __forceinline__ half2_t dpp_h2(half2_t v) { return as_h2(dpp_u<CTRL>(as_u32(v))); }

// ---- a row in four lanes ------------------------------------------------------------------------------------------
// The 64 lanes of a wave hold 16 rows.  Lane = q0 ^ 2 q1 ^ 7 b ^ 8 ip inside its 16 lanes (exclusive-or of the masks whose
// lane exchanges are single DPP moves: 1 and 2 inside a quad, 7 the mirror of eight lanes, 8 a rotation by half a row):
// q = 2 q1 + q0 is the lane's place in its row -- channels 32 m + 8 q + e, m = 0..3, e = 0..7 -- and (rho, ip, b) name one of
// the 16 rows, rho = lane / 16.
struct RowLane {
  int q, b, ip, rho;
};
__device__ __forceinline__ RowLane row_lane(int lane) {
  RowLane r;
  r.b = (lane >> 2) & 1;
  r.ip = (lane >> 3) & 1;
  r.q = (lane & 3) ^ (r.b ? 3 : 0);
  r.rho = lane >> 4;
  return r;
}
struct Row {
  uint4 p[4];  // piece m: channels 32 m + 8 q .. + 7
};
__device__ __forceinline__ void load_row(Row& r, const half_t* __restrict__ row, int q) {
#pragma unroll
  for (int m = 0; m < 4; ++m) r.p[m] = *reinterpret_cast<const uint4*>(row + 32 * m + 8 * q);
}
__device__ __forceinline__ void row_pairs(const Row& r, half2_t (&h)[16]) {  // h[4 m + i]: channels 32 m + 8 q + 2 i, + 1
#pragma unroll
  for (int m = 0; m < 4; ++m) {
    h[4 * m] = as_h2(r.p[m].x); h[4 * m + 1] = as_h2(r.p[m].y);
    h[4 * m + 2] = as_h2(r.p[m].z); h[4 * m + 3] = as_h2(r.p[m].w);
  }
}

// Sum and difference of the two binary16 numbers of a register in binary32, one instruction each.
__device__ __forceinline__ float pair_sum(half2_t h) {
  float r;
  asm("v_fma_mix_f32 %0, %1, 1.0, %1 op_sel:[0,0,1] op_sel_hi:[1,0,1]" : "=v"(r) : "v"(as_u32(h)));
  return r;
}
__device__ __forceinline__ float pair_difference(half2_t h) {
  float r;
  asm("v_fma_mix_f32 %0, %1, 1.0, -%1 op_sel:[0,0,1] op_sel_hi:[1,0,1]" : "=v"(r) : "v"(as_u32(h)));
  return r;
}

// Rotation of 16 rows by a wave.  Stage order h = 1, 2, ..., 64 with (x[i], x[i+h]) <- (x[i] + x[i+h], x[i] - x[i+h]) for
// (i & h) == 0, in binary32, then the binary32 scale and one rounding to fp16.  Five stages pair registers of one lane,
// two pair neighbouring lanes (other + own in the lower lane, other - own in the upper: one move and one exact
// multiply-add).
__device__ __forceinline__ void rotate_rows(half2_t (&h)[16], int q) {
  float x[32];
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    x[2 * i] = pair_sum(h[i]);
    x[2 * i + 1] = pair_difference(h[i]);
  }
#pragma unroll
  for (int s = 2; s <= 4; s <<= 1) {
#pragma unroll
    for (int i = 0; i < 32; ++i) {
      if ((i & s) == 0) {
        const float a = x[i], b = x[i + s];
        x[i] = a + b;
        x[i + s] = a - b;
      }
    }
  }
  const float s0 = (q & 1) ? -1.0f : 1.0f, s1 = (q & 2) ? -1.0f : 1.0f;
#pragma unroll
  for (int i = 0; i < 32; ++i) x[i] = __builtin_fmaf(x[i], s0, dpp_f<kQuadSwap1>(x[i]));
#pragma unroll
  for (int i = 0; i < 32; ++i) x[i] = __builtin_fmaf(x[i], s1, dpp_f<kQuadSwap2>(x[i]));
#pragma unroll
  for (int s = 8; s <= 16; s <<= 1) {
#pragma unroll
    for (int i = 0; i < 32; ++i) {
      if ((i & s) == 0) {
        const float a = x[i], b = x[i + s];
        x[i] = a + b;
        x[i + s] = a - b;
      }
    }
  }
  const float c = 0x1.6a09e6p-4f;  // fl32(1/sqrt(128))
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    float a = x[2 * i] * c, b = x[2 * i + 1] * c;
    // The contract rounds the product to binary32 first and to fp16 afterwards.  Keep the two roundings apart: a
    // fused multiply-and-convert instruction would round the exact product once and differ in rare near-tie cases.
    asm("" : "+v"(a), "+v"(b));
    h[i] = half2_t{(half_t)a, (half_t)b};
  }
}

// ---- Eq. 1 --------------------------------------------------------------------------------------------------------

// Eq. 1 at 2 or 4 bits against the stored fp16 scale / zero-point, decided in binary32 without a division.
struct QP {
  float z;  // value of the stored fp16 zero-point
  float s;  // value of the stored fp16 scale
  half_t z16, s16;
};

template <int BITS>
__device__ inline QP q_params(float mn, float mx) {
  mn = (mn == 0.0f) ? 0.0f : mn;  // a zero of either sign counts as +0
  mx = (mx == 0.0f) ? 0.0f : mx;
  QP r;
  r.z16 = (half_t)mn;  // exact: mn is an fp16 value
  r.z = mn;
  const float d32 = mx - mn;
  const float q32 = d32 / (float)Rec<BITS>::kLevels;  // IEEE-correct binary32 division
  r.s16 = (half_t)q32;
  r.s = (float)r.s16;
  return r;
}

// 4 bits.  The code is the number of thresholds (k + 0.5) s, k = 0 .. 14, that t = fl32(x - z) lies above -- strictly for
// even k, or on for odd k: round-half-to-even of t / s, clamped.  An estimate e from an approximate quotient (off by one at
// most, and only next to a threshold), then r = t - e s decides: e stands if |r| < s / 2, or |r| = s / 2 and e even.  r is
// exact: t >= s / 2 where e > 0, so t is a multiple of 2^-25 s at least as coarse as r needs (|r| <= s), e s has 15
// significant bits, and r = t where e = 0.  "Or on" for odd e is "above" the binary32 number next below s / 2.  t is never
// negative; a code beyond the last level can only come from a scale that was rounded down among the fp16 subnormals, and is
// clamped like the count of thresholds is.
// (13 vector instructions; the two thresholds around e formed and compared one by one took 24: 32 ragged prompts up to 4100
// tokens in three chunks 410 -> 376 us.)
__device__ inline float q_code4(float x, float z, float s, float inv_s) {
  constexpr float kTop = (float)Rec<4>::kLevels;
  const float t = x - z;
  const float e = __builtin_amdgcn_fmed3f(__builtin_rintf(t * inv_s), 0.0f, kTop);
  const float r = __builtin_fmaf(-e, s, t);
  const float half = __builtin_bit_cast(float, __builtin_bit_cast(uint32_t, 0.5f * s) - ((uint32_t)(int)e & 1u));
  const float c = fminf(e + (fabsf(r) > half ? __builtin_copysignf(1.0f, r) : 0.0f), kTop);
  return s == 0.0f ? 0.0f : c;
}

// 2 bits: code = (t > 0.5 s) + (t >= 1.5 s) + (t > 2.5 s) with t = fl32(x - z); 0 when s == 0.  Each of the three tests is a
// monotone function of x, so it is x > T_k for one binary16 number T_k: the largest x that fails it.  With h = (k + 0.5) s
// (exact in binary32, and even there: at most 14 significant bits) and u = half a unit in the last place of h,
// fl32(d) > h <=> d > h + u and fl32(d) >= h <=> d >= h - u (ties go to h), so T_k is the largest binary16 number <= z + h + u
// (k = 0, 2) or < z + h - u (k = 1).  The sum is taken in binary64: z is a multiple of 2^-24 and h of 2^-25, both below
// 2^18, and u a power of two; either the sum is exact (u >= 2^-35) or u is less than half the distance to the next
// binary16 number on its side, so its rounding cannot cross one.
__device__ inline uint32_t threshold2(float z, float s, int k) {
  const float h = ((float)k + 0.5f) * s;
  const float u = __builtin_bit_cast(float, (((__builtin_bit_cast(uint32_t, h) >> 23) & 255u) - 24u) << 23);  // (s > 0: h >= 2^-25)
  const bool strict = k == 1;
  const double y = (double)z + (double)h + (strict ? -(double)u : (double)u);
  half_t c = (half_t)(float)y;  // one of the two binary16 neighbours of y
  c = (float)c > 65504.0f ? (half_t)65504.0f : c;
  uint32_t bits = __builtin_bit_cast(unsigned short, c);
  const double cd = (double)(float)c;
  if (strict ? cd >= y : cd > y)  // step down to the next binary16 number
    bits = (bits & 0x7fffu) == 0u ? 0x8001u : (bits & 0x8000u) ? bits + 1u : bits - 1u;
  bits = bits == 0x8000u ? 0u : bits;  // never -0: x = +0 is not above it
  return s == 0.0f ? 0x7bffu : bits;   // 65504: no finite x is above it
}

// Bit pairs of the codes of four elements (two registers of binary16): hi in bit 7, lo in bit 5 of every byte; a code 0, 1,
// 2, 3 is (1,1), (1,0), (0,0), (0,1).  The sign of T_k - x tells x > T_k (never confused by zeros: T_k is not -0).  sel: the
// order of the bytes (1, 3 = the elements of xa, 5, 7 = those of xb).
__device__ __forceinline__ uint32_t symbols2(half2_t xa, half2_t xb, half2_t t1a, half2_t t2a, half2_t t3a, half2_t t1b, half2_t t2b,
                                             half2_t t3b, uint32_t sel) {
  const uint32_t la = ~as_u32(t1a - xa) | as_u32(t3a - xa), lb = ~as_u32(t1b - xb) | as_u32(t3b - xb);
  const uint32_t d2 = __builtin_amdgcn_perm(as_u32(t2b - xb), as_u32(t2a - xa), sel), lo = __builtin_amdgcn_perm(lb, la, sel);
  return (~d2 & 0x80808080u) | ((lo >> 2) & 0x20202020u);
}
// The same for four 2-bit codes (digits), one per byte in bits `at`, `at` + 1: hi in bit 7, lo in bit 5 of every byte.
template <int AT>
__device__ __forceinline__ uint32_t symbols_of_digits(uint32_t c) {
  const uint32_t hi = ~c & (0x02020202u << AT), lo = ~(c ^ (c >> 1)) & (0x01010101u << AT);
  return (hi << (6 - AT)) | (lo << (5 - AT));
}
__device__ __forceinline__ uint32_t splat16(uint32_t bits) { return bits | (bits << 16); }

// ---- a whole group ------------------------------------------------------------------------------------------------

// LDS of quantize_group besides the record image; NW = waves of the workgroup.
template <int NW>
struct QuantLds {
  half_t kmn[NW][kGroup], kmx[NW][kGroup];  // per-channel key minima / maxima of each wave's tokens
  half_t thr[3][kGroup];                    // 2 bits: T_k of every channel
  float s[kGroup], z[kGroup];               // 4 bits
};

// Value part of a record: one pass of a wave over 16 tokens.  Pass P takes the tokens 16 i + tok with
// i = 2 (P / 2) + ip and tok = 8 (P % 2) + 2 rho + b: byte P / 2 of the tile words holds the codes of i = 2 (P / 2) and + 1,
// and the codes of tok, tok + 1 share a word, so the four lanes that differ in (ip, b) fill one byte of a word.
__device__ __forceinline__ int value_pass_token(int pass, const RowLane& rl) {
  return 16 * (2 * (pass >> 1) + rl.ip) + 8 * (pass & 1) + 2 * rl.rho + rl.b;
}

// out[k] = bytes of the channels 32 (k / 2) + 8 q + 4 (k % 2) + 0..3 with hi / lo of this lane's token in bits 7 / 5.  They
// are moved to their place in the byte, the four lanes that share bytes are combined (each ends up with the channels of
// two of the k), and every lane stores its 8 bytes.  plane: the LDS words of the tile (plane).
__device__ __forceinline__ void put_value_bytes(uint32_t (&out)[8], int pass, const RowLane& rl, uint32_t* plane) {
  const int sh = 4 - 4 * rl.ip + rl.b;
#pragma unroll
  for (int k = 0; k < 8; ++k) out[k] >>= sh;
  uint32_t v[4], w[2];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const uint32_t keep = rl.ip ? out[4 + j] : out[j], send = rl.ip ? out[j] : out[4 + j];
    v[j] = keep | dpp_u<kRowRor8>(send);
  }
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const uint32_t keep = rl.b ? v[2 + j] : v[j], send = rl.b ? v[j] : v[2 + j];
    w[j] = keep | dpp_u<kRowHalfMirror>(send);
  }
  // tile word of (channel 16 n + jr, quarter g, w): ((n / 2) * 64 + jr + 16 g) * 4 + 2 (n % 2) + w; with tok0 = 4 a + 2 h the
  // first of the two tokens, a = (2 g + w) % 4 and h = g / 2
  const int m = 2 * rl.ip + rl.b, g = 2 * (rl.rho & 1) + (pass & 1), wd = rl.rho >> 1;
  unsigned char* bytes = reinterpret_cast<unsigned char*>(plane) +
                         4 * ((m * 64 + 8 * (rl.q & 1) + 16 * g) * 4 + 2 * (rl.q >> 1) + wd) + (pass >> 1);
#pragma unroll
  for (int j = 0; j < 2; ++j)
#pragma unroll
    for (int c = 0; c < 4; ++c) bytes[16 * (4 * j + c)] = (unsigned char)(w[j] >> (8 * c));
}

// Quantizes the rotated values of the pass's 16 tokens (h: as row_pairs) and writes their codes, scales and zero-points to
// the record image.  Returns whether a value of the lane's token is not finite.
template <int BITS>
__device__ __forceinline__ bool quantize_value_pass(const half2_t (&h)[16], int pass, const RowLane& rl, int lane, uint32_t* img) {
  using R = Rec<BITS>;
  half2_t mn = h[0], mx = h[0];
#pragma unroll
  for (int i = 1; i < 16; ++i) {
    mn = h2_min(mn, h[i]);
    mx = h2_max(mx, h[i]);
  }
  // the minimum and the negated maximum ride in one register
  half2_t u = h2_min(half2_t{mn[0], (half_t)-mx[0]}, half2_t{mn[1], (half_t)-mx[1]});
  u = h2_min(u, dpp_h2<kQuadSwap1>(u));
  u = h2_min(u, dpp_h2<kQuadSwap2>(u));
  const bool bad = nonfinite_pair(as_u32(u));
  const QP p = q_params<BITS>((float)u[0], -(float)u[1]);
  const int t = value_pass_token(pass, rl);
  if ((lane & 3) == 0)  // token 16 n + j at word 8 j + n of the field
    img[R::kValueSZ + 8 * (t & 15) + (t >> 4)] = as_u32(half2_t{p.s16, p.z16});
  uint32_t out[8];
  if constexpr (BITS == 2) {
    const int lq = lane & 3;
    const uint32_t mine = splat16(threshold2(p.z, p.s, lq < 2 ? lq : 2));  // lane k of the quad: T_k
    const half2_t t1 = as_h2(dpp_u<0x00>(mine)), t2 = as_h2(dpp_u<0x55>(mine)), t3 = as_h2(dpp_u<0xAA>(mine));
#pragma unroll
    for (int k = 0; k < 8; ++k)
      out[k] = symbols2(h[2 * k], h[2 * k + 1], t1, t2, t3, t1, t2, t3, 0x07050301u);
    put_value_bytes(out, pass, rl, img + R::kValueTile);
  } else {
    uint32_t low[8];
    const float inv_s = __builtin_amdgcn_rcpf(p.s);
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      uint32_t c = 0;
#pragma unroll
      for (int e = 0; e < 4; ++e) c = __builtin_amdgcn_cvt_pk_u8_f32(q_code4((float)h[2 * k + (e >> 1)][e & 1], p.z, p.s, inv_s), e, c);
      out[k] = symbols_of_digits<2>(c);
      low[k] = symbols_of_digits<0>(c);
    }
    put_value_bytes(out, pass, rl, img + R::kValueTile);
    put_value_bytes(low, pass, rl, img + R::kValueTile + kPlaneWords);
  }
  return bad;
}

// Keys of a group in registers: 16 lanes per row, lane = 8 channels of the tokens 4 NW i + 4 wave + lane / 16.
template <int NW>
struct KeyTile {
  uint4 raw[32 / NW];
};
template <int NW>
__device__ __forceinline__ int key_token(int i, int wave, int lane) { return 4 * NW * i + 4 * wave + (lane >> 4); }

// First half of the key quantizer: minima and maxima per channel over each wave's tokens, left in LDS.
template <int NW>
__device__ __forceinline__ void key_minmax(const KeyTile<NW>& k, int valid, QuantLds<NW>& L, int wave, int lane) {
  const half2_t top = {(half_t)INFINITY, (half_t)INFINITY};
  half2_t mn[4] = {top, top, top, top}, mx[4] = {-top, -top, -top, -top};
#pragma unroll
  for (int i = 0; i < 32 / NW; ++i) {
    if (valid == kGroup || key_token<NW>(i, wave, lane) < valid) {
      const half2_t x[4] = {as_h2(k.raw[i].x), as_h2(k.raw[i].y), as_h2(k.raw[i].z), as_h2(k.raw[i].w)};
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        mn[v] = h2_min(mn[v], x[v]);
        mx[v] = h2_max(mx[v], x[v]);
      }
    }
  }
  // over the wave's four rows of lanes; row 0 keeps the minima, row 1 the maxima
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    uint32_t a = as_u32(mn[v]), b = as_u32(mx[v]);
    mn[v] = h2_min(as_h2(a), as_h2(__shfl_xor(a, 16, 64)));
    mx[v] = h2_max(as_h2(b), as_h2(__shfl_xor(b, 16, 64)));
    a = as_u32(mn[v]); b = as_u32(mx[v]);
    mn[v] = h2_min(as_h2(a), as_h2(__shfl_xor(a, 32, 64)));
    mx[v] = h2_max(as_h2(b), as_h2(__shfl_xor(b, 32, 64)));
  }
  if (lane < 16) *reinterpret_cast<uint4*>(&L.kmn[wave][8 * lane]) = make_uint4(as_u32(mn[0]), as_u32(mn[1]), as_u32(mn[2]), as_u32(mn[3]));
  else if (lane < 32) *reinterpret_cast<uint4*>(&L.kmx[wave][8 * (lane & 15)]) = make_uint4(as_u32(mx[0]), as_u32(mx[1]), as_u32(mx[2]), as_u32(mx[3]));
}

// Between two barriers: scale and zero-point of channel tid (< 128), into the record image and for key_codes.  Returns
// whether a key of the channel is not finite.
template <int BITS, int NW>
__device__ __forceinline__ bool key_params(QuantLds<NW>& L, int tid, uint32_t* img) {
  half_t mn = L.kmn[0][tid], mx = L.kmx[0][tid];
  half2_t u = {mn, (half_t)-mx};
#pragma unroll
  for (int w = 1; w < NW; ++w) u = h2_min(u, half2_t{L.kmn[w][tid], (half_t)-L.kmx[w][tid]});
  const QP p = q_params<BITS>((float)u[0], -(float)u[1]);
  half_t* img16 = reinterpret_cast<half_t*>(img);
  img16[2 * Rec<BITS>::kKeyScale + tid] = p.s16;
  img16[2 * Rec<BITS>::kKeyZero + tid] = p.z16;
  if constexpr (BITS == 2) {
#pragma unroll
    for (int k = 0; k < 3; ++k) L.thr[k][tid] = __builtin_bit_cast(half_t, (unsigned short)threshold2(p.z, p.s, k));
  } else {
    L.s[tid] = p.s;
    L.z[tid] = p.z;
  }
  return nonfinite_pair(as_u32(u));
}

// Second half: codes and key tile.  Tile word ((n / 2) * 64 + j + 16 g) * 4 + 2 (n % 2) + w holds, for the row 16 n + j (token),
// the positions (channels) 32 g + 16 w + 8 (p % 2) + p / 2, p = 0..15: this lane's 8 channels are the p % 2 = sub % 2 half of
// the word of (g, w) = (sub / 4, (sub / 2) % 2), its neighbour has the other half; the neighbours take turns storing.
template <int BITS, int NW>
__device__ __forceinline__ void key_codes(KeyTile<NW>& k, int valid, const QuantLds<NW>& L, int wave, int lane, uint32_t* img) {
  const int sub = lane & 15;
  constexpr int kPlanes = BITS / 2;
  half2_t t[3][4];
  float s[8], z[8], inv_s[8];
  if constexpr (BITS == 2) {
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      const uint4 r = *reinterpret_cast<const uint4*>(&L.thr[i][8 * sub]);
      t[i][0] = as_h2(r.x); t[i][1] = as_h2(r.y); t[i][2] = as_h2(r.z); t[i][3] = as_h2(r.w);
    }
  } else {
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      s[e] = L.s[8 * sub + e];
      z[e] = L.z[8 * sub + e];
      inv_s[e] = __builtin_amdgcn_rcpf(s[e]);
    }
  }
  if (BITS == 2 && valid < kGroup) {  // padding tokens: -65504, above no T_k
    constexpr uint32_t kLowest = 0xFBFFFBFFu;
#pragma unroll
    for (int i = 0; i < 32 / NW; ++i)
      if (key_token<NW>(i, wave, lane) >= valid) k.raw[i] = make_uint4(kLowest, kLowest, kLowest, kLowest);
  }
  const int wbase = 16 * (sub >> 2) * 4 + ((sub >> 1) & 1);
#pragma unroll
  for (int i = 0; i < 32 / NW; i += 2) {
    uint32_t word[2][kPlanes];
#pragma unroll
    for (int d = 0; d < 2; ++d) {
      const uint4 r = k.raw[i + d];
      const uint32_t x[4] = {r.x, r.y, r.z, r.w};
      const bool live = BITS == 2 || valid == kGroup || key_token<NW>(i + d, wave, lane) < valid;  // padding tokens: code 0
      if constexpr (BITS == 2) {
        const uint32_t y01 = symbols2(as_h2(x[0]), as_h2(x[1]), t[0][0], t[1][0], t[2][0], t[0][1], t[1][1], t[2][1], 0x07030501u);
        const uint32_t y23 = symbols2(as_h2(x[2]), as_h2(x[3]), t[0][2], t[1][2], t[2][2], t[0][3], t[1][3], t[2][3], 0x07030501u);
        const uint32_t even = __builtin_amdgcn_perm(y23, y01, 0x05040100u), odd = __builtin_amdgcn_perm(y23, y01, 0x07060302u);
        word[d][0] = (odd | (even >> 4)) >> (sub & 1);
      } else {
        uint32_t c[2] = {0, 0};  // codes of the even / odd channels, one per byte
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const float code = live ? q_code4((float)as_h2(x[e >> 1])[e & 1], z[e], s[e], inv_s[e]) : 0.0f;
          c[e & 1] = __builtin_amdgcn_cvt_pk_u8_f32(code, e >> 1, c[e & 1]);
        }
        word[d][0] = (symbols_of_digits<2>(c[1]) | (symbols_of_digits<2>(c[0]) >> 4)) >> (sub & 1);
        word[d][kPlanes - 1] = (symbols_of_digits<0>(c[1]) | (symbols_of_digits<0>(c[0]) >> 4)) >> (sub & 1);
      }
    }
#pragma unroll
    for (int pl = 0; pl < kPlanes; ++pl) {
#pragma unroll
      for (int d = 0; d < 2; ++d) word[d][pl] |= dpp_u<kQuadSwap1>(word[d][pl]);
      // (values, not places: a choice between two elements of the array would put the array into memory)
      const uint32_t first = word[0][pl], second = word[1][pl], mine = (sub & 1) ? second : first;
      const int tk = key_token<NW>((sub & 1) ? i + 1 : i, wave, lane), nb = tk >> 4, jr = tk & 15;
      img[Rec<BITS>::kKeyTile + kPlaneWords * pl + ((nb >> 1) * 64 + jr) * 4 + 2 * (nb & 1) + wbase] = mine;
    }
  }
}

// Window values live 4 slots per channel; this brings the first `rows` slots into LDS rows of kRowH halfs (threads of a
// workgroup of 64 NW; a barrier has to follow).
template <int NW>
struct WindowValues {
  uint4 w[2048 / (64 * NW)];  // 16-byte pieces: 4 slots of 2 channels
};
template <int NW>
__device__ __forceinline__ void request_window_values(WindowValues<NW>& r, const half_t* __restrict__ v_win, int rows, int tid) {
  const int n = ((rows + 3) >> 2) * 64;
#pragma unroll
  for (int i = 0; i < 2048 / (64 * NW); ++i) {
    const int it = tid + 64 * NW * i;
    r.w[i] = make_uint4(0, 0, 0, 0);
    if (it < n) r.w[i] = *reinterpret_cast<const uint4*>(v_win + ((long long)(it >> 6) * kHeadDim + 2 * (it & 63)) * 4);
  }
}
template <int NW>
__device__ __forceinline__ void put_window_values(const WindowValues<NW>& r, int rows, half_t (*st)[kRowH], int tid) {
  const int n = ((rows + 3) >> 2) * 64;
#pragma unroll
  for (int i = 0; i < 2048 / (64 * NW); ++i) {
    const int it = tid + 64 * NW * i;
    if (it < n) {
      const uint4 w = r.w[i];
      uint32_t* row = reinterpret_cast<uint32_t*>(&st[4 * (it >> 6)][2 * (it & 63)]);
      row[0] = __builtin_amdgcn_perm(w.z, w.x, 0x05040100u);
      row[kRowH / 2] = __builtin_amdgcn_perm(w.z, w.x, 0x07060302u);
      row[kRowH] = __builtin_amdgcn_perm(w.w, w.y, 0x05040100u);
      row[3 * kRowH / 2] = __builtin_amdgcn_perm(w.w, w.y, 0x07060302u);
    }
  }
}
template <int NW>
__device__ __forceinline__ void stage_window_values(const half_t* __restrict__ v_win, int rows, half_t (*st)[kRowH], int tid) {
  WindowValues<NW> r;
  request_window_values<NW>(r, v_win, rows, tid);
  put_window_values<NW>(r, rows, st, tid);
}

// The record of one group into the LDS image img (Rec<BITS>::kWords).  Tokens 0 .. nrg - 1 come from the window (raw keys
// k_win, slot = token; rotated values staged in st), the others up to `valid` are the new rows k_src, v_src + 128 (token - nrg);
// padding tokens beyond are zero rows.  st may lie in the same LDS as img: where rows come from it they are all read before
// anything is written.  Returns whether this thread saw a value or key that is not finite.  Ends with a barrier.
template <int BITS, int NW>
__device__ __forceinline__ bool quantize_group(const half_t* __restrict__ k_win, const half_t* __restrict__ k_src,
                                               const half_t* __restrict__ v_src, half_t (*st)[kRowH], int nrg, int valid,
                                               QuantLds<NW>& L, uint32_t* img, int wave, int lane) {
  constexpr int kPasses = 8 / NW;
  const int tid = 64 * wave + lane;
  bool bad = false;
  KeyTile<NW> k;
#pragma unroll
  for (int i = 0; i < 32 / NW; ++i) {
    const int t = key_token<NW>(i, wave, lane);
    const half_t* row = t < nrg ? k_win + (long long)t * kHeadDim : k_src + (long long)(t - nrg) * kHeadDim;
    k.raw[i] = make_uint4(0, 0, 0, 0);
    if (t < valid) k.raw[i] = *reinterpret_cast<const uint4*>(row + 8 * (lane & 15));
  }
  const RowLane rl = row_lane(lane);
  Row v[kPasses];
#pragma unroll
  for (int i = 0; i < kPasses; ++i) {
    const int t = value_pass_token(kPasses * wave + i, rl);
#pragma unroll
    for (int m = 0; m < 4; ++m) v[i].p[m] = make_uint4(0, 0, 0, 0);
    if (t >= nrg && t < valid) load_row(v[i], v_src + (long long)(t - nrg) * kHeadDim, rl.q);
  }
  key_minmax<NW>(k, valid, L, wave, lane);
  half2_t h[kPasses][16];
#pragma unroll
  for (int i = 0; i < kPasses; ++i) {
    row_pairs(v[i], h[i]);
    if (nrg < kGroup) rotate_rows(h[i], rl.q);
    if (nrg > 0) {
      const int t = value_pass_token(kPasses * wave + i, rl);
      Row w;
      load_row(w, st[t], rl.q);
      half2_t hw[16];
      row_pairs(w, hw);
#pragma unroll
      for (int e = 0; e < 16; ++e) h[i][e] = t < nrg ? hw[e] : h[i][e];
    }
  }
  if (nrg > 0) lds_barrier();
#pragma unroll
  for (int i = 0; i < kPasses; ++i) bad |= quantize_value_pass<BITS>(h[i], kPasses * wave + i, rl, lane, img);
  lds_barrier();
  if (tid < kGroup) bad |= key_params<BITS, NW>(L, tid, img);
  lds_barrier();
  key_codes<BITS, NW>(k, valid, L, wave, lane, img);
  lds_barrier();
  return bad;
}

}  // namespace
}  // namespace kvlinc
