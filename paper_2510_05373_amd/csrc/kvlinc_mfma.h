// Device helpers shared by the kernels of libkvlinc: binary16 vector types, lane-quad data movement and the 4x4x4
// matrix-core instruction with a broadcast A operand (not part of the C ABI).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace kvlinc {
namespace {

typedef _Float16 half_t;
typedef _Float16 half2_t __attribute__((ext_vector_type(2)));
typedef _Float16 half4_t __attribute__((ext_vector_type(4)));
typedef float float4_t __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));


__device__ __forceinline__ uint32_t as_u32(half2_t v) { return __builtin_bit_cast(uint32_t, v); }
__device__ __forceinline__ half2_t as_h2(uint32_t v) { return __builtin_bit_cast(half2_t, v); }
__device__ __forceinline__ half4_t as_h4(uint32_t a, uint32_t b) {
  u32x2_t v = {a, b};
  return __builtin_bit_cast(half4_t, v);
}


template <int CTRL>
__device__ __forceinline__ float dpp_f(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xf, 0xf, true));
}
template <int CTRL>
__device__ __forceinline__ uint32_t dpp_u(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xf, 0xf, true);
}
constexpr int kQuadSwap1 = 0xB1;   // quad_perm [1,0,3,2]
constexpr int kQuadSwap2 = 0x4E;   // quad_perm [2,3,0,1]

constexpr int kRowRor4 = 0x124, kRowRor8 = 0x128, kRowRor1 = 0x121, kRowRor2 = 0x122;
constexpr int kQuadMirror = 0x1B, kRowHalfMirror = 0x141;  // lane ^ 3, lane ^ 7

// v as its neighbours at lane ^ N hold it: x takes v of the lane of the pair whose bit N is clear, y that of the other (N = 16, 32).
template <int N>
__device__ __forceinline__ void pair_across(float v, float& x, float& y) {
  static_assert(N == 16 || N == 32, "the rows and the halves of a wave");
  const uint32_t p = __builtin_bit_cast(uint32_t, v);
  const auto r = N == 16 ? __builtin_amdgcn_permlane16_swap(p, p, false, false) : __builtin_amdgcn_permlane32_swap(p, p, false, false);
  const uint32_t lower = r[0], upper = r[1];  // (a bit cast of r[1] itself would take r[0]: it goes by the address of the vector)
  x = __builtin_bit_cast(float, lower);
  y = __builtin_bit_cast(float, upper);
}

// reductions over the 64 lanes of a wave, result in every lane: rotations inside the rows of 16 lanes, then two
// cross-row exchanges
__device__ __forceinline__ float wave_allmax(float v) {
  v = fmaxf(v, dpp_f<kRowRor1>(v));
  v = fmaxf(v, dpp_f<kRowRor2>(v));
  v = fmaxf(v, dpp_f<kRowRor4>(v));
  v = fmaxf(v, dpp_f<kRowRor8>(v));
  float x, y;
  pair_across<16>(v, x, y);
  pair_across<32>(fmaxf(x, y), x, y);
  return fmaxf(x, y);
}
__device__ __forceinline__ float wave_allsum(float v) {
  v += dpp_f<kRowRor1>(v);
  v += dpp_f<kRowRor2>(v);
  v += dpp_f<kRowRor4>(v);
  v += dpp_f<kRowRor8>(v);
  float x, y;
  pair_across<16>(v, x, y);
  pair_across<32>(x + y, x, y);
  return x + y;
}

// Butterflies between the lanes of a wave, strides 1, 2, 4, ..., 32 in this order: the lane whose bit is clear takes own + other,
// the one whose bit is set other - own, each rounded once (a multiply-add with +-1 is exact up to the sum).  In registers: six
// exchanges through LDS (ds_bpermute) cost a wave that waits for nothing else about 0.3 us.  (Here, in the reductions above and in the
// combine of the decode workgroups: a step of 1 sequence of 300 tokens 12.7 -> 12.1 us, 16 of 8k 25.9 -> 25.3, 1 of 131072
// 25.1 -> 24.5.)  NV vectors at once.
template <int NV>
__device__ __forceinline__ void row_butterflies(float (&v)[NV], int lane) {  // strides 1 .. 16: inside the halves of a wave
  auto sign = [&](int bit) { return (lane & bit) != 0 ? -1.0f : 1.0f; };
  const float s1 = sign(1), s2 = sign(2), s4 = sign(4), s8 = sign(8), s16 = sign(16);
#pragma unroll
  for (int u = 0; u < NV; ++u) v[u] = __builtin_fmaf(v[u], s1, dpp_f<kQuadSwap1>(v[u]));
#pragma unroll
  for (int u = 0; u < NV; ++u) v[u] = __builtin_fmaf(v[u], s2, dpp_f<kQuadSwap2>(v[u]));
#pragma unroll
  for (int u = 0; u < NV; ++u) v[u] = __builtin_fmaf(v[u], s4, dpp_f<kQuadMirror>(dpp_f<kRowHalfMirror>(v[u])));
#pragma unroll
  for (int u = 0; u < NV; ++u) v[u] = __builtin_fmaf(v[u], s8, dpp_f<kRowRor8>(v[u]));
#pragma unroll
  for (int u = 0; u < NV; ++u) {
    float x, y;
    pair_across<16>(v[u], x, y);
    v[u] = __builtin_fmaf(y, s16, x);
  }
}
template <int NV>
__device__ __forceinline__ void lane_butterflies(float (&v)[NV], int lane) {
  row_butterflies<NV>(v, lane);
  const float s32 = (lane & 32) != 0 ? -1.0f : 1.0f;
#pragma unroll
  for (int u = 0; u < NV; ++u) {
    float x, y;
    pair_across<32>(v[u], x, y);
    v[u] = __builtin_fmaf(y, s32, x);
  }
}

// D = A B + C on the sixteen 4x4 blocks of a wave, k = 4, binary16 operands, binary32 accumulate.  Lane 4 b + i holds
// row i of A_b (4 halves), column i of B_b (4 halves) and column i of D_b (4 floats).  Here every block uses the A
// of block `abid` (broadcast), so one register pair can carry the A operands of 16 successive steps.
__device__ __forceinline__ float4_t mfma_bcast(half4_t a, half4_t b, float4_t c, int abid) {
  switch (abid) {
    case 0: return __builtin_amdgcn_mfma_f32_4x4x4f16(a, b, c, 4, 0, 0);
    case 1: return __builtin_amdgcn_mfma_f32_4x4x4f16(a, b, c, 4, 1, 0);
    case 2: return __builtin_amdgcn_mfma_f32_4x4x4f16(a, b, c, 4, 2, 0);
    case 3: return __builtin_amdgcn_mfma_f32_4x4x4f16(a, b, c, 4, 3, 0);
    case 4: return __builtin_amdgcn_mfma_f32_4x4x4f16(a, b, c, 4, 4, 0);
    case 5: return __builtin_amdgcn_mfma_f32_4x4x4f16(a, b, c, 4, 5, 0);
    case 6: return __builtin_amdgcn_mfma_f32_4x4x4f16(a, b, c, 4, 6, 0);
    case 7: return __builtin_amdgcn_mfma_f32_4x4x4f16(a, b, c, 4, 7, 0);
    case 8: return __builtin_amdgcn_mfma_f32_4x4x4f16(a, b, c, 4, 8, 0);
    case 9: return __builtin_amdgcn_mfma_f32_4x4x4f16(a, b, c, 4, 9, 0);
    case 10: return __builtin_amdgcn_mfma_f32_4x4x4f16(a, b, c, 4, 10, 0);
    case 11: return __builtin_amdgcn_mfma_f32_4x4x4f16(a, b, c, 4, 11, 0);
    case 12: return __builtin_amdgcn_mfma_f32_4x4x4f16(a, b, c, 4, 12, 0);
    case 13: return __builtin_amdgcn_mfma_f32_4x4x4f16(a, b, c, 4, 13, 0);
    case 14: return __builtin_amdgcn_mfma_f32_4x4x4f16(a, b, c, 4, 14, 0);
    default: return __builtin_amdgcn_mfma_f32_4x4x4f16(a, b, c, 4, 15, 0);
  }
}

}  // namespace
}  // namespace kvlinc
