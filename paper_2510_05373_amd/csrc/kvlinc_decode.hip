// Decode: single-query attention read directly from the packed 2-bit cache on the CDNA4 matrix cores, with the
// linear correction and the fp16 window (Sec. 3.3, Alg. 1; Sec. 3.2, Eq. 5-6; Sec. 3.1 for the rotated value basis).
//
// decode_main_kernel, one launch per decode step, two kinds of workgroups:
//   streaming workgroups (sequence, kv head, split): the four waves take groups of 128 tokens from a static schedule
//   that is the same for every sequence length; a wave keeps its own (m, l, acc).  The number of splits of a
//   sequence follows its share of the batch's groups, so that sequences of unequal lengths end together.  A group record is fetched in two
//   parts, each requested again for the wave's next group as soon as its contraction has consumed it.  The four
//   waves of split 0 of a (sequence, kv head) also take a share of the fp16 window each, as one more block of tokens.  The
//   waves are combined through LDS and the workgroup writes one (m, l, Y_s) per query head (Alg. 1 line 11);
//   correction workgroups (kv head, part of phi, 1 to 8 sequences): C_n = phi_q S and C_d = phi_q P, cut into parts over
//   the rows of S, on the matrix cores.
// Every workgroup counts itself in at its (sequence, kv head); the streaming workgroup that arrives last, or the correction
// workgroup where that is later and not awaited (see kvlinc_handoff.h), merges: it weighs the splits by 2^(m_j - M), adds the
// correction as (num + 2^-M C_n) / (den + 2^-M C_d), applies H^T and stores fp16 (Alg. 1 lines 13-15 with Eq. 5).  A wait
// is bounded: if it runs out, whoever comes last merges.
//
// The two contractions of a group (Alg. 1 lines 5-10) run on v_mfma_scale_f32_16x16x128_f8f6f4, 16 rows x 16 columns x
// 128 contraction positions per instruction, 8 instructions per contraction and block of 4 query heads:
//   q K^T : columns = 16 tokens, positions = the 128 channels;  E V : columns = 16 channels, positions = the 128 tokens.
// B operand = the codes, read as FP4 (E2M1).  A code c is stored as a bit pair (hi, lo) such that the nibble hi|0|lo|1 is
// the FP4 number c - 1.5; a word keeps the pairs of two codes interleaved in every nibble, so one AND-OR (and one shift
// for the second code of the nibbles) turns 8 codes into a B register.  Codes are never dequantized, and the centred
// codes keep the sums free of a common sign (the matrix cores add with a truncating adder: all-positive products
// would leave a bias that the zero-point term, summed exactly, does not share).
// A operand = the small side, (q * key scale) resp. (p * value scale), as FP8 (E4M3) in three terms per value:
//   x = 2^e (t0 + t1 / 16 + t2 / 256), t_k = fp8 of what the earlier terms left, each term in a row of its own,
//   rows = 4 heads x (3 terms + 1 spare), the factor 2^(e - 4 k) in the row's block scale.
// The terms leave 2^-12 of x at most (better than binary16); e follows the largest |x| of the head in that group, so
// no operand overflows or flushes whatever the magnitude of keys, queries and values.  The three rows of a head are
// summed after the instruction.
// Zero-points never touch the tiles: sum_c q_c (s_c code + z_c) = sum_c (q_c s_c) (code - 1.5) + sum_c q_c (z_c + 1.5 s_c),
// and likewise for the values per token.  Scores live in the log2 domain: x = q.k * log2(e)/sqrt(d).
#include <hip/hip_runtime.h>
#include <hip/hip_ext.h>

#include "kvlinc_handoff.h"
#include "kvlinc_internal.h"
#include "kvlinc_mfma.h"
#include "kvlinc_schedule.h"

namespace kvlinc {
namespace {

constexpr int kThreads = 64 * kWaves;
constexpr float kLog2e = 1.4426950408889634f;
constexpr float kAlpha = kLog2e * 0.08838834764831845f;  // log2(e) / sqrt(128)

typedef int v8i_t __attribute__((ext_vector_type(8)));
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
typedef short short2_t __attribute__((ext_vector_type(2)));
typedef float float2_t __attribute__((ext_vector_type(2)));
typedef _Float16 half8_t __attribute__((ext_vector_type(8)));

// ---- small helpers ----------------------------------------------------------------------------------------------

// Results that one workgroup writes and another reads inside the same launch (split partials, correction parts) go
// through stores and loads that are coherent across the chip's L2 slices: a workgroup-wide cache write-back /
// invalidate (what a device-scope fence costs here) would throw away the streamed records.
__device__ __forceinline__ void st_coherent(float* p, float v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}
__device__ __forceinline__ void st_coherent2(float* p, float x, float y) {  // two neighbours, 8-byte aligned
  __hip_atomic_store(reinterpret_cast<unsigned long long*>(p), __builtin_bit_cast(unsigned long long, float2_t{x, y}), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}
__device__ __forceinline__ float2 ld_coherent2(const float* p) {  // two neighbours, 8-byte aligned
  const unsigned long long v = __hip_atomic_load(reinterpret_cast<const unsigned long long*>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  return __builtin_bit_cast(float2, v);
}
// A number that the launch only reads, through the scalar cache: it does not wait behind the vector loads requested before it.
__device__ __forceinline__ int scalar_load(const int32_t* p) {
  typedef const __attribute__((address_space(4))) int32_t* constant_ptr;
  return *reinterpret_cast<constant_ptr>(reinterpret_cast<uintptr_t>(p));
}
// Cache policy of a buffer load that is coherent in the same way: sc0 and sc1.
constexpr int kCoherentLoad = 1 | 16;
constexpr int kAllLoads = 0x0f70;  // s_waitcnt vmcnt(0)

__device__ __forceinline__ float as_f32(uint32_t v) { return __builtin_bit_cast(float, v); }
__device__ __forceinline__ uint32_t as_bits(float v) { return __builtin_bit_cast(uint32_t, v); }

// Reductions with the result in every participating lane.  row: the 16 lanes of a DPP row; quad: 4 adjacent lanes;
// xrow: the 4 lanes l, l ^ 16, l ^ 32, l ^ 48 (row swaps: odd rows of one copy against even rows of the other, then
// the upper 32 lanes of one against the lower 32 of the other).  The *_umax forms take bit patterns of non-negative
// numbers, which order like the numbers themselves (one instruction per step, no NaN handling).
__device__ __forceinline__ float row_allmax(float v) {
  v = fmaxf(v, dpp_f<kRowRor1>(v));
  v = fmaxf(v, dpp_f<kRowRor2>(v));
  v = fmaxf(v, dpp_f<kRowRor4>(v));
  return fmaxf(v, dpp_f<kRowRor8>(v));
}
__device__ __forceinline__ float row_allsum(float v) {
  v += dpp_f<kRowRor1>(v);
  v += dpp_f<kRowRor2>(v);
  v += dpp_f<kRowRor4>(v);
  return v + dpp_f<kRowRor8>(v);
}
__device__ __forceinline__ uint32_t row_umax(uint32_t v) {
  v = max(v, dpp_u<kRowRor1>(v));
  v = max(v, dpp_u<kRowRor2>(v));
  v = max(v, dpp_u<kRowRor4>(v));
  return max(v, dpp_u<kRowRor8>(v));
}
__device__ __forceinline__ uint32_t quad_umax(uint32_t v) {
  v = max(v, dpp_u<kQuadSwap1>(v));
  return max(v, dpp_u<kQuadSwap2>(v));
}
__device__ __forceinline__ float quad_allsum(float v) {
  v += dpp_f<kQuadSwap1>(v);
  return v + dpp_f<kQuadSwap2>(v);
}
__device__ __forceinline__ uint32_t xrow_umax(uint32_t v) {
  auto a = __builtin_amdgcn_permlane16_swap(v, v, false, false);
  v = max(a[0], a[1]);
  auto b = __builtin_amdgcn_permlane32_swap(v, v, false, false);
  return max(b[0], b[1]);
}
__device__ __forceinline__ float xrow_allsum(float v) {
  auto a = __builtin_amdgcn_permlane16_swap(as_bits(v), as_bits(v), false, false);
  v = as_f32(a[0]) + as_f32(a[1]);
  auto b = __builtin_amdgcn_permlane32_swap(as_bits(v), as_bits(v), false, false);
  return as_f32(b[0]) + as_f32(b[1]);
}

// The compiler may not move LDS traffic of one wave across this point (the hardware keeps a wave's LDS instructions
// in order, which is all a wave needs to hand data from lane to lane through LDS).
__device__ __forceinline__ void lds_order() { asm volatile("" ::: "memory"); }

// ---- operand layouts of v_mfma_scale_f32_16x16x128_f8f6f4 (measured on gfx950) ---------------------------------------
// D:  lane l holds column l % 16, rows 4 (l / 16) + r in its 4 registers.
// B (FP4, 4 registers): lane l holds column l % 16, positions k = 32 (l / 16) + e, nibble e = 0..31 in register order.
// A (FP8, 8 registers): lane l holds row l % 16, byte e = 0..31 in register order at position
//     k = 64 (e / 16) + 16 (l / 16) + e % 16.
// Block scales (E8M0 byte, value 2^(byte - 127)): the scale operand of lane l applies to row / column l % 16 and the
// positions 32 (l / 16) .. 32 (l / 16) + 31.
//
// Roles of a lane.  As a holder of D registers ("row role"): head hd = lane / 16 of the head block, column jd.  As a
// holder of A registers: row 4 ha + ua = (head ha, term ua), quarter ga.  The A registers are built by the lanes in
// 8-byte chunks -- chunk u of (head, quarter g) = bytes 8 u .. 8 u + 7 = positions 64 (u / 2) + 16 g + 8 (u % 2) + 0..7 --
// and handed over through LDS: the builder of (head h, quarter g, chunk u) writes its three terms at
// ex[160 h + 32 term + 2 (4 g + u)], the holder of (head h, term, quarter g) reads 8 words at ex[160 h + 32 term + 8 g].
// Term 3 of every head stays zero.  Word 128 of a head carries the block exponent where builder and holder differ.
constexpr int kExHead = 160;              // words per head in an exchange region (stride 640 B: two heads cover all banks)
constexpr int kExWords = 4 * kExHead;     // one region: 4 heads
constexpr int kExExp = 128;               // word of the block exponent

// B registers from packed words: nibble = hi|0|lo|1 = FP4 (code - 1.5).  One bit-field insert per register: the code bits of the word where `pick` has ones, the constant mantissa bit elsewhere.
// `pick` is 0xAAAAAAAA held in a scalar register (see code_bits_mask) so that the insert is a single instruction.
__device__ __forceinline__ uint32_t centred_nibbles(uint32_t w, uint32_t pick) {
  return 0x11111111u ^ (pick & (w ^ 0x11111111u));  // = (w & pick) | (0x11111111 & ~pick), in the form that selects v_bfi_b32
}
__device__ __forceinline__ uint32_t code_bits_mask() {
  uint32_t m = 0xAAAAAAAAu;
  asm volatile("" : "+s"(m));  // opaque to constant folding, so that the insert stays one instruction
  return m;
}
struct Roles {
  int lane;
  int jd, hd;      // row role
  int ua, ha, ga;  // operand role
  int c0;          // first of the 8 channels whose (q * key scale) this lane builds: chunk ua of (ha, ga)
  int wq;          // where this lane writes its chunk as a builder of q K^T operands (it builds for its own quad)
  int wp;          // ... as a builder of E V operands (it builds from the probabilities it holds in the row role)
  int rd;          // where this lane reads its operand registers
  uint32_t* ex_qk;  // this wave's exchange regions
  uint32_t* ex_pv;
  uint32_t pick;    // code_bits_mask()
};

__device__ __forceinline__ Roles make_roles(int lane, uint32_t* ex_wave) {
  Roles r;
  r.lane = lane;
  r.jd = lane & 15; r.hd = lane >> 4;
  r.ua = lane & 3; r.ha = (lane >> 2) & 3; r.ga = lane >> 4;
  r.c0 = 64 * (r.ua >> 1) + 16 * r.ga + 8 * (r.ua & 1);
  r.wq = kExHead * r.ha + 2 * (4 * r.ga + r.ua);
  r.wp = kExHead * r.hd + 2 * r.jd;
  r.rd = kExHead * r.ha + 32 * r.ua + 8 * r.ga;
  r.ex_qk = ex_wave;
  r.ex_pv = ex_wave + kExWords;
  r.pick = code_bits_mask();
  return r;
}

// x[0..7] as three FP8 terms: with sc = 2^e (sc_bits its binary32 pattern, e chosen so that |x| / sc < 256),
// t_k = fp8((x - what t_0 .. t_{k-1} stand for) / (sc / 16^k)), round to nearest even.  Every residual is exact in
// binary32 (the term agrees with it in its leading bits).  t[k][v] holds values 4 v .. 4 v + 3, lowest byte first.
__device__ __forceinline__ void split_fp8x3(const float (&x)[8], uint32_t sc_bits, uint32_t (&t)[3][2]) {
  float r[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) r[i] = x[i];
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const float sc = as_f32(sc_bits - ((uint32_t)(4 * k) << 23));
#pragma unroll
    for (int v = 0; v < 2; ++v) {
      short2_t w;
      asm volatile("" : "=v"(w));  // any free register: both halves are written below (a live value would be copied first)
      w = __builtin_amdgcn_cvt_scalef32_pk_fp8_f32(w, r[4 * v], r[4 * v + 1], sc, false);
      w = __builtin_amdgcn_cvt_scalef32_pk_fp8_f32(w, r[4 * v + 2], r[4 * v + 3], sc, true);
      const uint32_t bits = __builtin_bit_cast(uint32_t, w);
      t[k][v] = bits;
      if (k < 2) {
        const float2_t f0 = __builtin_amdgcn_cvt_scalef32_pk_f32_fp8(bits, sc, false);
        const float2_t f1 = __builtin_amdgcn_cvt_scalef32_pk_f32_fp8(bits, sc, true);
        r[4 * v] -= f0[0]; r[4 * v + 1] -= f0[1];
        r[4 * v + 2] -= f1[0]; r[4 * v + 3] -= f1[1];
      }
    }
  }
}

// Biased binary32 exponent eb of the largest magnitude of a block, from its bit pattern (kept away from the low end of
// the range), for sc = 2^(eb - 127 - 7): |x| / sc < 256, inside FP8's range.  Row `term` then carries the block scale
// byte eb - 7 - 4 term.
__device__ __forceinline__ uint32_t block_exponent(uint32_t mx_bits) { return max(mx_bits, as_bits(0x1p-100f)) >> 23; }
__device__ __forceinline__ uint32_t block_scale_bits(uint32_t eb) { return (eb - 7u) << 23; }

// Builder side of the hand-over: the three terms of this lane's chunk; holder side: the 8 operand registers.
__device__ __forceinline__ void put_terms(uint32_t* ex, int at, const uint32_t (&t)[3][2]) {
#pragma unroll
  for (int k = 0; k < 3; ++k) *reinterpret_cast<u32x2_t*>(ex + at + 32 * k) = u32x2_t{t[k][0], t[k][1]};
}
__device__ __forceinline__ v8i_t get_operand(const uint32_t* ex, int at) {
  const u32x4_t a = *reinterpret_cast<const u32x4_t*>(ex + at), b = *reinterpret_cast<const u32x4_t*>(ex + at + 4);
  return v8i_t{(int)a[0], (int)a[1], (int)a[2], (int)a[3], (int)b[0], (int)b[1], (int)b[2], (int)b[3]};
}

// D = A B + C with B = 32 centred codes per lane from two packed words (see centred_nibbles); kScaleB: the block scale
// byte of B (127 = 1, 129 = 4).
template <int kScaleB = 127>
__device__ __forceinline__ float4_t mfma_codes(v8i_t a, uint32_t w0, uint32_t w1, float4_t c, int scale_a, uint32_t pick) {
  const v8i_t b = {(int)centred_nibbles(w0, pick), (int)centred_nibbles(w0 << 1, pick), (int)centred_nibbles(w1, pick),
                   (int)centred_nibbles(w1 << 1, pick), 0, 0, 0, 0};
  return __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(a, b, c, 0 /* A: FP8 E4M3 */, 4 /* B: FP4 E2M1 */, 0, scale_a,
                                                         0, kScaleB);
}
// 4-bit codes: a tile is two planes of 2-bit codes, the base-4 digits of the codes, and
// code - 7.5 = 4 (high digit - 1.5) + (low digit - 1.5): the contraction with the codes is the contraction with the high
// plane under a block scale of 4 plus the contraction with the low plane.
__device__ __forceinline__ float4_t mfma_codes_high(v8i_t a, uint32_t w0, uint32_t w1, float4_t c, int scale_a, uint32_t pick) {
  return mfma_codes<129>(a, w0, w1, c, scale_a, pick);
}

// Register image of one group; BITS / 2 planes per tile.
template <int BITS>
struct KeyRegs {
  uint4 kw[2 * BITS];  // key tile: kw[4 plane + m] = the words of token blocks 2 m (x, y) and 2 m + 1 (z, w) for this lane's (column, quarter)
  uint4 ks, kz;  // key scale / zero-point of the 8 channels c0 .. c0 + 7 this lane builds operands for
};
template <int BITS>
struct ValueRegs {
  uint4 vw[2 * BITS];  // value tile, channel blocks 2 m and 2 m + 1 of every plane
  uint4 sz[2];  // value (scale, zero-point) pairs of tokens 16 n + jd, n = 0..7
};

// A record is fetched in two parts so that each part can be requested again for the next group as soon as its
// contraction has consumed it: the key part flies during E V, the value part during the next q K^T.
// The tiles are read once per launch and by one wave only: non-temporal loads (measured: config 2 23.7 -> 22.2 us,
// config 4 83.7 -> 77.5 us; the short contexts of config 7 lose 2 %).
__device__ __forceinline__ uint4 load_once(const uint4* p) {
  const u32x4_t t = __builtin_nontemporal_load(reinterpret_cast<const u32x4_t*>(p));
  return make_uint4(t[0], t[1], t[2], t[3]);
}
template <int BITS>
__device__ __forceinline__ void load_keys(KeyRegs<BITS>& r, const uint32_t* __restrict__ rec, const Roles& lr) {
  const uint4* kt = reinterpret_cast<const uint4*>(rec + Rec<BITS>::kKeyTile);
#pragma unroll
  for (int m = 0; m < 2 * BITS; ++m) r.kw[m] = load_once(kt + m * 64 + lr.lane);  // (the planes follow each other)
  r.ks = *reinterpret_cast<const uint4*>(reinterpret_cast<const half_t*>(rec + Rec<BITS>::kKeyScale) + lr.c0);
  r.kz = *reinterpret_cast<const uint4*>(reinterpret_cast<const half_t*>(rec + Rec<BITS>::kKeyZero) + lr.c0);
}

template <int BITS>
__device__ __forceinline__ void load_values(ValueRegs<BITS>& r, const uint32_t* __restrict__ rec, const Roles& lr) {
  const uint4* vt = reinterpret_cast<const uint4*>(rec + Rec<BITS>::kValueTile);
#pragma unroll
  for (int m = 0; m < 2 * BITS; ++m) r.vw[m] = load_once(vt + m * 64 + lr.lane);
  const uint4* sz = reinterpret_cast<const uint4*>(rec + Rec<BITS>::kValueSZ) + 2 * lr.jd;
  r.sz[0] = sz[0];
  r.sz[1] = sz[1];
}

// NB = head blocks of 4 query heads (1: up to 4 heads per KV head, 2: up to 8).  State of a wave, row role.
template <int NB>
struct WaveState {
  float m[NB];          // reference maximum of this lane's head (equal in the 16 lanes of the row), log2 domain
  float l[NB];          // per-lane partial sum of p
  float pz[NB];         // per-lane partial sum of p * (value zero-point + 1.5 value scale)
  float acc[NB][8];     // E V of channel 16 n + jd
};

template <int NB>
__device__ __forceinline__ void empty_state(WaveState<NB>& st) {
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) {
    st.m[nb] = -INFINITY; st.l[nb] = 0.f; st.pz[nb] = 0.f;
#pragma unroll
    for (int n = 0; n < 8; ++n) st.acc[nb][n] = 0.f;
  }
}

// q K^T of one group for all heads (Alg. 1 line 7): sc[nb][n] = q.k of head 4 nb + hd, token 16 n + jd (the factor
// log2(e) / sqrt(d) enters with the reference maximum, see exponent()).
// qh = this lane's 8 query values (head 4 nb + ha, channels c0 ..) in binary16 pairs.
// off[nb] = what the zero-points and the centring of the codes add to every score of the head: sc leaves it out.
// valid: tokens of the group that exist (only the newest group of a sequence may be partial; the loop over the others passes
// the constant).
template <int NB, int BITS>
__device__ __forceinline__ void qk_phase(const KeyRegs<BITS>& g, int valid, const uint32_t (&qh)[NB][4], const Roles& lr,
                                         float (&sc)[NB][8], float (&off)[NB]) {
  const uint32_t S[4] = {g.ks.x, g.ks.y, g.ks.z, g.ks.w};
  const uint32_t Z[4] = {g.kz.x, g.kz.y, g.kz.z, g.kz.w};
  v8i_t A[NB];
  int scale_a[NB];
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) {
    float x[8], bz = 0.0f, mx = 0.0f;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      x[i] = fmaf((float)as_h2(qh[nb][i >> 1])[i & 1], (float)as_h2(S[i >> 1])[i & 1], 0.0f);  // exact; the fused form reads binary16 operands as they are
      mx = fmaxf(mx, fabsf(x[i]));
    }
    // sum_c q_c (z_c + 1.5 s_c): what the zero-points and the centring of the codes add to every score of the group.
    // Mid-points and query in binary16 pairs, products summed in binary32: the term is a common offset of the
    // group's scores and small (keys are centred), its rounding (2^-12 of it) is of no account.
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const half2_t mid = as_h2(S[i]) * half2_t{(half_t)Rec<BITS>::kCentre, (half_t)Rec<BITS>::kCentre} + as_h2(Z[i]);
      bz = __builtin_amdgcn_fdot2(as_h2(qh[nb][i]), mid, bz, false);
    }
    const uint32_t eb = block_exponent(xrow_umax(quad_umax(as_bits(mx))));  // over the 128 channels of the head
    bz = xrow_allsum(quad_allsum(bz));
    uint32_t t[3][2];
    split_fp8x3(x, block_scale_bits(eb), t);
    // (two head blocks: the second one goes through the other exchange region, so that one hand-over serves both)
    put_terms(nb == 0 ? lr.ex_qk : lr.ex_pv, lr.wq, t);
    if (NB == 1) {
      lds_order();
      A[nb] = get_operand(lr.ex_qk, lr.rd);
      lds_order();
    }
    scale_a[nb] = (int)eb - 7 - 4 * lr.ua;
    // the head's zero-point term, from a lane that holds head hd in the operand role (lane 4 hd)
    off[nb] = __builtin_bit_cast(float, __builtin_amdgcn_ds_bpermute(16 * lr.hd, __builtin_bit_cast(int, bz)));
  }
  if (NB == 2) {
    lds_order();
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) A[nb] = get_operand(nb == 0 ? lr.ex_qk : lr.ex_pv, lr.rd);
    lds_order();
  }
  const float4_t zero = {0.f, 0.f, 0.f, 0.f};
  if constexpr (BITS == 2 && NB == 1) {
    // All eight matrix instructions first, each into registers of its own, then the sums of the term rows: written
    // as one loop the compiler reuses the result registers and every instruction waits for the one before (a dozen
    // idle cycles each; config 3 24.0 -> 22.9 us, config 2 21.5 -> 21.25 us; two head blocks do not gain).
    float4_t dq[8];
#pragma unroll
    for (int m = 0; m < 4; ++m) {
      const uint32_t w[4] = {g.kw[m].x, g.kw[m].y, g.kw[m].z, g.kw[m].w};
#pragma unroll
      for (int hf = 0; hf < 2; ++hf) dq[2 * m + hf] = mfma_codes(A[0], w[2 * hf], w[2 * hf + 1], zero, scale_a[0], lr.pick);
    }
#pragma unroll
    for (int n = 0; n < 8; ++n) sc[0][n] = (dq[n][0] + dq[n][1]) + dq[n][2];
  }
#pragma unroll
  for (int m = 0; m < 4; ++m) {
    const uint32_t w[4] = {g.kw[m].x, g.kw[m].y, g.kw[m].z, g.kw[m].w};
    if constexpr (BITS == 2 && NB == 1) {
    } else if constexpr (BITS == 2) {
#pragma unroll
      for (int hf = 0; hf < 2; ++hf)
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
          const float4_t d = mfma_codes(A[nb], w[2 * hf], w[2 * hf + 1], zero, scale_a[nb], lr.pick);
          sc[nb][2 * m + hf] = (d[0] + d[1]) + d[2];
        }
    } else {
      const uint32_t wl[4] = {g.kw[4 + m].x, g.kw[4 + m].y, g.kw[4 + m].z, g.kw[4 + m].w};  // low plane
      float4_t d[2][NB];
#pragma unroll
      for (int hf = 0; hf < 2; ++hf)
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) d[hf][nb] = mfma_codes_high(A[nb], w[2 * hf], w[2 * hf + 1], zero, scale_a[nb], lr.pick);
#pragma unroll
      for (int hf = 0; hf < 2; ++hf)
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
          d[hf][nb] = mfma_codes(A[nb], wl[2 * hf], wl[2 * hf + 1], d[hf][nb], scale_a[nb], lr.pick);
          sc[nb][2 * m + hf] = (d[hf][nb][0] + d[hf][nb][1]) + d[hf][nb][2];
        }
    }
  }
  if (valid < kGroup) {  // partial last group: tokens >= valid do not exist
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
      for (int n = 0; n < 8; ++n)
        if (16 * n + lr.jd >= valid) sc[nb][n] = -INFINITY;
  }
}

// Reference maximum (Alg. 1 line 8).  Any reference m works as long as 2^(x - m) stays moderate, so the reference of a
// head is only raised -- with a maximum over the row and a rescale of the accumulated state -- when some score of the
// group exceeds it by more than `slack`; most groups pay one comparison per register.  (The literal form of Alg. 1's
// last lines adds the correction to sums that are shifted by the TRUE maximum: there the slack is 0, which makes the
// reference the running maximum itself.)
constexpr float kSlack = 5.0f;
// What 2 is raised to for a score (its head's offset off apart) and the reference m: s kAlpha + base.
__device__ __forceinline__ float exponent_base(float off, float m) { return fmaf(off, kAlpha, -m); }
__device__ __forceinline__ float exponent(float s, float base) { return fmaf(s, kAlpha, base); }
// The reference is rounded in another way than the exponents, so the exponent of the largest score is not 0 but what the
// roundings of off kAlpha - m and of m leave: 1/8 at most while both stay below this bound, and beyond anything that a power
// of two can hold a few thousand times further up.
constexpr float kFusedBound = 0x1p20f;

// base[nb] = what exponent() takes with a score of the head.  Above kFusedBound (no ordinary keys and queries get there) the
// scores themselves are replaced by their distance from the reference, rounded as the reference is, and the base is 0.  (The look
// takes 0 to 0.9 % of a step: 16 sequences of 8k tokens 26.29 -> 26.36 us, one of 131072 tokens 24.95 -> 25.10 us; one branch for
// both looks takes the same.)
template <int NB>
__device__ __forceinline__ void update_reference(float (&sc)[NB][8], const float (&off)[NB], float (&base)[NB], WaveState<NB>& st, float slack) {
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) {
    float mloc = sc[nb][0];
#pragma unroll
    for (int n = 1; n < 8; ++n) mloc = fmaxf(mloc, sc[nb][n]);
    mloc = (mloc + off[nb]) * kAlpha;
    if (__builtin_amdgcn_ballot_w64(mloc > st.m[nb] + slack) != 0) {
      const float mnew = fmaxf(st.m[nb], row_allmax(mloc));
      const float f = mnew == -INFINITY ? 1.0f : exp2f(st.m[nb] - mnew);  // 0 when the old reference is -inf
      st.l[nb] *= f;
      st.pz[nb] *= f;
#pragma unroll
      for (int n = 0; n < 8; ++n) st.acc[nb][n] *= f;
      st.m[nb] = mnew;
    }
    base[nb] = exponent_base(off[nb], st.m[nb]);
    if (__builtin_amdgcn_ballot_w64(fmaxf(fabsf(base[nb]), fabsf(st.m[nb])) > kFusedBound) != 0) {
#pragma clang fp contract(off)
#pragma unroll
      for (int n = 0; n < 8; ++n) sc[nb][n] = ((sc[nb][n] + off[nb]) * kAlpha - st.m[nb]) * (1.0f / kAlpha);
      base[nb] = 0.0f;
    }
  }
}

// p = 2^(x - m), its sums, and E V of one group (Alg. 1 lines 9-10).  MASKED: tokens from `fp16_from` on count in the
// sums of p but not in E V: their values are taken from the fp16 window (pv_window_tail).
template <int NB, int BITS, bool MASKED = false>
__device__ __forceinline__ void pv_phase(const ValueRegs<BITS>& g, const float (&sc)[NB][8], const float (&base)[NB], const Roles& lr,
                                         WaveState<NB>& st, int fp16_from = kGroup) {
  const uint32_t SZ[8] = {g.sz[0].x, g.sz[0].y, g.sz[0].z, g.sz[0].w, g.sz[1].x, g.sz[1].y, g.sz[1].z, g.sz[1].w};
  v8i_t A[NB];
  int scale_a[NB];
  // z + 1.5 s of the lane's tokens: what the zero-point and the centring of the codes give for every channel
  float mid[8];
#pragma unroll
  for (int n = 0; n < 8; ++n) mid[n] = fmaf((float)as_h2(SZ[n])[0], Rec<BITS>::kCentre, (float)as_h2(SZ[n])[1]);
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) {
    float y[8], mx = 0.0f;
#pragma unroll
    for (int n = 0; n < 8; ++n) {
      const float p = __builtin_amdgcn_exp2f(exponent(sc[nb][n], base[nb]));
      const half2_t sz = as_h2(SZ[n]);
      st.l[nb] += p;
      const bool coded = !MASKED || 16 * n + lr.jd < fp16_from;
      y[n] = coded ? fmaf(p, (float)sz[0], 0.0f) : 0.0f;  // p * value scale: the weight of the token's codes
      st.pz[nb] = coded ? fmaf(p, mid[n], st.pz[nb]) : st.pz[nb];
      mx = fmaxf(mx, y[n]);
    }
    const uint32_t eb = block_exponent(row_umax(as_bits(mx)));  // over the 128 tokens of the head
    uint32_t t[3][2];
    split_fp8x3(y, block_scale_bits(eb), t);
    uint32_t* region = nb == 0 ? lr.ex_pv : lr.ex_qk;
    put_terms(region, lr.wp, t);
    region[kExHead * lr.hd + kExExp] = eb;  // the same value from the 16 lanes of the row
    if (NB == 1) {
      lds_order();
      A[nb] = get_operand(lr.ex_pv, lr.rd);
      scale_a[nb] = (int)lr.ex_pv[kExHead * lr.ha + kExExp] - 7 - 4 * lr.ua;
      lds_order();
    }
  }
  if (NB == 2) {
    lds_order();
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
      const uint32_t* region = nb == 0 ? lr.ex_pv : lr.ex_qk;
      A[nb] = get_operand(region, lr.rd);
      scale_a[nb] = (int)region[kExHead * lr.ha + kExExp] - 7 - 4 * lr.ua;
    }
    lds_order();
  }
  // Every instruction starts from zero and its three term rows are added to the state at once: one register per channel
  // and head block instead of four (NB = 1: 8 for 32) for three additions, and the sum over the groups is rounded like
  // any binary32 sum rather than truncated by the matrix cores' adder.
#pragma unroll
  for (int m = 0; m < 4; ++m) {
    const uint32_t w[4] = {g.vw[m].x, g.vw[m].y, g.vw[m].z, g.vw[m].w};
    float4_t d[2][NB];
#pragma unroll
    for (int hf = 0; hf < 2; ++hf)
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) {
        const float4_t zero = {0.f, 0.f, 0.f, 0.f};
        d[hf][nb] = BITS == 2 ? mfma_codes(A[nb], w[2 * hf], w[2 * hf + 1], zero, scale_a[nb], lr.pick)
                              : mfma_codes_high(A[nb], w[2 * hf], w[2 * hf + 1], zero, scale_a[nb], lr.pick);
      }
    if constexpr (BITS == 4) {  // the low plane
      const uint32_t wl[4] = {g.vw[4 + m].x, g.vw[4 + m].y, g.vw[4 + m].z, g.vw[4 + m].w};
#pragma unroll
      for (int hf = 0; hf < 2; ++hf)
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) d[hf][nb] = mfma_codes(A[nb], wl[2 * hf], wl[2 * hf + 1], d[hf][nb], scale_a[nb], lr.pick);
    }
#pragma unroll
    for (int hf = 0; hf < 2; ++hf)
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) st.acc[nb][2 * m + hf] += (d[hf][nb][0] + d[hf][nb][1]) + d[hf][nb][2];
  }
}

// The values that pv_window_tail will read, one word of every line of 128 bytes, requested while the scores of the group are formed:
// nobody else reads these slots (the window's share ends at its live tokens), and the trip to memory would come after everything.
constexpr int kWindowLines = kGroup * kHeadDim * 2 / 128;  // R is kGroup where values slide
__device__ __forceinline__ void touch_window_tail(uint32_t (&touched)[kWindowLines / 64], const half_t* __restrict__ v_win, int from, int lane) {
#pragma unroll
  for (int u = 0; u < kWindowLines / 64; ++u)
    touched[u] = reinterpret_cast<const uint32_t*>(v_win)[32 * min(8 * (from >> 2) + 64 * u + lane, kWindowLines - 1)];
}

// Sliding value window (Sec. 4.1, setup: the newest 128 tokens in full precision): the tokens j >= from of the newest
// group still have their fp16 rotated values in the window slots j.  Their share of E V is formed here from those values
// by the one wave that has the newest group, on v_mfma_f32_4x4x4_16B_f16: rows = the 4 heads of a head
// block, columns = 64 channels (lane = channel), k = 4 window slots, the probabilities (binary16, through LDS) broadcast
// from one lane quad per block of 4 slots.  The result is added to the accumulators by way of `out`, this wave's
// [NB * 4][128] slice of the combine buffer.
template <int NB>
__device__ __forceinline__ void pv_window_tail(const half_t* __restrict__ v_win, const float (&sc)[NB][8], const float (&base)[NB], int from,
                                               const Roles& lr, WaveState<NB>& st, int lane, float (*out)[kHeadDim]) {
  half_t* pb = reinterpret_cast<half_t*>(lr.ex_pv);  // [NB * 4 heads][128 tokens]
#pragma unroll
  for (int nb = 0; nb < NB; ++nb)
#pragma unroll
    for (int n = 0; n < 8; ++n) {
      const int j = 16 * n + lr.jd;
      pb[(nb * 4 + lr.hd) * kGroup + j] = j >= from ? (half_t)__builtin_amdgcn_exp2f(exponent(sc[nb][n], base[nb])) : (half_t)0.0f;
    }
  lds_order();
  const int quad = lane >> 2, hrow = lane & 3;
  half4_t A[NB][2];
#pragma unroll
  for (int nb = 0; nb < NB; ++nb)
#pragma unroll
    for (int hf = 0; hf < 2; ++hf) A[nb][hf] = *reinterpret_cast<const half4_t*>(pb + (nb * 4 + hrow) * kGroup + 64 * hf + 4 * quad);
  const uint2* vb = reinterpret_cast<const uint2*>(v_win);  // [slot / 4][channel] -> 4 slots
  // (blocks requested together: with 16 two head blocks at 4 bits spilled 30 registers, with 4 two)
  constexpr int kBlocks = NB == 2 ? 4 : 16;
  const int first = from >> 2;                              // blocks of 4 slots below it hold no such token
  float4_t acc[NB][2];
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) acc[nb][0] = acc[nb][1] = float4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int part = 0; part < kGroup / 4 / kBlocks; ++part) {
    uint2 vx[2][kBlocks];
#pragma unroll
    for (int bq = 0; bq < kBlocks; ++bq)
#pragma unroll
      for (int ch = 0; ch < 2; ++ch) {
        const int blk = kBlocks * part + bq;
        vx[ch][bq] = blk >= first ? vb[(long long)blk * kHeadDim + 64 * ch + lane] : make_uint2(0, 0);
      }
#pragma unroll
    for (int bq = 0; bq < kBlocks; ++bq)
#pragma unroll
      for (int ch = 0; ch < 2; ++ch) {
        const half4_t bop = as_h4(vx[ch][bq].x, vx[ch][bq].y);
        const int blk = kBlocks * part + bq;
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) acc[nb][ch] = mfma_bcast(A[nb][blk / 16], bop, acc[nb][ch], blk % 16);
      }
    asm volatile("" ::: "memory");  // (the next blocks' loads stay behind these products)
  }
  // (lane = channel, registers = heads) -> (row = head, lane = channel % 16, register = channel block n)
#pragma unroll
  for (int nb = 0; nb < NB; ++nb)
#pragma unroll
    for (int h = 0; h < 4; ++h) {
      out[nb * 4 + h][lane] = acc[nb][0][h];
      out[nb * 4 + h][64 + lane] = acc[nb][1][h];
    }
  lds_order();
#pragma unroll
  for (int nb = 0; nb < NB; ++nb)
#pragma unroll
    for (int n = 0; n < 8; ++n) st.acc[nb][n] += out[nb * 4 + lr.hd][16 * n + lr.jd];
  lds_order();
  // the spare term row of every head of this exchange region reads as zero again
  uint32_t* ex = reinterpret_cast<uint32_t*>(lr.ex_pv);
  for (int i = lane; i < 4 * 32; i += 64) ex[(i >> 5) * kExHead + 96 + (i & 31)] = 0u;
  lds_order();
}

// ---- a wave's share of the fp16 window as one more block of tokens (raw keys, rotated values) -----------------------------
// On v_mfma_f32_16x16x32_f16, in the row role of the groups: D register nb of lane (hd, jd) is head 4 nb + hd, row 4 hd + nb of
// the A operand; the other rows are zero.
//   q K^T : columns = 16 tokens, positions = 32 channels: step kk takes from lane (hd, jd) the channels
//           64 (kk / 2) + 16 hd + 8 (kk % 2) + 0..7 of token 16 tt + jd, which is what the lanes of a quad hold of q in the operand
//           role (lane kk of the quad), so that A comes from qh by broadcasts inside the quads;
//   E V   : columns = 16 channels, positions = 32 tokens: lane (hd, jd) has tokens 8 hd + 0..7, two 4-slot pieces of v_res.
// Runs before the wave's first group, on empty state.  Bound: latency and, where many short sequences fill the chip, bytes: what
// lies beyond the window's tokens is not read (lanes without a token take the last one's rows).
// Two waves with 64 tokens each, on the 4x4x4 blocks, waited for their first record, then for the keys (each a 16-byte piece of
// 64 lines, in 16 instructions), then for the values, then for q.  Steps before and after (with the requests laid out as they are in
// the kernel below): 144 sequences of 1280 tokens 70.7 -> 64.0 us, 32 x 32 single heads of 1280 45.4 -> 42.0, one sequence of
// 131072 24.4 -> 22.8, of 300 11.8 -> 10.9 (of which the host's two calls take 9.7), 16 of 8k 25.1 -> 24.5, 32 of 32k with 7 heads
// 75.6 -> 72.4.
struct WindowShare {
  int first, end;  // tokens first .. end - 1, at most 32 and first a multiple of 4; none: end <= first
};
// k of the waves share, the last ones: as many as have no group in the last round of a sequence with one split (count: its groups),
// as many as are needed, or all.  (Four waves always, and the whole window requested ahead of the counters in small launches: 0.9265
// instead of 0.9200 of the time of two waves with 64 tokens each, on average over some 4900 decode launches.)
__device__ __forceinline__ WindowShare window_share(int nr, int count, bool one_split, int wave) {
  int k = one_split ? -count & (kWaves - 1) : 0;
  k = max(k == 0 ? kWaves : k, (nr + 31) / 32);
  const int fours = (nr + 3) / 4;  // at most 32: exact below
  const int per = 4 * (k == 4 ? (fours + 3) >> 2 : k == 3 ? ((fours + 2) * 171) >> 9 : k == 2 ? (fours + 1) >> 1 : fours);
  const int at = per * (wave - (kWaves - k));
  return WindowShare{max(at, 0), min(at + per, nr)};  // (at < 0: empty, for at + per <= 0)
}
struct WindowRegs {
  uint4 k[2][4];  // [tt][kk]
  uint4 v[8];     // [channel block]: slots 8 hd + 0..3 (x, y) and + 4..7 (z, w)
};
__device__ __forceinline__ void request_window(WindowRegs& w, const kvlinc_cache& c, int bh, const WindowShare& sh, const Roles& lr) {
  const half_t* keys = reinterpret_cast<const half_t*>(c.k_res) + (long long)bh * c.R * kHeadDim;
  const uint2* vb = reinterpret_cast<const uint2*>(reinterpret_cast<const half_t*>(c.v_res) + (long long)bh * c.R * kHeadDim) + lr.jd;
  const int last = max(sh.end - 1, 0);
#pragma unroll
  for (int tt = 0; tt < 2; ++tt) {
    const uint4* krow = reinterpret_cast<const uint4*>(keys + min(sh.first + 16 * tt + lr.jd, last) * kHeadDim);
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) w.k[tt][kk] = krow[8 * (kk >> 1) + 2 * lr.hd + (kk & 1)];
  }
  const int u = sh.first / 4 + 2 * lr.hd;
  const uint2 *v0 = vb + min(u, last >> 2) * kHeadDim, *v1 = vb + min(u + 1, last >> 2) * kHeadDim;
#pragma unroll
  for (int n = 0; n < 8; ++n) {
    const uint2 a = v0[16 * n], b = v1[16 * n];
    w.v[n] = make_uint4(a.x, a.y, b.x, b.y);
  }
}

// The share is not empty: the maxima are finite.
template <int NB>
__device__ __forceinline__ void window_part(const WindowRegs& w, const uint32_t (&qh)[NB][4], const WindowShare& sh, const Roles& lr, WaveState<NB>& st) {
  float4_t d[2];
  d[0] = d[1] = float4_t{0.f, 0.f, 0.f, 0.f};
  const uint32_t row0 = lr.ua == 0 ? ~0u : 0u, row1 = lr.ua == 1 ? ~0u : 0u;
#pragma unroll
  for (int kk = 0; kk < 4; ++kk) {
    const auto from_quad = [&](uint32_t v) { return kk == 0 ? dpp_u<0x00>(v) : kk == 1 ? dpp_u<0x55>(v) : kk == 2 ? dpp_u<0xAA>(v) : dpp_u<0xFF>(v); };
    uint32_t a[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      a[i] = from_quad(qh[0][i]) & row0;
      if (NB == 2) a[i] |= from_quad(qh[NB - 1][i]) & row1;
    }
    const half8_t A = __builtin_bit_cast(half8_t, make_uint4(a[0], a[1], a[2], a[3]));
#pragma unroll
    for (int tt = 0; tt < 2; ++tt) d[tt] = __builtin_amdgcn_mfma_f32_16x16x32_f16(A, __builtin_bit_cast(half8_t, w.k[tt][kk]), d[tt], 0, 0, 0);
  }
  half_t* pb = reinterpret_cast<half_t*>(lr.ex_pv);  // head 4 nb + hd: 32 halves at words 160 hd + 16 nb (clear of the spare term rows)
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) {
    float sc[2];
#pragma unroll
    for (int tt = 0; tt < 2; ++tt) sc[tt] = sh.first + 16 * tt + lr.jd < sh.end ? d[tt][nb] * kAlpha : -INFINITY;
    const float m = row_allmax(fmaxf(sc[0], sc[1]));
    float p[2];
#pragma unroll
    for (int tt = 0; tt < 2; ++tt) {
      p[tt] = __builtin_amdgcn_exp2f(sc[tt] - m);
      pb[2 * (kExHead * lr.hd + 16 * nb) + 16 * tt + lr.jd] = (half_t)p[tt];
    }
    st.m[nb] = m;
    st.l[nb] = p[0] + p[1];
    st.pz[nb] = 0.0f;
  }
  lds_order();
  const uint4 t = *reinterpret_cast<const uint4*>(pb + 2 * (kExHead * lr.ha + 16 * min(lr.ua, NB - 1)) + 8 * lr.hd);
  const half8_t A = __builtin_bit_cast(half8_t, lr.ua < NB ? t : make_uint4(0, 0, 0, 0));
  lds_order();
#pragma unroll
  for (int n = 0; n < 8; ++n) {
    const float4_t zero = {0.f, 0.f, 0.f, 0.f};
    const float4_t e = __builtin_amdgcn_mfma_f32_16x16x32_f16(A, __builtin_bit_cast(half8_t, w.v[n]), zero, 0, 0, 0);
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) st.acc[nb][n] = e[nb];
  }
}

// ---- correction terms (Sec. 3.3: C_n = phi_q(q) S, C_d = phi_q(q) P; Eq. 6 for phi) -----------------------------------
// The work of a kv head is cut into kCorrParts parts over the rows of S: part r covers the kPartFeat features
// kPartFeat (r % kPartsPerHalf) .. of half hs = r / kPartsPerHalf of phi.  A correction workgroup serves one part
// for 1, 2, 4 or 8 sequences, on the matrix cores:
//   phase 1, wave w = query head w of a block of four: logits[s][f] = sum_c q[s][c] W[c][f] on v_mfma_f32_16x16x32_f16 with
//            the sequences s as rows and features as columns.  The W rows are read in their natural order: a lane takes 4
//            neighbouring features of the 8 channels whose products it feeds, so that the B operands of 4 column tiles
//            (feature 4 (lane % 16) + i in tile i) are byte permutations of its own registers.
//   phase 2, wave w = sequences w, w + 4, ..., or, of one or two sequences, the channel half w % 2 of sequence w / 2:
//            e_f = exp(logit_f - m_r) with the part's own maximum m_r, Z_r = sum_f e_f, Cd_r = sum_f e_f P[f], and Cn_r = e S
//            on the 4x4x4 blocks with the 4 heads as rows, block = 4 channels, k = 4 features (kPartSteps steps per channel
//            half), S taken from its binary16 tile copy.
// Output per (query head, part): {Cd_r, m_r, Z_r, -, Cn_r[128]}; the softmax normalisation of each half of phi over
// its parts is left to the merge.
// Bound: latency, a chain of loads, two products and a hand-over.  Phase 1 on the 4x4x4 blocks took a transpose inside lane quads
// (8 vector instructions a load, 256 a wave) and a chain of 32 dependent products where it now takes 64 byte permutations and 4
// chains of 4; the reductions of phase 2 went through LDS; W, needed first, came behind the S tiles; and with fewer than 4 heads
// the other waves waited.  Step (append and decode), before and after: 1 sequence of 300 tokens 14.3 -> 12.7 us, 16 of 8k
// 26.3 -> 25.9, 144 of 1280 81.6 -> 75.0; 32 sequences of 32 single heads 50.7 -> 46.5.  Requesting all S tiles ahead of the
// first product, or ahead of W, gained nothing and spilled with two head blocks.

// Workgroup barrier for data exchanged through LDS by ordinary LDS writes.
__device__ __forceinline__ void barrier_lds_only() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

constexpr int kCorrParts = 4;
constexpr int kPartFeat = 256 / kCorrParts;  // features per part
constexpr int kPartSteps = kPartFeat / 4;    // feature steps per part
constexpr int kPartsPerHalf = kCorrParts / 2;
static_assert(kPartFeat == 64, "a row of 16 lanes takes the features of a part, four each");
constexpr int kMaxCorrSeqs = 8;  // sequences a correction workgroup may serve, at most the 16 rows of its matrix products
// binary16 tile copy of S: tile (part r, channel half hh, feature step fs) holds, for lane = 4 blk + j, the 4 halves
// S[64 r + 4 fs + k][64 hh + lane], k = 0..3: what lane (blk, j) feeds as B operand of that step.
constexpr int kStateTileHalfs = 256;  // halves per tile (64 lanes x 4)
// r64 = 64-feature block of S (0..3), hh = channel half, fs = feature step inside the block (0..15)
__device__ __forceinline__ long long state_tile(int r64, int hh, int fs) { return ((r64 * 2 + hh) * 16 + fs) * kStateTileHalfs; }

// over the 16 lanes that share lane & 3
__device__ __forceinline__ float quadgroup_allmax(float v) {
  v = fmaxf(v, dpp_f<kRowRor4>(v));
  v = fmaxf(v, dpp_f<kRowRor8>(v));
  float x, y;
  pair_across<16>(v, x, y);
  pair_across<32>(fmaxf(x, y), x, y);
  return fmaxf(x, y);
}
__device__ __forceinline__ float quadgroup_allsum(float v) {
  v += dpp_f<kRowRor4>(v);
  v += dpp_f<kRowRor8>(v);
  float x, y;
  pair_across<16>(v, x, y);
  pair_across<32>(x + y, x, y);
  return x + y;
}

// Phase 1 for one head: channels 32 kk .. + 31 for the KS steps kk from k0 on.  logits: [sequence][..][kPartFeat], `stride` floats
// from one sequence to the next, this head's first.
template <int KS>
struct CorrWeights {
  uint2 w[KS][8];
  half8_t q[KS];
};
template <int KS>
__device__ __forceinline__ void request_weights(CorrWeights<KS>& x, const half_t* __restrict__ W0, const half_t* __restrict__ q0, int k0, int lane) {
  const int l16 = lane & 15, kq = lane >> 4;
#pragma unroll
  for (int kk = 0; kk < KS; ++kk) {
    x.q[kk] = *reinterpret_cast<const half8_t*>(q0 + 32 * (k0 + kk) + 8 * kq);
#pragma unroll
    for (int i = 0; i < 8; ++i)
      x.w[kk][i] = *reinterpret_cast<const uint2*>(W0 + (32 * (k0 + kk) + 8 * kq + i) * (kRank / 2) + 4 * l16);
  }
}
template <int KS>
__device__ __forceinline__ void part_logits(const CorrWeights<KS>& x, int n_seq, int stride, float* logits, int lane) {
  const int l16 = lane & 15, kq = lane >> 4;
  float4_t d[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) d[i] = float4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int kk = 0; kk < KS; ++kk)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      uint32_t b[4];
#pragma unroll
      for (int p = 0; p < 4; ++p) {
        const uint2 lo = x.w[kk][2 * p], hi = x.w[kk][2 * p + 1];
        b[p] = __builtin_amdgcn_perm(i < 2 ? hi.x : hi.y, i < 2 ? lo.x : lo.y, (i & 1) == 0 ? 0x05040100u : 0x07060302u);
      }
      d[i] = __builtin_amdgcn_mfma_f32_16x16x32_f16(x.q[kk], __builtin_bit_cast(half8_t, make_uint4(b[0], b[1], b[2], b[3])), d[i], 0, 0, 0);
    }
#pragma unroll
  for (int r = 0; r < 4; ++r)
    if (4 * kq + r < n_seq) *reinterpret_cast<float4*>(logits + (4 * kq + r) * stride + 4 * l16) = make_float4(d[0][r], d[1][r], d[2][r], d[3][r]);
}

// sLogit: [n_seq][4 n_head_blocks][kPartFeat] floats of LDS.
// FEW_HEADS: fewer than 4 query heads per kv head (one head block); the waves whose head does not exist then take a share of
// the channels of the others, and the sums over the shares are left to phase 2.  (A variant of its own, down to the kernel: a
// second copy of this function in one kernel costs that kernel registers.)
template <bool FEW_HEADS, int NB>
__device__ __forceinline__ void correction_workgroup(const kvlinc_cache& c, const half_t* __restrict__ q,
                                                     float* __restrict__ corr, int gq, int g, int r, int b_first,
                                                     int n_seq, int lane, int wave, float* sLogit) {
  const int hs = r / kPartsPerHalf, fpart = kPartFeat * (r % kPartsPerHalf);  // features 128 hs + fpart ..
  const int blk = lane >> 2, j = lane & 3;
  const half_t* Wq = reinterpret_cast<const half_t*>(c.Wq);
  const half_t* S16 = reinterpret_cast<const half_t*>(c.S16);
  constexpr int kRows = 4 * NB;  // logit rows of a sequence
  auto w_of = [&](int h) { return Wq + ((((long long)g * gq + h) * 2 + hs) * kHeadDim) * (kRank / 2) + fpart; };
  auto q_of = [&](int h) { return q + ((long long)(b_first + min(lane & 15, n_seq - 1)) * c.H_q + g * gq + h) * kHeadDim; };
  // One or two sequences: two waves share each, a channel half a wave; otherwise a wave takes whole sequences.
  const bool halves = n_seq <= 2;
  const int s_first = halves ? wave >> 1 : wave, s_step = halves ? 2 : kWaves, hh_first = halves ? wave & 1 : 0;
  // S tiles and P of the wave's sequence
  uint2 sreg[2][kPartSteps];
  float4 p4;
  auto request_state = [&](int s, int hh) {  // (hh: first or second of the wave's channel halves)
    const long long bh = (long long)(b_first + min(s, n_seq - 1)) * c.H_kv + g;
    const half_t* tiles = S16 + bh * kRank * kHeadDim + state_tile(r, halves ? hh_first : hh, 0) + 4 * lane;
#pragma unroll
    for (int fs = 0; fs < kPartSteps; ++fs) sreg[hh][fs] = *reinterpret_cast<const uint2*>(tiles + fs * kStateTileHalfs);
    if (hh == 0) p4 = *reinterpret_cast<const float4*>(c.P + bh * kRank + kPartFeat * r + 4 * blk);
  };
  int n_shares = 1;  // shares of the channels that the logits are in
  if constexpr (FEW_HEADS) {
    if (gq == 1) {
      n_shares = 4;
      CorrWeights<1> x;
      request_weights<1>(x, w_of(0), q_of(0), wave, lane);
      request_state(s_first, 0);
      part_logits<1>(x, n_seq, 4 * kPartFeat, sLogit + wave * kPartFeat, lane);
    } else if (gq == 2) {
      n_shares = 2;
      CorrWeights<2> x;
      request_weights<2>(x, w_of(wave >> 1), q_of(wave >> 1), 2 * (wave & 1), lane);
      request_state(s_first, 0);
      part_logits<2>(x, n_seq, 4 * kPartFeat, sLogit + wave * kPartFeat, lane);
    } else {
      CorrWeights<4> x;
      if (wave < gq) request_weights<4>(x, w_of(wave), q_of(wave), 0, lane);
      request_state(s_first, 0);
      if (wave < gq) part_logits<4>(x, n_seq, 4 * kPartFeat, sLogit + wave * kPartFeat, lane);
    }
  } else {
#pragma unroll
    for (int hb = 0; hb < NB; ++hb) {
      const int h = min(hb * 4 + wave, gq - 1);
      CorrWeights<4> x;
      request_weights<4>(x, w_of(h), q_of(h), 0, lane);
      if (hb == NB - 1) request_state(s_first, 0);
      part_logits<4>(x, n_seq, kRows * kPartFeat, sLogit + (hb * 4 + wave) * kPartFeat, lane);
    }
  }
  if (!halves) request_state(s_first, 1);
  barrier_lds_only();
  // ---- phase 2: the wave's sequences in turn, the four heads of a block; lane = (feature step fs = blk, head j) ----
  for (int s = s_first; s < n_seq; s += s_step) {
    half4_t aop[NB];
    float cd[NB], mx[NB], z[NB];
#pragma unroll
    for (int hb = 0; hb < NB; ++hb) {
      const float* row = sLogit + (long long)s * kRows * kPartFeat + 4 * blk;
      float4 l4;
      if (FEW_HEADS && n_shares > 1) {
        const int first = n_shares * min(j, gq - 1);  // (rows of heads that do not exist: a copy, nothing of which is stored)
        l4 = *reinterpret_cast<const float4*>(row + first * kPartFeat);
        for (int i = 1; i < n_shares; ++i) {
          const float4 t = *reinterpret_cast<const float4*>(row + (first + i) * kPartFeat);
          l4.x += t.x; l4.y += t.y; l4.z += t.z; l4.w += t.w;
        }
      } else {
        l4 = *reinterpret_cast<const float4*>(row + (hb * 4 + (FEW_HEADS ? min(j, gq - 1) : j)) * kPartFeat);
      }
      mx[hb] = quadgroup_allmax(fmaxf(fmaxf(l4.x, l4.y), fmaxf(l4.z, l4.w)));
      const float e0 = __expf(l4.x - mx[hb]), e1 = __expf(l4.y - mx[hb]), e2 = __expf(l4.z - mx[hb]), e3 = __expf(l4.w - mx[hb]);
      z[hb] = quadgroup_allsum((e0 + e1) + (e2 + e3));
      cd[hb] = quadgroup_allsum(fmaf(e0, p4.x, fmaf(e1, p4.y, fmaf(e2, p4.z, e3 * p4.w))));
      aop[hb] = half4_t{(half_t)e0, (half_t)e1, (half_t)e2, (half_t)e3};
    }
    const bool more = s + s_step < n_seq;  // (never with halves)
    float4_t acc[NB][2];
#pragma unroll
    for (int hh = 0; hh < 2; ++hh) {
      if (hh == 1 && halves) break;
      // (two chains per channel half)
#pragma unroll
      for (int hb = 0; hb < NB; ++hb) {
        float4_t a0 = {0.f, 0.f, 0.f, 0.f}, a1 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int fs = 0; fs < kPartSteps; fs += 2) {
          a0 = mfma_bcast(aop[hb], __builtin_bit_cast(half4_t, sreg[hh][fs]), a0, fs);
          a1 = mfma_bcast(aop[hb], __builtin_bit_cast(half4_t, sreg[hh][fs + 1]), a1, fs + 1);
        }
        acc[hb][hh] = a0 + a1;
      }
      if (more) request_state(s + s_step, hh);
    }
    const int b = b_first + s;
#pragma unroll
    for (int hb = 0; hb < NB; ++hb) {
      float* out0 = corr + ((long long)b * c.H_q + g * gq + hb * 4) * kCorrParts * kPartStride;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        if (hb * 4 + i < gq) {
          float* dst = out0 + ((long long)i * kCorrParts + r) * kPartStride;
          st_coherent(dst + 4 + 64 * hh_first + lane, acc[hb][0][i]);
          if (!halves) st_coherent(dst + 4 + 64 + lane, acc[hb][1][i]);
        }
      }
      if (hh_first == 0 && blk == 0 && hb * 4 + j < gq) {
        float* dst = out0 + ((long long)j * kCorrParts + r) * kPartStride;
        st_coherent(dst, cd[hb]);
        st_coherent(dst + 1, mx[hb]);
        st_coherent(dst + 2, z[hb]);
      }
    }
  }
}

// ---- merge the splits of one (sequence, query head), add the correction, rotate back (Alg. 1 lines 13-15; Eq. 5;
// Sec. 3.1).  Run by one wave of the split that arrives last. ----------------------------------------------------------

// The parts of each half of phi share one softmax: phi_f = e_f exp(m_r - M_hs) / Z_hs.  N channels a lane: cn += their C_n, cd += C_d.
// p[r] = {Cd_r, m_r, Z_r, -}, x[r] = the lane's channels of Cn_r.
template <int N>
__device__ __forceinline__ void add_correction(const u32x4_t (&p)[kCorrParts], const float (&x)[kCorrParts][N], float (&cn)[N], float& cd) {
#pragma unroll
  for (int hs = 0; hs < 2; ++hs) {
    float zsum = 0.f, Mh = -INFINITY;
#pragma unroll
    for (int i = 0; i < kPartsPerHalf; ++i) {
      zsum += as_f32(p[kPartsPerHalf * hs + i][2]);
      Mh = fmaxf(Mh, as_f32(p[kPartsPerHalf * hs + i][1]));
    }
    float zz = 0.f, xx[N], dd = 0.f;
#pragma unroll
    for (int c = 0; c < N; ++c) xx[c] = 0.f;
#pragma unroll
    for (int i = 0; i < kPartsPerHalf; ++i) {
      const int rr = kPartsPerHalf * hs + i;
      const float wgt = __expf(as_f32(p[rr][1]) - Mh);
      zz = fmaf(wgt, as_f32(p[rr][2]), zz);
      dd = fmaf(wgt, as_f32(p[rr][0]), dd);
#pragma unroll
      for (int c = 0; c < N; ++c) xx[c] = fmaf(wgt, x[rr][c], xx[c]);
    }
    const float inv = 1.0f / zz;
    const bool any = zsum > 0.f;  // (selected, not multiplied away: what is left out may not be a number)
    cd = any ? fmaf(dd, inv, cd) : cd;
#pragma unroll
    for (int c = 0; c < N; ++c) cn[c] = any ? fmaf(xx[c], inv, cn[c]) : cn[c];
  }
}
// (num + 2^-M C_n) / (den + 2^-M C_d), M the log2-domain maximum, with both sums scaled by 2^M but not below 2^-64 (den counts the
// maximum itself as 1; C_d and C_n stay in range under a factor of 2^64, and the divisor is a normal number however little is added);
// where nothing is added (C_d = 0) the factor cancels and is left out.  (Scaled by 2^min(M, 0) the reciprocal overflowed, and
// in the end the divisor was zero, for rows whose logits are all below -88 and to which next to nothing is added.)  The literal
// form of Alg. 1's last lines leaves the factor 2^-M out.  M = -inf: no tokens, 0.
template <int N>
__device__ __forceinline__ void normalise(float (&n)[N], float den, const float (&cn)[N], float cd, float M, bool literal) {
  const float Ms = fmaxf(M, -64.f);
  float fa = literal ? 1.0f : exp2f(M - Ms);
  const float fb = literal ? 1.0f : exp2f(-Ms);
  fa = cd != 0.f ? fa : 1.0f;
  const float inv = M != -INFINITY ? 1.0f / (fa * den + fb * cd) : 0.f;
#pragma unroll
  for (int c = 0; c < N; ++c) n[c] = M != -INFINITY ? (fa * n[c] + fb * cn[c]) * inv : 0.f;
}
constexpr float kRotation = 0.08838834764831845f;  // 1 / sqrt(128)
constexpr int kPartBytes = kPartStride * 4;

// More than kPairSplits splits: a row a wave.
// Lane j holds (m, l) of split j, so that the weights of all splits come from one load and one reduction; the rows are
// requested all at once, two splits per load, 16 bytes a lane.  (A walk over the splits in batches of 8 that each waited for
// their own m took 4.5 us for the 30 splits of a sequence of 131072 tokens; a step 27.6 -> 25.0 us.)
// NP: loads, at least n_splits / 2.  Lane l ends up with the channels 4 (l % 32) + 2 (l / 32), + 1.
// p0: the row's partial results, n_splits of kPartStride floats; corr: of all rows.
template <int NP>
__device__ __forceinline__ void merge_row(const float* __restrict__ p0, const float* __restrict__ corr, int n_splits, int row, int lane,
                                          bool literal, half_t* __restrict__ out) {
  const int half = lane >> 5, ch0 = 4 * (lane & 31) + 2 * half;
  u32x4_t cp[kCorrParts];
  float cx[kCorrParts][2];
  if (corr != nullptr) {  // (first: their values are needed last)
    const float* cr = corr + (long long)row * kCorrParts * kPartStride;
    const __amdgpu_buffer_rsrc_t parts = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(cr), 0, kCorrParts * kPartBytes, 0x00027000);
#pragma unroll
    for (int r = 0; r < kCorrParts; ++r) {
      cp[r] = __builtin_amdgcn_raw_buffer_load_b128(parts, r * kPartBytes, 0, kCoherentLoad);
      const float2 xy = ld_coherent2(cr + r * kPartStride + 4 + ch0);
      cx[r][0] = xy.x; cx[r][1] = xy.y;
    }
  }
  const float2 ml = ld_coherent2(p0 + (long long)min(lane, n_splits - 1) * kPartStride);
  u32x4_t a[NP];
  const __amdgpu_buffer_rsrc_t rows = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(p0), 0, n_splits * kPartBytes, 0x00027000);
#pragma unroll
  for (int k = 0; k < NP; ++k)
    a[k] = __builtin_amdgcn_raw_buffer_load_b128(rows, min(2 * k + half, n_splits - 1) * kPartBytes + 16 + 16 * (lane & 31), 0, kCoherentLoad);
  // (the lanes beyond n_splits hold a copy of the last split: its m does not change the maximum, its weight is cleared)
  const float M = wave_allmax(ml.x);
  const float w = lane < n_splits && ml.x != -INFINITY ? exp2f(ml.x - M) : 0.f;
  const float den = wave_allsum(w * ml.y);
  float n[4] = {0.f, 0.f, 0.f, 0.f}, y[2];
#pragma unroll
  for (int k = 0; k < NP; ++k) {
    const float w0 = as_f32(__builtin_amdgcn_readlane(as_bits(w), 2 * k)), w1 = as_f32(__builtin_amdgcn_readlane(as_bits(w), 2 * k + 1));
    const float wk = half != 0 ? w1 : w0;
#pragma unroll
    for (int i = 0; i < 4; ++i) n[i] = fmaf(wk, as_f32(a[k][i]), n[i]);
  }
  // the even splits of the lower 32 lanes and the odd ones of the upper: the lower lanes finish the first two channels
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const auto t = __builtin_amdgcn_permlane32_swap(as_bits(n[i]), as_bits(n[i + 2]), false, false);
    y[i] = as_f32(t[0]) + as_f32(t[1]);
  }
  float cn[2] = {0.f, 0.f}, cd = 0.f;
  if (corr != nullptr) add_correction<2>(cp, cx, cn, cd);
  normalise<2>(y, den, cn, cd, M, literal);
  // y = y_rot H^T: butterflies over the 128 channels, two per lane (bit 1 of the channel is bit 5 of the lane)
  const float s = y[0] + y[1], d = y[0] - y[1];
  y[0] = s; y[1] = d;
  lane_butterflies<2>(y, lane);
  const half2_t r = {(half_t)(y[0] * kRotation), (half_t)(y[1] * kRotation)};
  *reinterpret_cast<uint32_t*>(out + (long long)row * kHeadDim + ch0) = as_u32(r);
}

// Up to kPairSplits splits: two rows a wave, one in each half, four channels a lane -- the instructions of one row.  row: the first
// of two heads of a sequence (has_two: there is a second one).  own: the rows' only partial results are this workgroup's and lie in
// LDS, row after row; otherwise p0 as in merge_row, max_splits from one row to the next.
// Bound: latency, of the trip to memory and of code that few workgroups of a launch run, cold; so it is there once, for both kinds
// of workgroups, and short.  With a copy in each, one row at a time, a correction workgroup that arrived last at its sequences took
// 3 to 10 us for them, and launches where the streaming workgroups are the faster ones up to 1.5 times as long.
constexpr int kPairSplits = 4;
__device__ __forceinline__ void merge_pair(const float* __restrict__ p0, const float* own, const float* __restrict__ corr, int n_splits,
                                           int max_splits, int row, bool has_two, int lane, bool literal, half_t* __restrict__ out) {
  const int second = has_two ? lane >> 5 : 0, l32 = lane & 31, ch0 = 4 * l32;
  u32x4_t cp[kCorrParts];
  float cx[kCorrParts][4];
  if (corr != nullptr) {
    const float* cr = corr + (long long)row * kCorrParts * kPartStride;
    const __amdgpu_buffer_rsrc_t parts = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(cr), 0, 2 * kCorrParts * kPartBytes, 0x00027000);
#pragma unroll
    for (int r = 0; r < kCorrParts; ++r) {
      cp[r] = __builtin_amdgcn_raw_buffer_load_b128(parts, second * (kCorrParts * kPartBytes) + r * kPartBytes, 0, kCoherentLoad);
      const u32x4_t x = __builtin_amdgcn_raw_buffer_load_b128(parts, second * (kCorrParts * kPartBytes) + 16 * l32 + 16 + r * kPartBytes, 0, kCoherentLoad);
#pragma unroll
      for (int i = 0; i < 4; ++i) cx[r][i] = as_f32(x[i]);
    }
  }
  float M, den, n[4];
  if (own != nullptr) {
    const float* mine = own + second * kPartStride;
    M = mine[0];
    den = mine[1];
#pragma unroll
    for (int i = 0; i < 4; ++i) n[i] = mine[4 + ch0 + i];
  } else {
    const __amdgpu_buffer_rsrc_t rows = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(p0), 0, (has_two ? 2 : 1) * max_splits * kPartBytes, 0x00027000);
    float2 ml[kPairSplits];
    u32x4_t a[kPairSplits];
#pragma unroll
    for (int k = 0; k < kPairSplits; ++k) {
      const int at = min(k, n_splits - 1) * kPartBytes;
      const auto t = __builtin_amdgcn_raw_buffer_load_b64(rows, second * (max_splits * kPartBytes), at, kCoherentLoad);
      ml[k] = make_float2(as_f32(t[0]), as_f32(t[1]));
      a[k] = __builtin_amdgcn_raw_buffer_load_b128(rows, second * (max_splits * kPartBytes) + 16 * l32 + 16, at, kCoherentLoad);
    }
    M = fmaxf(fmaxf(ml[0].x, ml[1].x), fmaxf(ml[2].x, ml[3].x));  // (a copy of the last split in place of those that do not exist)
    den = 0.f;
#pragma unroll
    for (int i = 0; i < 4; ++i) n[i] = 0.f;
#pragma unroll
    for (int k = 0; k < kPairSplits; ++k) {
      const float w = k < n_splits && ml[k].x != -INFINITY ? exp2f(ml[k].x - M) : 0.f;
      den = fmaf(w, ml[k].y, den);
#pragma unroll
      for (int i = 0; i < 4; ++i) n[i] = fmaf(w, as_f32(a[k][i]), n[i]);
    }
  }
  float cn[4] = {0.f, 0.f, 0.f, 0.f}, cd = 0.f;
  if (corr != nullptr) add_correction<4>(cp, cx, cn, cd);
  normalise<4>(n, den, cn, cd, M, literal);
  // y = y_rot H^T: the first two stages in the lane, the others between the 32 lanes of the row
  {
    const float a0 = n[0] + n[1], a1 = n[0] - n[1], a2 = n[2] + n[3], a3 = n[2] - n[3];
    n[0] = a0 + a2; n[1] = a1 + a3; n[2] = a0 - a2; n[3] = a1 - a3;
  }
  row_butterflies<4>(n, lane);
  const half2_t r0 = {(half_t)(n[0] * kRotation), (half_t)(n[1] * kRotation)}, r1 = {(half_t)(n[2] * kRotation), (half_t)(n[3] * kRotation)};
  *reinterpret_cast<uint2*>(out + (long long)(row + second) * kHeadDim + ch0) = make_uint2(as_u32(r0), as_u32(r1));
}

constexpr int kMaxSplits = 32;  // splits a sequence may take at most: a lane of the merge, and a pair of its registers, each
// Splits the groups of a sequence are cut into.  The host fixes the average over the batch (avg_splits) and the most
// one sequence may take (max_splits; grid and workspace are sized for it).  A sequence takes its share of
// B * avg_splits in proportion to its number of groups, rounded up from a quarter on, so that the long and the short
// sequences of a batch end together; a batch of equal lengths gives avg_splits to every sequence.  Integer
// arithmetic only: every wave of the launch that needs the number gets the same one from the same counters.
// A split has at least one group per wave; where a sequence has one split on average, at least kAloneGroups / 2 of them: the chip is
// full there, and a second workgroup, whose place in the grid is behind the first ones of all sequences, starts when most of them
// are done.  Decode launches of unequal lengths, more than 100 sequences and kv heads (2900 shapes of up to 32 groups), as a part of the
// time with one group per wave: 16 groups 0.92 (9 to 16 groups) and 0.99 (17 to 32), 32 groups 0.92 and 0.955, but up to 1.12;
// 144 sequences of 640 to 1280 tokens, 8 kv heads, 47.8 -> 42.1 us a launch, 41.0 without the second workgroups in the grid.
constexpr int kAloneGroups = 24;
__device__ __forceinline__ int groups_of(int nq) { return (nq + kGroup - 1) / kGroup; }

// n_quant of the sequences lane, lane + 64, ... of the first 64 kCounterRows, all requested at once and ahead of the first record
// (a batch beyond 64 sequences was a further trip to memory for every 64, in the workgroups that stream and in those of the
// correction: a step of 144 sequences of 1280 tokens 73.0 -> 70.5 us, 64 of 1k to 16k 85.3 -> 84.8).
constexpr int kCounterRows = 4;
struct BatchCounters {
  int n[kCounterRows];
};
__device__ __forceinline__ BatchCounters request_counters(const kvlinc_cache& c, int lane) {
  BatchCounters r;
#pragma unroll
  for (int u = 0; u < kCounterRows; ++u) r.n[u] = c.n_quant[min(lane + 64 * u, c.B - 1)];
  return r;
}
// Groups of the whole batch, in a scalar register.
__device__ __forceinline__ int batch_groups(const kvlinc_cache& c, const BatchCounters& r, int lane) {
  uint32_t total = 0;
#pragma unroll
  for (int u = 0; u < kCounterRows; ++u) total += lane + 64 * u < c.B ? groups_of(r.n[u]) : 0;
  for (int first = 64 * kCounterRows; first < c.B; first += 64) {  // (no lane goes its own way: see the callers)
    int n = c.n_quant[min(first + lane, c.B - 1)];
    asm volatile("" : "+v"(n));
    total += first + lane < c.B ? groups_of(n) : 0;
  }
  total += dpp_u<kRowRor1>(total);
  total += dpp_u<kRowRor2>(total);
  total += dpp_u<kRowRor4>(total);
  total += dpp_u<kRowRor8>(total);
  const auto a = __builtin_amdgcn_permlane16_swap(total, total, false, false);
  total = a[0] + a[1];
  const auto b = __builtin_amdgcn_permlane32_swap(total, total, false, false);
  return __builtin_amdgcn_readfirstlane((int)(b[0] + b[1]));
}

// count = the sequence's groups (the same in every lane), total = the batch's.  ceil(avg count B / total - 1/4) is the
// number of k >= 0 with 4 avg count B - total > 4 k total: the 64 lanes try one k each (max_splits is at most 32).
__device__ __forceinline__ int sequence_splits(const kvlinc_cache& c, int count, int total, int avg_splits, int max_splits,
                                               int lane) {
  if (c.B == 1) return avg_splits;
  int s = avg_splits;
  if (total > 0) {
    const long long num = 4ll * avg_splits * count * c.B - total;
    s = __builtin_popcountll(__builtin_amdgcn_ballot_w64(num > 4ll * total * lane));
  }
  s = min(s, min(max_splits, avg_splits == 1 ? (count + kAloneGroups - 1) / kAloneGroups : (count + kWaves - 1) / kWaves));
  return __builtin_amdgcn_readfirstlane(max(s, 1));            // the same in every lane: keep it in a scalar register
}

// The counter of a (sequence, kv head), which its workgroups arrive at: see kvlinc_handoff.h for who merges.
// (Why a streaming workgroup rather than one of the correction, which may be awaited: that has the rows of up to 8 sequences to merge, a
// streaming workgroup those of one, which the single split of a sequence has in LDS besides; see decode_launch for what awaiting
// gives.  Looks without s_sleep(16) between them, 2 instead: 1.002 of the time on average and 1.30 instead of 1.27 at most; 48: 1.003.)
#ifndef KVLINC_LOOKS
#define KVLINC_LOOKS 64  // (tests build a library with none, in which every wait runs out at once)
#endif
constexpr int kLooks = KVLINC_LOOKS;
struct ArrivalCounter {
  int* count;
  __device__ __forceinline__ int add(int n) { return __hip_atomic_fetch_add(count, n, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM); }
  __device__ __forceinline__ int look() { return __hip_atomic_load(count, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM); }
  __device__ __forceinline__ void pause() { __builtin_amdgcn_s_sleep(16); }  // (about half a microsecond: more looks get in the way of the arrivals they wait for)
};

// Grid: B H_kv max_splits streaming workgroups, split-major (workgroup = split * B H_kv + sequence * H_kv + kv head),
// each streaming the groups and the window share of one split of a (sequence, kv head), or leaving at once when its
// sequence uses fewer splits; and, when the correction is on, the correction workgroups: after them (corr_first = 0)
// or leading the first corr_first runs of 256 workgroups (1: all of them first -- they are long chains of dependent
// steps and should start at once).  All of them count themselves in at split_done; who merges: above.
// SLIDING: the variant with the sliding value window (KVLINC_FLAG_SLIDING_VALUES) is a kernel of its own, so that the
// default one carries none of its code.
// BITS: so is the one for caches with 4-bit codes (it holds twice the tile words in registers).
// FEW_HEADS: and the one for fewer than 4 query heads per kv head (see correction_workgroup).
// What the way to the first requests takes comes in 14 words, which are in scalar registers when a wave starts (see
// append_token_kernel): five pointers, and counts that stay below 2^24 with small numbers above them.
struct LaunchWords {
  uint32_t batch;   // B - 1, splits of a sequence on average << 24, correction awaited << 30, on << 31
  uint32_t heads;   // H_kv - 1, most splits of a sequence << 24, runs of the grid that the correction leads << 30
  uint32_t groups;  // max_groups - 1, query heads per kv head - 1 << 24, log2 of the sequences of a correction workgroup << 27,
                    // rounds that split 0 sits out - 1 << 29
  uint32_t magic;   // ceil(2^32 / H_kv), or 0 where that does not give quotients by H_kv
};
constexpr uint32_t kLow24 = (1u << 24) - 1u;

template <int NB, bool SLIDING = false, int BITS = 2, bool FEW_HEADS = false>
__global__ __launch_bounds__(kThreads, BITS == 4 || (NB == 2 && SLIDING) ? 2 : 3) void decode_main_kernel(uint32_t* groups, int32_t* n_quant, const half_t* __restrict__ q,
                                                                   const kvlinc_half* Wq, kvlinc_half* S16, uint32_t batch_word, uint32_t heads_word,
                                                                   uint32_t groups_word, uint32_t magic, kvlinc_cache cache,
                                                                   float* __restrict__ corr, float* __restrict__ part, half_t* __restrict__ out) {
  const LaunchWords words = {batch_word, heads_word, groups_word, magic};
  const int max_splits = (words.heads >> 24) & 63, avg_splits = (words.batch >> 24) & 63, L = words.heads >> 30, gq = ((words.groups >> 24) & 7) + 1;
  const int log_seqs = (words.groups >> 27) & 3, corr_seqs = 1 << log_seqs;
  const bool has_corr = words.batch >> 31, awaited = (words.batch >> 30) & 1;
  kvlinc_cache c = cache;
  c.groups = groups; c.n_quant = n_quant; c.Wq = Wq; c.S16 = S16;
  c.max_groups = (int)(words.groups & kLow24) + 1; c.B = (int)(words.batch & kLow24) + 1; c.H_kv = (int)(words.heads & kLow24) + 1; c.H_q = gq * c.H_kv;
  auto by_heads = [&](int n) { return words.magic != 0 ? (int)__umulhi((uint32_t)n, words.magic) : n / c.H_kv; };
  constexpr int kCombine = 2 * kWaves * NB * 4 + kWaves * NB * 4 * kHeadDim;
  __shared__ __align__(16) float lds[kCombine + kWaves * 2 * kExWords];
  static_assert(kCombine + kWaves * 2 * kExWords >= kMaxCorrSeqs * NB * 4 * kPartFeat, "the logits of a correction workgroup");
  uint32_t (*ex)[2 * kExWords] = reinterpret_cast<uint32_t (*)[2 * kExWords]>(lds + kCombine);  // per wave: operand hand-over of q K^T and of E V
  __shared__ int sFlag;

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // wave-uniform: keeps the schedule in scalar registers
  const int n_corr = has_corr ? c.H_kv * kCorrParts * ((c.B + corr_seqs - 1) >> log_seqs) : 0;
  const int n_parts = has_corr ? kCorrParts : 0;

  // L = 0: the correction workgroups come last; L >= 1: they lead each of the first L runs of 256
  // workgroups in equal shares.  The dispatcher deals workgroup i to compute unit i mod 256 while places are free, so
  // with L = 2 the correction workgroups pair up on compute units of their own and no streaming workgroup has one
  // as a neighbour.
  bool is_corr;
  int corr_id, stream_id;
  if (L == 0) {
    corr_id = blockIdx.x - c.B * c.H_kv * max_splits;
    is_corr = corr_id >= 0;
    stream_id = blockIdx.x;
  } else if (L == 1) {
    is_corr = (int)blockIdx.x < n_corr;
    corr_id = blockIdx.x;
    stream_id = blockIdx.x - n_corr;
  } else {
    const int per = L == 2 ? (n_corr + 1) >> 1 : (n_corr + 2) / 3;
    const int layer = min((int)blockIdx.x / 256, L), pos = layer < L ? (int)blockIdx.x % 256 : 0;
    const int before = min(n_corr, layer * per + min(pos, per));  // correction workgroups ahead of this one
    is_corr = layer < L && pos < per && before < n_corr;
    corr_id = before;
    stream_id = blockIdx.x - before;
  }

  // What is left to merge when the workgroup has done its part: the sequences done (bit s: sequence m_first + s) of kv head m_g, of
  // as many splits as the bytes of `splits` say.
  int m_first, m_g;
  uint32_t done = 0;
  uint64_t splits = 0;
  bool direct = false;

  if (is_corr) {
    // ---- one part of the correction (Sec. 3.3: C_n, C_d) for up to corr_seqs sequences of one kv head ----
    const int id = corr_id;
    // The workgroups that read the same slice of W (same kv head and part, different sequences) are H_kv * kCorrParts
    // apart in the grid: workgroups are dealt to the 8 XCDs in turn, so with an even H_kv they share one L2.
    const int r = id % kCorrParts, sb = by_heads(id / kCorrParts), g = id / kCorrParts - sb * c.H_kv;
    const int b_first = sb * corr_seqs;
    const int n_seq = min(corr_seqs, c.B - b_first);
    // A sequence without quantized tokens has S = P = 0 (the states only change at a flush), so its parts come out
    // as zero without looking at n_quant.
    // (the counters are requested first and looked at last: by then they have long arrived)
    const BatchCounters counters = request_counters(c, lane);
    const int nq_mine = c.n_quant[b_first + min(lane, n_seq - 1)];
    correction_workgroup<FEW_HEADS, NB>(c, q, corr, gq, g, r, b_first, n_seq, lane, wave, lds);
    const int total = batch_groups(c, counters, lane);
    // count this workgroup in at each of its sequences; merge those it completes
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    int* sFlags = reinterpret_cast<int*>(lds);
    if (tid < n_seq)
      sFlags[tid] = ArrivalCounter{c.split_done + (b_first + tid) * c.H_kv + g}.add(kCorrArrival);
    __syncthreads();
    m_first = b_first;
    m_g = g;
    for (int s = 0; s < n_seq; ++s) {
      const int n_splits = sequence_splits(c, groups_of(__builtin_amdgcn_readlane(nq_mine, s)), total, avg_splits, max_splits, lane);
      splits |= (uint64_t)n_splits << (8 * s);
      if (correction_merges(__builtin_amdgcn_readfirstlane(sFlags[s]), n_splits, n_parts, awaited)) done |= 1u << s;
    }
  } else {
  // ---- one split of the groups and of the window (Alg. 1, the loop over blocks) ----
  const int wg = stream_id;
  // split-major: the splits that only long sequences use come last in the grid, and the workgroups of any one split
  // index are dealt evenly to the XCDs
  int bh = wg, sp = 0;  // (at most 32 splits: a division by shifts)
#pragma unroll
  for (int i = 4; i >= 0; --i) {
    const int run = (c.B * c.H_kv) << i;
    const bool past = bh >= run;
    bh -= past ? run : 0;
    sp += past ? 1 << i : 0;
  }
  const int b = by_heads(bh), g = bh - b * c.H_kv;

  // Static schedule, the same for every sequence length, so that a wave knows its first group before it knows the length (GroupOrder).
  int n_splits = avg_splits;  // first guess: right for a batch of equal lengths
  const int skip = BITS == 2 ? (int)((words.groups >> 29) & 1) + 1 : 1;
  int rd, idx;
  GroupOrder order(n_splits, sp, wave, skip);
  auto plan = [&]() {
    order = GroupOrder(n_splits, sp, wave, skip);
    rd = sp == 0 ? skip : 0;
    idx = order.group(rd);
  };

  // What the wave works on first -- its part of the window, a record -- is requested before the sequence length is known (any group
  // index below the capacity is readable memory, and so are the window's slots); what it holds is used only if it exists.
  constexpr int kRecordWords = Rec<BITS>::kWords;
  const uint32_t* rec0 = c.groups + (long long)bh * c.max_groups * kRecordWords;
  const Roles lr = make_roles(lane, ex[wave]);
  KeyRegs<BITS> kr;
  ValueRegs<BITS> vr;
  uint32_t qh[NB][4];  // q of the head this lane builds operands for (head 4 nb + ha, or the last one), channels c0 .. c0 + 7
  auto request_q = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
      const uint4 raw = *reinterpret_cast<const uint4*>(q + ((long long)b * c.H_q + g * gq + min(nb * 4 + lr.ha, gq - 1)) * kHeadDim + lr.c0);
      qh[nb][0] = raw.x; qh[nb][1] = raw.y; qh[nb][2] = raw.z; qh[nb][3] = raw.w;
    }
  };
  auto request_record = [&](bool with_q) __attribute__((always_inline)) {
    const long long first = idx < c.max_groups ? idx : c.max_groups - 1;
    // (in the order of the loop below, whatever the way here: the wait for a part is then for that part alone)
    load_keys(kr, rec0 + first * kRecordWords, lr);
    asm volatile("" ::: "memory");
    if (with_q) request_q();
    asm volatile("" ::: "memory");
    load_values(vr, rec0 + first * kRecordWords, lr);
    asm volatile("" ::: "memory");
  };
  int nq, nr, count;
  auto splits_of_sequence = [&](BatchCounters& counters) __attribute__((always_inline)) {
    nq = scalar_load(c.n_quant + b);
    nr = scalar_load(c.n_res + b);
    count = groups_of(nq);
    // the spare term row of every head reads as zero from here on (this wave's own regions: no barrier needed)
#pragma unroll
    for (int k = 0; k < 4; ++k) ex[wave][(k >> 1) * kExWords + (2 * (k & 1) + (lane >> 5)) * kExHead + 96 + (lane & 31)] = 0u;
    lds_order();
    // (waited for in any case: see the end of the branch below)
#pragma unroll
    for (int u = 0; u < kCounterRows; ++u) asm volatile("" : "+v"(counters.n[u]));
    return sequence_splits(c, count, c.B > 1 ? batch_groups(c, counters, lane) : 0, avg_splits, max_splits, lane);
  };
  WaveState<NB> st;
  // (The counters are requested in every branch by itself: a load from ahead of the branches counts as under way on a path that takes
  // none of them, which the compiler keeps, and its wait in the loop over the groups would be for the next record, too.  The
  // statements that open the branches differ so that their loads are not joined ahead of them.)
  if (sp == 0) {
    asm volatile("; with the window" ::: "memory");
    BatchCounters counters = request_counters(c, lane);
    plan();
    request_record(true);
    asm volatile("" ::: "memory");
    const WindowShare sh = window_share(scalar_load(c.n_res + b), groups_of(scalar_load(c.n_quant + b)), avg_splits == 1, wave);
    WindowRegs w;
    if (sh.first < sh.end) request_window(w, c, bh, sh, lr);
    asm volatile("" ::: "memory");
    const int mine = splits_of_sequence(counters);
    if (mine != n_splits) {
      n_splits = mine;
      plan();
      request_record(false);
    }
    if (sh.first < sh.end) window_part<NB>(w, qh, sh, lr, st);
    else empty_state<NB>(st);
    // (nothing is under way any more: registers that a load may still write make the compiler wait in every round of the loop over
    // the groups, and that for the next record, too)
    __builtin_amdgcn_s_waitcnt(kAllLoads);
  } else if (sp < avg_splits) {
    asm volatile("; groups" ::: "memory");
    BatchCounters counters = request_counters(c, lane);
    plan();
    request_record(true);
    empty_state<NB>(st);
    const int mine = splits_of_sequence(counters);
    if (mine != n_splits) {  // lengths differ within the batch: plan again, request the right first record
      n_splits = mine;
      if (sp < n_splits) {
        plan();
        request_record(true);
      }
    }
  } else {  // a split that only the longest sequences of a batch use
    asm volatile("; groups, perhaps" ::: "memory");
    BatchCounters counters = request_counters(c, lane);
    empty_state<NB>(st);
    n_splits = splits_of_sequence(counters);
    if (sp < n_splits) {
      plan();
      request_record(true);
    }
  }
  if (sp >= n_splits) return;  // this sequence uses fewer splits than the grid provides
  // q has arrived from here on: left to its first use, the compiler would wait in every round of the loop for all that may be under
  // way behind it, the next record among it.
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) asm volatile("" : "+v"(qh[nb][0]), "+v"(qh[nb][1]), "+v"(qh[nb][2]), "+v"(qh[nb][3]));

  float (*sM)[NB * 4] = reinterpret_cast<float (*)[NB * 4]>(lds);                    // [kWaves][NB*4]
  float (*sL)[NB * 4] = reinterpret_cast<float (*)[NB * 4]>(lds + kWaves * NB * 4);  // [kWaves][NB*4]
  float (*sAcc)[NB * 4][kHeadDim] = reinterpret_cast<float (*)[NB * 4][kHeadDim]>(lds + 2 * kWaves * NB * 4);

  if (idx < count) {
    // While a group is consumed the wave's next record is already requested: its key part right after the scores,
    // its value part right after E V.  The wave's last group is a copy of the loop body without requests (a request
    // past the end would be a second trip to memory for a record that the non-temporal loads did not leave in the
    // caches, and the combine would wait for it: config 7 68.8 -> 65.3 us, config 6 53.0 -> 50.2 us).
    // sliding value window: the newest group's tokens from n_res on take their values from the window
    // (the newest group is left to the code below when its last tokens take their values from the window)
    const float slack = (c.flags & KVLINC_FLAG_ALG1_LITERAL) != 0 ? 0.0f : kSlack;
    const bool sliding = SLIDING && nq % kGroup == 0 && nr < kGroup;
    const int count_plain = sliding ? count - 1 : count;
    while (idx < count_plain) {
      const int nxt = order.group(++rd);
      if (nxt >= count) break;
      const uint32_t* src = rec0 + (long long)nxt * kRecordWords;
      float sc[NB][8], off[NB], base[NB];
      qk_phase<NB, BITS>(kr, kGroup, qh, lr, sc, off);
      load_keys(kr, src, lr);
      update_reference<NB>(sc, off, base, st, slack);
      pv_phase<NB, BITS>(vr, sc, base, lr, st);
      load_values(vr, src, lr);
      idx = nxt;
    }
    if (idx < count_plain) {  // the wave's last group: nothing more to request
      float sc[NB][8], off[NB], base[NB];
      qk_phase<NB, BITS>(kr, min(kGroup, nq - idx * kGroup), qh, lr, sc, off);
      update_reference<NB>(sc, off, base, st, slack);
      pv_phase<NB, BITS>(vr, sc, base, lr, st);
      idx = count;
    }
    if (SLIDING && idx < count) {  // sliding value window: the newest group, whose tokens from n_res on have fp16 values
      const half_t* const v_win = reinterpret_cast<const half_t*>(c.v_res) + (long long)bh * c.R * kHeadDim;
      float sc[NB][8], off[NB], base[NB];
      uint32_t touched[kWindowLines / 64];
      touch_window_tail(touched, v_win, nr, lane);
      qk_phase<NB, BITS>(kr, kGroup, qh, lr, sc, off);
      update_reference<NB>(sc, off, base, st, slack);
#pragma unroll
      for (int u = 0; u < kWindowLines / 64; ++u) asm volatile("" ::"v"(touched[u]));
      pv_phase<NB, BITS, true>(vr, sc, base, lr, st, nr);
      pv_window_tail<NB>(v_win, sc, base, nr, lr, st, lane, sAcc[wave]);
    }
  }

  // A sequence with a single split merges what its one workgroup holds, without the trip of its partial result through memory, when
  // the correction parts have all arrived (or the correction is off) or are awaited.  The first look at the counter is taken here
  // so that its latency passes during the combine.
  __shared__ int sDirect;
  ArrivalCounter counter{c.split_done + bh};
  if (tid == 0) sDirect = n_splits == 1 && (n_parts == 0 || parts_arrived(counter.look()) == n_parts);
  // combine the four waves (Alg. 1 lines 13-14 restricted to this workgroup) and write (m, l, Y_s)
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) {
    const float l = row_allsum(st.l[nb]);
    const float pz = row_allsum(st.pz[nb]);
    const int h = nb * 4 + lr.hd;
    if (lr.jd == 0) { sM[wave][h] = st.m[nb]; sL[wave][h] = l; }
#pragma unroll
    for (int n = 0; n < 8; ++n)
      sAcc[wave][h][16 * n + lr.jd] = st.acc[nb][n] + pz;
  }
  __syncthreads();
  direct = __builtin_amdgcn_readfirstlane(sDirect) != 0;
  const bool keep = direct || (awaited && n_splits == 1);  // the result stays here for now
  // (a wave takes whole heads, a lane two channels: the weights of the four waves are formed once a head)
  float* own = reinterpret_cast<float*>(&ex[0][0]);  // [gq][kPartStride]: the exchange regions are free by now
  for (int h = wave; h < gq; h += kWaves) {
    float M = -INFINITY;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) M = fmaxf(M, sM[w][h]);
    float a0 = 0.f, a1 = 0.f, l = 0.f;
    if (M != -INFINITY) {
#pragma unroll
      for (int w = 0; w < kWaves; ++w) {
        const float f = __builtin_amdgcn_exp2f(sM[w][h] - M);  // 0 for a wave without tokens
        const float2 x = *reinterpret_cast<const float2*>(&sAcc[w][h][2 * lane]);
        a0 = fmaf(f, x.x, a0);
        a1 = fmaf(f, x.y, a1);
        l = fmaf(f, sL[w][h], l);
      }
    }
    if (keep) {
      float* dst = own + h * kPartStride;
      if (lane == 0) { dst[0] = M; dst[1] = l; }
      *reinterpret_cast<float2*>(dst + 4 + 2 * lane) = make_float2(a0, a1);
    } else {
      float* dst = part + (((long long)b * c.H_q + g * gq + h) * max_splits + sp) * kPartStride;
      if (lane == 0) st_coherent2(dst, M, l);
      st_coherent2(dst + 4 + 2 * lane, a0, a1);
    }
  }
  m_first = b;
  m_g = g;
  splits = n_splits;
  if (keep) {
    barrier_lds_only();
    if (!direct) {
      if (tid == 0) sDirect = await_parts(counter, n_parts, kLooks);
      barrier_lds_only();
      direct = __builtin_amdgcn_readfirstlane(sDirect) != 0;
    }
    if (!direct) {  // given up: the result goes to memory after all
      for (int h = wave; h < gq; h += kWaves) {
        const float* src = own + h * kPartStride;
        float* dst = part + ((long long)b * c.H_q + g * gq + h) * max_splits * kPartStride;
        if (lane == 0) st_coherent2(dst, src[0], src[1]);
        st_coherent2(dst + 4 + 2 * lane, src[4 + 2 * lane], src[5 + 2 * lane]);
      }
    }
  }
  if (direct) {
    done = 1;
  } else {
    // Every wave first waits until its write-through stores have been acknowledged, then one thread counts the workgroup in.  If it
    // merges (Alg. 1 lines 13-15) it reads what the others wrote with coherent loads.
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (tid == 0) sFlag = stream_arrives(counter, n_splits, n_parts, awaited, keep, kLooks);  // (keep: it has given up)
    __syncthreads();
    done = __builtin_amdgcn_readfirstlane(sFlag) != 0;
  }
  }

  // ---- merge (Alg. 1 lines 13-15) ----
  const bool literal = (c.flags & KVLINC_FLAG_ALG1_LITERAL) != 0;
  int turn = 0;
  for (uint32_t left = done; left != 0; left &= left - 1) {
    const int s = __builtin_ctz(left), n_splits = (int)(splits >> (8 * s)) & 255, row0 = (m_first + s) * c.H_q + m_g * gq;
    if (n_splits <= kPairSplits) {
      for (int h = 0; h < gq; h += 2, ++turn)
        if (turn % kWaves == wave)
          merge_pair(part + (long long)(row0 + h) * max_splits * kPartStride, direct ? reinterpret_cast<float*>(&ex[0][0]) + h * kPartStride : nullptr, corr,
                     n_splits, max_splits, row0 + h, h + 1 < gq, lane, literal, out);
    } else {
      for (int h = wave; h < gq; h += kWaves) {
        const float* p0 = part + (long long)(row0 + h) * max_splits * kPartStride;
        if (n_splits <= 12) merge_row<6>(p0, corr, n_splits, row0 + h, lane, literal, out);
        else merge_row<kMaxSplits / 2>(p0, corr, n_splits, row0 + h, lane, literal, out);
      }
    }
    if (tid == 0) c.split_done[(m_first + s) * c.H_kv + m_g] = 0;
  }
}

}  // namespace

// Groups of the longest context that a launch can meet.
static long long longest_groups(const kvlinc_cache& c, int max_context) {
  const long long cap = (long long)c.max_groups * kGroup + c.R;
  const long long ctx = (max_context > 0 && max_context < cap) ? max_context : cap;
  return ctx > kGroup ? (ctx + kGroup - 1) / kGroup : 1;
}

// Splits per (sequence, kv head).  Measured on MI355X (256 compute units): the launch is fastest when all its
// workgroups, the correction workgroups included, are resident at once at about two per compute unit -- a second
// generation of workgroups pays the start-up and the merge tail again, and a compute unit that hosts a correction
// workgroup next to two streaming ones finishes late.  The kernel for more than 4 query heads per kv head spends more on
// a group: there the streaming workgroups alone make up the two per compute unit (32 sequences of 32k tokens, 7 heads:
// 3 splits 84.0 us, 4 76.5, 5 76.9 a step).  At most 32 splits (the merge holds a row of each
// in registers; 40 to 64 for one sequence of 131072 tokens, two workgroups per compute unit: 28.2 to 30.8 us a step against 25.0 with 30),
// at least one group per wave.
constexpr long long kPlaces = 768;  // workgroups that the chip holds at three per compute unit
DecodeSplits decode_splits(const kvlinc_cache& c, int max_context) {
  constexpr int kTargetWorkgroups = 512;
  const long long groups = longest_groups(c, max_context);
  const long long bh = (long long)c.B * c.H_kv;
  const int gq = c.H_q / c.H_kv;
  long long n_corr = 0;
  // Sequences per correction workgroup: 4, one for each wave.  8 in turn (8 against 4, decode launches)
  //   - with 1 or 2 query heads per kv head and 2 bits, where workgroups of 4 and the streaming ones do not fit the chip at once
  //     (three per compute unit), workgroups of 8 do, and contexts are 12 to 63 groups: equal lengths 0.79 to 1.07 of the time,
  //     0.89 on average, unequal ones 0.80 to 1.15 and 0.98 (1 to 64 kv heads, 830 shapes; with 4, the streaming workgroups that do
  //     not fit start behind a whole correction workgroup and end a round later).
  //     Shorter contexts 0.90 to 1.39, 1.14 on average; longer ones, where the correction goes last (below), 0.82 to 1.23; where 4
  //     fit, or 8 do not, 0.88 to 1.80;
  //   - with one query head and 1024 workgroups of 4 or more, where the weights are a small part of what a workgroup reads: 0.96
  //     to 1.10 at 2 bits, mostly 0.98 to 1.02, 0.94 to 1.04 at 4 bits (8 to 64 kv heads, 300 to 4000 tokens).  An empirical cut:
  //     from 768 to 1023 0.98 to 1.17 at 2 bits, 0.94 to 1.03 at 4.
  auto corr_workgroups = [&](int seqs) { return (long long)c.H_kv * kCorrParts * ((c.B + seqs - 1) / seqs); };
  const bool eight_fit = bh + corr_workgroups(4) > kPlaces && bh + corr_workgroups(8) <= kPlaces;
  const bool eight = (gq == 1 && corr_workgroups(4) >= 1024) || (gq <= 2 && c.bits == 2 && eight_fit && groups >= 12 && groups < 64);
  const int corr_seqs = eight ? 8 : 4;
  if (c.S16 != nullptr && gq <= 4) n_corr = corr_workgroups(corr_seqs);
  long long s = (kTargetWorkgroups - n_corr + bh / 2) / bh;  // rounded to nearest
  if (s > kMaxSplits) s = kMaxSplits;
  const long long most = (groups + kWaves - 1) / kWaves;
  if (s > most) s = most;
  if (s < 1) s = 1;
  // Head room for the longest sequences of a batch of unequal lengths (a single sequence has nobody to differ from).
  long long m = c.B > 1 ? 2 * s : s;
  if (m > kMaxSplits) m = kMaxSplits;
  if (m > most) m = most;
  if (m < s) m = s;
  // The correction workgroups are chains of dependent steps and go first in the grid, except when they alone would
  // fill most of the chip while the streaming workgroups have long contexts ahead of them (many sequences, 16 or
  // more groups per wave): then the streaming workgroups go first, the longest of them decide when the launch ends,
  // and the correction fills the places the short sequences leave.
  const long long all_corr = c.S16 != nullptr ? corr_workgroups(corr_seqs) : 0;
  // (More than 4 heads per kv head: the correction takes the third place of a compute unit, and going last it does not
  // hold up the streaming workgroups.  Launches of 5 to 8 heads, 1 to 8 kv heads, 8 to 64 sequences of 8k to 64k tokens, last
  // against first: at 2 bits, from 8 groups per wave on, 0.86 to 1.01 of the time, with 4 and fewer 0.86 to 1.48; at 4 bits, from
  // 16 on, 0.98 to 1.02.)
  const int long_wave = gq > 4 && c.bits == 2 ? 8 : 16;
  int corr_first = ((gq > 4 || 2 * all_corr > 768) && groups >= long_wave * kWaves * s) ? 0 : 1;
  // Between one and two workgroups per compute unit, the correction included.  Where the splits can be cut back by a quarter at
  // most, the correction workgroups may pair up on compute units of their own (two runs of the grid lead with them): what 4 bits
  // take, where a unit holds two workgroups and the streaming ones that share one with a correction workgroup finish late (1.00
  // to 1.12 with the correction last).  At 2 bits a unit holds three: the streaming workgroups go first then, with all splits, and
  // the correction shares the units it finds, but only
  //   - from 2 splits on, 4 for more than 4 heads, and for 3 and 4 heads where the splits could be cut back: 0.60 to 1.48 of the
  //     time the others take, 0.94 on average (the splits follow the context here, 512 tokens each; with 2 and 3 of them 5 to 8
  //     heads take 0.93 to 1.74 times as long, 1.34 on average, and 3 and 4 heads, where they cannot be cut back, 0.89 to 1.58, 1.23
  //     on average);
  //   - with one split from 24 groups on and 2 or more heads: 0.88 to 1.09, 0.99 on average.  A single split merges what it holds
  //     when it finds the correction done, and below that the correction is the longer chain: 0.87 to 1.45, 1.10 on average.
  // (Decode launches of 2 to 64 sequences of 140 to 131072 tokens, equal ones and lengths spread by 0.3, 0.6 and 0.9, 1 to 8 heads,
  // 1 to 32 kv heads: 1471 shapes, twice.)
  // A single sequence is left on units of its own and 30 splits, the stated policy for it: 131072 tokens, 8 kv heads, 20.5 us a
  // launch, where 32 splits with the correction last would take 19.9.
  // One or two sequences a correction workgroup instead of 4 where that gives no compute unit another workgroup: two or four waves
  // share a sequence then, and a workgroup that arrives last has fewer rows to merge.  More splits than one, decode launches with the
  // fewest that fit so, against 4, on average (0.1 to 0.3 of the time between single shapes, either way): 0.99 to 1.01 on one workgroup
  // per unit, 0.88 to 0.98 on two, 0.98 on three.  A unit more: 1.04 to 1.35.  (4 bits, where a unit holds two: 2 sequences rather
  // than 1 on two, 0.98 against 1.01; the sliding window's kernel for more than 4 heads holds two as well: with workgroups of 1 and 2 as if
  // it held three, 59 such launches took up to 1.16 of the time of the kernels before, 1.09 with 4.)  One split (7700 shapes of up to 1100 tokens): 2 sequences where all workgroups have a unit of
  // their own, 0.97 and 0.98 of the time of 4, 1 sequence 1.01; beyond that 2 take 1.02.
  const int held = c.bits == 4 || (gq > 4 && (c.flags & KVLINC_FLAG_SLIDING_VALUES) != 0) ? 2 : 3;  // workgroups on a unit (launch bounds)
  auto launch = [&](long long avg, long long most_splits, int first) {
    int seqs = corr_seqs;
    const long long per_unit = (bh * avg + corr_workgroups(4) + 255) / 256;
    if (seqs == 4 && per_unit <= (avg == 1 ? 1 : held))
      for (int k = 2; k >= (avg == 1 || (held == 2 && per_unit == 2) ? 2 : 1); --k)
        if (bh * avg + corr_workgroups(k) <= 256 * per_unit) seqs = k;
    return DecodeSplits{(int)avg, (int)most_splits, first, seqs};
  };
  if (all_corr > 0 && bh * s <= 256 && bh * s + all_corr > 256) {
    const long long s2 = (256 - (all_corr + 1) / 2) / bh;
    const bool own_units = s2 >= 1 && 4 * s2 >= 3 * s;
    const bool long_enough = s == 1 ? gq >= 2 && groups >= 24 : s >= (gq > 4 ? 4 : 2) && (own_units || gq <= 2);
    if (c.bits == 2 && c.B > 1 && long_enough) return launch(s, m, 0);
    if (own_units) {
      s = s2 < s ? s2 : s;
      if (m > s) m = c.B > 1 ? 2 * s : s;
      if (m > kMaxSplits) m = kMaxSplits;
      if (m > most) m = most;
      if (m < s) m = s;
      // (All of them on units of their own, one run: the correction is the first to start, and awaited.  47 launches, most of them at
      // 4 bits: 0.77 of the time of two runs, 0.56 to 1.03.)
      if (bh * s + all_corr > 256) corr_first = 2;
    }
  }
  return launch(s, m, corr_first);
}

size_t decode_workspace_floats(const kvlinc_cache& c, int n_splits) {
  return (size_t)c.B * c.H_q * (n_splits + kCorrParts) * kPartStride;  // split partials, then the correction parts
}

DecodeLaunch decode_launch(const kvlinc_cache& c, int max_context) {
  const DecodeSplits sp = decode_splits(c, max_context);
  DecodeLaunch l;
  // The grid has no second workgroups where no sequence takes them (sequence_splits).  The workspace is sized for them all the same:
  // its size is the same for a program's buffers, and for the limit of the static scratch, whatever the launch makes of it.
  l.avg = sp.avg;
  l.splits = sp.avg == 1 && longest_groups(c, max_context) <= kAloneGroups ? 1 : sp.most;
  l.corr_seqs = sp.corr_seqs;
  const int BH = c.B * c.H_kv;
  const int n_corr = c.S16 != nullptr ? c.H_kv * kCorrParts * ((c.B + sp.corr_seqs - 1) / sp.corr_seqs) : 0;
  l.workgroups = BH * l.splits + n_corr;
  // every run that leads with correction workgroups must lie inside the grid and hold its share
  int L = n_corr != 0 ? sp.corr_first : 0;
  while (L > 1 && (l.workgroups < 256 * (L - 1) + (n_corr + L - 1) / L || (n_corr + L - 1) / L > 256)) --L;
  l.corr_first = L;
  // The correction is awaited only where all of its workgroups are ahead of the streaming ones (one run leads): they are given
  // their places first.  3000 such launches: 0.983 of the time of a merge by whoever arrives last, 0.71 to 1.21.  Streaming workgroups
  // ahead of it, or of half of it, would hold the very places that it waits for when launches of other streams have the rest of the
  // chip: three caches decoded on three streams, the correction last, took 0.97 to 1.37 of the time when it was awaited, 1.09 on
  // average (30 shapes); alone, launches with the correction last or in two runs take 0.99 of the time when it is not (1500 shapes).
  // Nor is it awaited by more than 256 sequences and heads with one split each, whose looks crowd the counters, nor by several splits of
  // a sequence whose correction workgroups have no other sequence's rows to merge: without the wait 2441 such launches took 0.996 of
  // the time, those of a single sequence 0.993 with up to 4 heads and 0.973 with more.
  l.awaited = L == 1 && (sp.avg > 1 ? sp.corr_seqs > 1 && c.B > 1 : BH <= 256);
  // (a context of the bound itself has one group less: its last tokens are the window's)
  const int count = (int)longest_groups(c, max_context) - 1;
  const int most = (count + kWaves - 1) / kWaves;  // splits that it takes at most (sequence_splits)
  l.skip = window_rounds(count, sp.avg < most ? sp.avg : most, c.bits);
  return l;
}

int launch_decode(const kvlinc_cache& c, const kvlinc_half* q, kvlinc_half* out, float* workspace, int max_context,
                  hipStream_t stream, hipEvent_t start, hipEvent_t stop) {
  const DecodeLaunch l = decode_launch(c, max_context);
  const int gq = c.H_q / c.H_kv;
  const half_t* qq = reinterpret_cast<const half_t*>(q);
  half_t* oo = reinterpret_cast<half_t*>(out);
  float* part = workspace;
  float* corr = c.S16 != nullptr ? workspace + (size_t)c.B * c.H_q * l.splits * kPartStride : nullptr;
  const bool sliding = (c.flags & KVLINC_FLAG_SLIDING_VALUES) != 0;
  const dim3 grid(l.workgroups), block(kThreads);
  // n / H_kv = umulhi(n, magic) for n below 2^32 / H_kv; n is at most 2^24 + 3 H_kv here
  const uint32_t magic = c.H_kv > 1 && c.H_kv <= 128 ? (uint32_t)(((1ull << 32) + c.H_kv - 1) / c.H_kv) : 0u;
  const LaunchWords words = {(uint32_t)(c.B - 1) | (uint32_t)l.avg << 24 | (uint32_t)l.awaited << 30 | (uint32_t)(corr != nullptr) << 31,
                             (uint32_t)(c.H_kv - 1) | (uint32_t)l.splits << 24 | (uint32_t)l.corr_first << 30,
                             (uint32_t)(c.max_groups - 1) | (uint32_t)(gq - 1) << 24 | (uint32_t)__builtin_ctz(l.corr_seqs) << 27 | (uint32_t)(l.skip - 1) << 29, magic};
  void (*kernel)(uint32_t*, int32_t*, const half_t*, const kvlinc_half*, kvlinc_half*, uint32_t, uint32_t, uint32_t, uint32_t, kvlinc_cache, float*, float*, half_t*) =
      c.bits == 4 ? (gq > 4   ? (sliding ? decode_main_kernel<2, true, 4> : decode_main_kernel<2, false, 4>)
                     : gq < 4 ? (sliding ? decode_main_kernel<1, true, 4, true> : decode_main_kernel<1, false, 4, true>)
                              : (sliding ? decode_main_kernel<1, true, 4> : decode_main_kernel<1, false, 4>))
                  : (gq > 4   ? (sliding ? decode_main_kernel<2, true> : decode_main_kernel<2, false>)
                     : gq < 4 ? (sliding ? decode_main_kernel<1, true, 2, true> : decode_main_kernel<1, false, 2, true>)
                              : (sliding ? decode_main_kernel<1, true> : decode_main_kernel<1, false>));
  if (start != nullptr)  // timestamps of the dispatch itself, no extra packets on the stream
    hipExtLaunchKernelGGL(kernel, grid, block, 0, stream, start, stop, 0, c.groups, c.n_quant, qq, c.Wq, c.S16, words.batch, words.heads, words.groups, words.magic, c, corr, part, oo);
  else
    hipLaunchKernelGGL(kernel, grid, block, 0, stream, c.groups, c.n_quant, qq, c.Wq, c.S16, words.batch, words.heads, words.groups, words.magic, c, corr, part, oo);
  return hipGetLastError() == hipSuccess ? KVLINC_OK : KVLINC_EHIP;
}

}  // namespace kvlinc

