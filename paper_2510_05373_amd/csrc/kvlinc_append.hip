// Append / flush path: Hadamard rotation of new values, 2-bit (or 4-bit) quantization of what leaves the fp16 window,
// tile packing, and the update of the linear-correction states (Sec. 3.1, Obs. 3; Sec. 2, Eq. 1; Sec. 3.2, Eq. 5-6;
// Sec. 3.3: the cache is quantized only after attention has used the new token).
//
// An append of one token, or of a few, is one launch (append_token_kernel): most of them only store rows, a sequence whose
// window is full has its group quantized and its states updated by two workgroups per kv head.  An append of more rows is two
// launches: append_quantize_kernel, one workgroup per group of 128 tokens, writes the records (and looks at every new row
// and stores those that stay in an empty window); append_states_kernel then walks the groups of a (sequence, kv head), adds
// their contributions to the states and commits the counters.
//
// This translation unit is compiled with floating-point contraction off: the rotation and the quantizer are
// bit-exact contracts (one binary32 rounding per written operation).
#include <hip/hip_runtime.h>

#include "kvlinc_internal.h"
#include "kvlinc_mfma.h"
#include "kvlinc_quantize.h"

#pragma clang fp contract(off)

namespace kvlinc {
namespace {

constexpr int kThreads = 512;
constexpr int kWaves = kThreads / 64;
constexpr int kParts = 2;      // workgroups that share the states of one (sequence, kv head): the two halves of phi
constexpr int kListCap = kThreads;  // items one workgroup looks at per round (one per thread)

__device__ inline bool nonfinite_bits(half_t x) {
  return (__builtin_bit_cast(unsigned short, x) & 0x7C00u) == 0x7C00u;
}

// One wave rotates one 128-vector: lane l holds elements 2l and 2l+1.  Stage order h = 1, 2, ..., 64 with
// (x[i], x[i+h]) <- (x[i] + x[i+h], x[i] - x[i+h]) for (i & h) == 0, then the binary32 scale and one rounding to fp16.
// NV independent vectors at once.
template <int NV>
__device__ inline void fwht128_wave(float (&x)[2 * NV], int lane) {  // x[2 u], x[2 u + 1]: vector u
#pragma unroll
  for (int u = 0; u < NV; ++u) {
    const float a = x[2 * u] + x[2 * u + 1], b = x[2 * u] - x[2 * u + 1];
    x[2 * u] = a;
    x[2 * u + 1] = b;
  }
  lane_butterflies<2 * NV>(x, lane);  // element stride h = 2, 4, ..., 64 is lane stride h / 2
  const float c = 0x1.6a09e6p-4f;  // fl32(1/sqrt(128))
#pragma unroll
  for (int u = 0; u < 2 * NV; ++u) {
    x[u] = x[u] * c;
    // The contract rounds the product to binary32 first and to fp16 afterwards.  Keep the two roundings apart: a
    // fused multiply-and-convert instruction would round the exact product once and differ in rare near-tie cases.
    asm volatile("" : "+v"(x[u]));
  }
}

// Every (sequence, kv head) has kParts * n_chunks owners in the grid, fixed by the launch shape alone (n_chunks > 1
// only in a bulk append of few sequences, whose groups are then shared out in chunks).  Each owner reads the sequence's
// counters once and counts itself in at the sequence's first split_done entry when it is done -- with a vote in the
// upper half of the counter if it found a fault; the counters change only in the arrival that completes the count
// (kParts n_chunks H_kv), i.e. after every reader has read them, and only if nobody voted against.  The launch that
// quantizes an append of several rows raises bit 30 of the same entry for a sequence with a non-finite new row: it reads as a
// vote.  The completing arrival leaves the entry at zero, as the decode kernel, which uses the same entries in the
// same way, expects.
constexpr int kFaultVote = 1 << 16;
constexpr int kScanFlag = 1 << 30;
__device__ inline bool arrive(const kvlinc_cache& c, int b, int n_chunks, bool vote, bool* clean) {
  int* counter = c.split_done + (long long)b * c.H_kv;
  const int before = __hip_atomic_fetch_add(counter, vote ? 1 + kFaultVote : 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  *clean = !vote && before < kFaultVote;
  return (before & (kFaultVote - 1)) == kParts * n_chunks * c.H_kv - 1;
}
// An arrival where nobody votes (the pairs' own counts share the entries then, see kPairShift).
__device__ inline bool arrive_unanimous(const kvlinc_cache& c, int b, int n_chunks) {
  const int before = __hip_atomic_fetch_add(c.split_done + (long long)b * c.H_kv, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  return (before & (kFaultVote - 1)) == kParts * n_chunks * c.H_kv - 1;
}
__device__ inline void finish(const kvlinc_cache& c, int b, int nq, int n, const AppendPlan& plan, bool clean) {
  if (clean && plan.err == 0 && n > 0) {
    c.n_quant[b] = nq + plan.n_flush;
    c.n_res[b] = plan.new_res;
  }
  c.split_done[(long long)b * c.H_kv] = 0;
}
__device__ inline bool scan_flag(const kvlinc_cache& c, int b) {
  return (__hip_atomic_load(c.split_done + (long long)b * c.H_kv, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM) & kScanFlag) != 0;
}

// One wave: raw key and rotated value of one new token into its window slot (values live 4 slots per channel: slot u,
// channel ch at [u / 4][ch][u % 4]).  Nothing of a row with a non-finite key or rotated value is stored; returns
// whether the row was such a row.
// (kk, vv: the lane's two elements of the new key and value row)
__device__ inline bool store_window_row(half_t* __restrict__ k_win, half_t* __restrict__ v_win, int slot, uint32_t kk,
                                        uint32_t vv, int lane) {
  const half2_t v2 = as_h2(vv);
  float x[2] = {(float)v2[0], (float)v2[1]};
  fwht128_wave<1>(x, lane);
  const half_t r0 = (half_t)x[0], r1 = (half_t)x[1];
  const bool mine = nonfinite_pair(kk) || nonfinite_bits(r0) || nonfinite_bits(r1);
  if (__builtin_amdgcn_ballot_w64(mine) != 0) return true;
  *reinterpret_cast<uint32_t*>(k_win + (long long)slot * kHeadDim + 2 * lane) = kk;
  v_win[((long long)(slot >> 2) * kHeadDim + 2 * lane) * 4 + (slot & 3)] = r0;
  v_win[((long long)(slot >> 2) * kHeadDim + 2 * lane + 1) * 4 + (slot & 3)] = r1;
  return false;
}
__device__ inline bool store_window_row(half_t* __restrict__ k_win, half_t* __restrict__ v_win, int slot,
                                        const half_t* __restrict__ ks, const half_t* __restrict__ vs, int lane) {
  return store_window_row(k_win, v_win, slot, *reinterpret_cast<const uint32_t*>(ks + 2 * lane),
                          *reinterpret_cast<const uint32_t*>(vs + 2 * lane), lane);
}

// An append of few rows: at most kFewRows a call, and at most kFewRowsOfAllHeads of them over the kv heads of a sequence (each
// workgroup that flushes looks at all of these; so does each wave that stores, where the values slide).  Measured, us a call in
// one launch and in the two that more rows take (2 bits, correction; every sequence flushes once in 128 / T calls):
//   1 kv head, 64 sequences       2 rows  5.0   9.1    8 rows  7.5  10.3
//   8 kv heads, 144 sequences     2 rows  9.5  18.0    8 rows 23.8  26.5
//   the same, sliding values      2 rows 13.0  50.2    8 rows 30.7  55.8
//   32 kv heads, 32 sequences     6 rows 18.9  21.9    8 rows 28.9  24.1
constexpr int kFewRows = 8, kFewRowsOfAllHeads = 192;

// Is a new row of any kv head of sequence b non-finite (key) or beyond fp16 once rotated (value)?  (n: new rows of the
// sequence, ROWS: what T may be at most; row i of the sequence is row i % n of head i / n.)  The caller's waves share the rows:
// wave `first` of `stride` takes the rows first, first + stride, ..., eight per batch; the verdicts of the waves still have to
// be combined.  g: a head whose row may be read in place of a missing one.
template <int N>
struct NewRows {
  uint32_t k[N], v[N];
};
template <int ROWS, int N>
__device__ inline void request_new_rows(NewRows<N>& r, const kvlinc_cache& c, int b, int g, const half_t* __restrict__ k_new,
                                        const half_t* __restrict__ v_new, int T, int n, int lane, int i0, int stride) {
#pragma unroll
  for (int u = 0; u < N; ++u) {
    const int i = i0 + stride * u;
    const int g2 = ROWS == 1 ? i : i / n;
    const bool exists = g2 < c.H_kv;
    long long row = (long long)b * c.H_kv + (exists ? g2 : g);
    if (ROWS > 1) row = row * T + (exists ? i - g2 * n : 0);
    r.k[u] = *reinterpret_cast<const uint32_t*>(k_new + row * kHeadDim + 2 * lane);
    r.v[u] = *reinterpret_cast<const uint32_t*>(v_new + row * kHeadDim + 2 * lane);
  }
}
// All T rows of one (sequence, kv head).
template <int ROWS>
__device__ inline void request_rows_of_pair(NewRows<ROWS>& r, int p, const half_t* __restrict__ k_new, const half_t* __restrict__ v_new, int T, int lane) {
#pragma unroll
  for (int u = 0; u < ROWS; ++u) {
    if (u >= T) break;
    const long long row = (long long)p * T + u;
    r.k[u] = *reinterpret_cast<const uint32_t*>(k_new + row * kHeadDim + 2 * lane);
    r.v[u] = *reinterpret_cast<const uint32_t*>(v_new + row * kHeadDim + 2 * lane);
  }
}
template <int N>
__device__ inline bool new_rows_bad(const NewRows<N>& r, int lane) {
  constexpr int kBatch = N < 4 ? N : 4;
  bool refuse = false;
  // A rotated value is at most sum_i |v_i| / sqrt(128): rows whose sum of magnitudes stays below
  // 65504 sqrt(128) cannot overflow fp16 and need no rotation here (a non-finite v makes the sum non-finite).
  float mag[N];
#pragma unroll
  for (int u = 0; u < N; ++u) {
    refuse |= nonfinite_pair(r.k[u]);
    const half2_t h = as_h2(r.v[u]);
    mag[u] = fabsf((float)h[0]) + fabsf((float)h[1]);
  }
#pragma unroll
  for (int u = 0; u < N; ++u) mag[u] = wave_allsum(mag[u]);
#pragma unroll
  for (int u0 = 0; u0 < N; u0 += kBatch) {
    bool small = true;
#pragma unroll
    for (int u = 0; u < kBatch; ++u) small &= mag[u0 + u] < 741000.0f;
    if (small) continue;
    float x[2 * kBatch];
#pragma unroll
    for (int u = 0; u < kBatch; ++u) {
      const half2_t h = as_h2(r.v[u0 + u]);
      x[2 * u] = (float)h[0];
      x[2 * u + 1] = (float)h[1];
    }
    fwht128_wave<kBatch>(x, lane);
#pragma unroll
    for (int u = 0; u < 2 * kBatch; ++u) refuse |= nonfinite_bits((half_t)x[u]);
  }
  return refuse;
}
template <int ROWS>
__device__ inline bool new_rows_of_all_heads_bad(const kvlinc_cache& c, int b, int g, const half_t* __restrict__ k_new,
                                                 const half_t* __restrict__ v_new, int T, int n, int lane, int first, int stride) {
  bool refuse = false;
  for (int i0 = first; i0 < c.H_kv * n; i0 += stride * 8) {
    NewRows<8> r;
    request_new_rows<ROWS>(r, c, b, g, k_new, v_new, T, n, lane, i0, stride);
    refuse |= new_rows_bad(r, lane);
  }
  return refuse;
}

// The same by one wave for the first n of the T rows of every kv head of sequence b, 32 rows on their way at a time (8 of them and a
// sum for each row took 20 us a launch for 32 kv heads of 2 rows, where this takes 12.5).  A row of magnitudes up to 5788 = 0x6DA7 cannot leave
// fp16 when it is rotated (128 * 5788 < 65504 sqrt(128)); where one is larger, the wave takes the way above.
__device__ inline bool few_rows_of_all_heads_bad(const kvlinc_cache& c, int b, const half_t* __restrict__ k_new,
                                                 const half_t* __restrict__ v_new, int T, int n, int lane) {
  typedef unsigned short ushort2_t __attribute__((ext_vector_type(2)));
  constexpr int kBatch = 32;
  const long long first = (long long)b * c.H_kv * T;
  ushort2_t k_max = {0, 0}, v_max = {0, 0};
  int at = 0;  // row within its head
  for (int i0 = 0; i0 < c.H_kv * T; i0 += kBatch) {
    uint32_t k[kBatch], v[kBatch];
#pragma unroll
    for (int u = 0; u < kBatch; ++u) {
      // (rows from n on, and beyond the last head, are not the caller's: the sequence's first row instead)
      const long long row = first + (at < n && i0 + u < c.H_kv * T ? i0 + u : 0);
      if (++at == T) at = 0;
      k[u] = *reinterpret_cast<const uint32_t*>(k_new + row * kHeadDim + 2 * lane);
      v[u] = *reinterpret_cast<const uint32_t*>(v_new + row * kHeadDim + 2 * lane);
    }
#pragma unroll
    for (int u = 0; u < kBatch; ++u) {
      k_max = __builtin_elementwise_max(k_max, __builtin_bit_cast(ushort2_t, k[u] & 0x7fff7fffu));
      v_max = __builtin_elementwise_max(v_max, __builtin_bit_cast(ushort2_t, v[u] & 0x7fff7fffu));
    }
  }
  if (__builtin_amdgcn_ballot_w64(k_max[0] >= 0x7c00 || k_max[1] >= 0x7c00) != 0) return true;
  if (__builtin_amdgcn_ballot_w64(v_max[0] > 0x6da7 || v_max[1] > 0x6da7) == 0) return false;
  return new_rows_of_all_heads_bad<kFewRows>(c, b, 0, k_new, v_new, T, n, lane, 0, 1);
}

struct Counters {
  int nq, nr, n;
  AppendPlan plan;
};
__device__ inline Counters read_counters(const kvlinc_cache& c, int b, const int32_t* __restrict__ n_new, int T, int keep) {
  Counters r;
  r.nq = c.n_quant[b];
  r.nr = c.n_res[b];
  int n = n_new ? n_new[b] : T;
  r.n = n < 0 ? 0 : (n > T ? T : n);
  r.plan = plan_append(r.nq, r.nr, r.n, c.R, keep, c.max_groups);
  return r;
}

// An append of few rows that quantizes nothing: one wave stores the new rows of one (sequence, kv head) behind the window's
// tokens.  The slots are dead storage until the counters advance, and they do not advance if any head of the sequence
// votes against.
// known: the sequence's counters as read before, and the lane's elements of the pair's new rows, read ahead into `rows`.
template <bool SLIDING, int ROWS>
__device__ inline void light_item(const kvlinc_cache& c, int p, const half_t* __restrict__ k_new,
                                  const half_t* __restrict__ v_new, const int32_t* __restrict__ n_new, int T, int lane,
                                  const Counters* known, NewRows<ROWS>& rows) {
  const int b = p / c.H_kv;
  if (known == nullptr) request_rows_of_pair(rows, p, k_new, v_new, T, lane);
  const Counters s = known != nullptr ? *known : read_counters(c, b, n_new, T, 0);
  half_t* k_win = reinterpret_cast<half_t*>(c.k_res) + (long long)p * c.R * kHeadDim;
  half_t* v_win = reinterpret_cast<half_t*>(c.v_res) + (long long)p * c.R * kHeadDim;
  bool row_bad = false;
  // With the sliding value window the value slots behind the key window are live (the values of the newest group's
  // last tokens): nothing may be written there before the new rows of ALL kv heads of the sequence have been looked at
  // (a single row: it is looked at before it is stored anyway).
  if (SLIDING && c.H_kv * s.n > 1)
    row_bad = __builtin_amdgcn_ballot_w64(ROWS == 1 ? new_rows_of_all_heads_bad<1>(c, b, p % c.H_kv, k_new, v_new, 1, 1, lane, 0, 1)
                                                    : few_rows_of_all_heads_bad(c, b, k_new, v_new, T, s.n, lane)) != 0;
#pragma unroll
  for (int r = 0; r < ROWS; ++r) {
    if (r >= s.n || row_bad) break;
    row_bad = store_window_row(k_win, v_win, s.nr + r, rows.k[r], rows.v[r], lane);
  }
  if (lane == 0) {
    if (row_bad) atomicOr(c.status, KVLINC_ST_NONFINITE);
    bool clean;
    if (arrive(c, b, 1, row_bad, &clean)) finish(c, b, s.nq, s.n, s.plan, clean);
  }
}

// ---- the window after an append of several rows --------------------------------------------------------------------
// Stream index u counts the old window tokens first, then the new rows.  Slot s of the window takes the row with
// u = s + n_flush if that row is a new one.  With the sliding value window the newest 128 tokens keep their fp16 values, token
// t in slot t % 128 (n_quant is a multiple of 128): the other value slots take the new rows among the last 128 that were
// quantized in this call, u = s + n_flush - 128 (old window tokens lie in their slots already).
// A workgroup of 64 NW threads writes the slots of one (sequence, kv head); st, ok: its LDS.  A row that is not finite is not
// stored; returns whether this thread saw one.  Ends with a barrier.
template <int NW, bool SLIDING>
__device__ __forceinline__ bool store_window(const kvlinc_cache& c, long long bh, const half_t* __restrict__ k_src,
                                             const half_t* __restrict__ v_src, int nr, int n, const AppendPlan& plan,
                                             half_t (*st)[kRowH], int* ok, int wave, int lane) {
  half_t* k_win = reinterpret_cast<half_t*>(c.k_res) + bh * c.R * kHeadDim;
  half_t* v_win = reinterpret_cast<half_t*>(c.v_res) + bh * c.R * kHeadDim;
  const int tid = 64 * wave + lane;
  const int first_new = max(plan.n_flush, nr), end = nr + n;
  const RowLane rl = row_lane(lane);
  const int in_pass = 4 * rl.rho + 2 * rl.ip + rl.b;
  bool bad = false;
  for (int pass = wave; 16 * pass < c.R; pass += NW) {
    const int s = 16 * pass + in_pass;
    const int u = s + plan.n_flush;
    const bool key = s < c.R && u >= first_new && u < end;
    const int uv = u - kGroup;
    const bool old = SLIDING && !key && uv >= max(nr, end - kGroup) && uv < plan.n_flush;
    const bool any = key || old;
    if (__builtin_amdgcn_ballot_w64(any) == 0) {
      if (rl.q == 0 && s < kGroup) ok[s] = 0;
      continue;
    }
    const long long row = any ? (key ? u : uv) - nr : 0;
    Row kr, vr;
    if (any) {
      load_row(kr, k_src + row * kHeadDim, rl.q);
      load_row(vr, v_src + row * kHeadDim, rl.q);
    } else {
#pragma unroll
      for (int m = 0; m < 4; ++m) kr.p[m] = vr.p[m] = make_uint4(0, 0, 0, 0);
    }
    half2_t h[16];
    row_pairs(vr, h);
    rotate_rows(h, rl.q);
    bool mine = false;
#pragma unroll
    for (int m = 0; m < 4; ++m)
      mine |= nonfinite_pair(kr.p[m].x) || nonfinite_pair(kr.p[m].y) || nonfinite_pair(kr.p[m].z) || nonfinite_pair(kr.p[m].w);
#pragma unroll
    for (int i = 0; i < 16; ++i) mine |= nonfinite_pair(as_u32(h[i]));
    // (the verdict of the row: over its four lanes)
    uint32_t verdict = mine ? 1u : 0u;
    verdict |= dpp_u<kQuadSwap1>(verdict);
    verdict |= dpp_u<kQuadSwap2>(verdict);
    bad |= verdict != 0;
    const bool store = any && verdict == 0;
    if (store && key) {
#pragma unroll
      for (int m = 0; m < 4; ++m) *reinterpret_cast<uint4*>(k_win + (long long)s * kHeadDim + 32 * m + 8 * rl.q) = kr.p[m];
    }
#pragma unroll
    for (int m = 0; m < 4; ++m)
      *reinterpret_cast<uint4*>(&st[s][32 * m + 8 * rl.q]) = make_uint4(as_u32(h[4 * m]), as_u32(h[4 * m + 1]), as_u32(h[4 * m + 2]), as_u32(h[4 * m + 3]));
    if (rl.q == 0) ok[s] = store ? 1 : 0;
  }
  __syncthreads();
  // values: 4 slots of 2 channels are one 16-byte store where all 4 slots take a new row
  for (int it = tid; it < (c.R >> 2) * 64; it += 64 * NW) {
    const int s0 = 4 * (it >> 6), cp = it & 63;
    const int4 f = *reinterpret_cast<const int4*>(&ok[s0]);
    if ((f.x | f.y | f.z | f.w) == 0) continue;
    uint32_t r[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) r[i] = *reinterpret_cast<const uint32_t*>(&st[s0 + i][2 * cp]);
    half_t* dst = v_win + ((long long)(s0 >> 2) * kHeadDim + 2 * cp) * 4;
    if ((f.x & f.y & f.z & f.w) != 0) {
      *reinterpret_cast<uint4*>(dst) =
          make_uint4(__builtin_amdgcn_perm(r[1], r[0], 0x05040100u), __builtin_amdgcn_perm(r[3], r[2], 0x05040100u),
                     __builtin_amdgcn_perm(r[1], r[0], 0x07060302u), __builtin_amdgcn_perm(r[3], r[2], 0x07060302u));
    } else {
      const int fl[4] = {f.x, f.y, f.z, f.w};
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (fl[i]) {
          dst[i] = as_h2(r[i])[0];
          dst[4 + i] = as_h2(r[i])[1];
        }
    }
  }
  __syncthreads();
  return bad;
}

// May append_quantize_kernel store the rows that stay in the window?  Only if no slot it writes is live whatever happens to
// the append: without the sliding value window, and where the old window's rows are not wanted any more.
__device__ __forceinline__ bool rows_stored_early(bool sliding, int nr, const AppendPlan& plan) {
  return !sliding && (plan.n_groups == 0 || nr == 0);
}

// ---- records of an append of several rows -------------------------------------------------------------------------
// One workgroup per (sequence, kv head) and group of the append, and one more for the rows that stay in the window.  The
// records lie beyond the counters: dead storage, whatever becomes of the append.  A key or rotated value that is not finite
// raises the sequence's flag (bit 30 of its first split_done entry), so that all workgroups of that sequence in the launch
// that follows refuse the append, whichever head or group the fault is in.
// Bound: the vector unit; 512 bytes in and 72 out per token and kv head come second.
// Workgroups of four waves, four per compute unit: 124 registers, and 38 KB of LDS because the record is put together where
// the window's rows have been (only a group that takes tokens from the window reads them, all of them before it writes).
// Measured, 16 prompts of 8192 tokens (8 kv heads; 611 MB): 130 us, 4.7 TB/s; 146 us with 50 KB and three workgroups a unit.  The
// calls around it: 460 -> 451 us there, 32 ragged prompts at 4 bits in three chunks (60 KB and two a unit before) 360 -> 343, one
// of 700 tokens 52.8 -> 49.7.
constexpr int kQuantWaves = 4;
template <bool SLIDING, int BITS>
__global__ __launch_bounds__(64 * kQuantWaves, 4) void append_quantize_kernel(kvlinc_cache c, const half_t* __restrict__ k_new,
                                                                            const half_t* __restrict__ v_new,
                                                                            const int32_t* __restrict__ n_new, int T, int keep,
                                                                            int per_pair, int first_pair) {
  using R = Rec<BITS>;
  constexpr int kStWords = kGroup * kRowH / 2;
  __shared__ __align__(16) uint32_t shared[kStWords > R::kWords ? kStWords : R::kWords];
  half_t (*st)[kRowH] = reinterpret_cast<half_t (*)[kRowH]>(shared);  // rotated rows of the window
  uint32_t* img = shared;                                             // the record, once they have been read
  __shared__ __align__(16) union {
    QuantLds<kQuantWaves> q;
    int ok[kGroup];
  } L;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int p = first_pair + blockIdx.x / per_pair, j = blockIdx.x % per_pair;
  const int b = p / c.H_kv;
  const long long bh = p;
  const Counters s = read_counters(c, b, n_new, T, keep);
  if (s.plan.err != 0 || s.n == 0 || j > s.plan.n_groups) return;
  const half_t* k_src = k_new + bh * (long long)T * kHeadDim;
  const half_t* v_src = v_new + bh * (long long)T * kHeadDim;
  bool bad;
  if (j < s.plan.n_groups) {
    const int valid = min(kGroup, s.plan.n_flush - j * kGroup);
    const int nrg = min(max(s.nr - j * kGroup, 0), valid);  // tokens of this group that come from the window (only if j == 0)
    const long long skip = (long long)j * kGroup + nrg - s.nr;  // first new row of the group
    if (nrg > 0) {
      stage_window_values<kQuantWaves>(reinterpret_cast<const half_t*>(c.v_res) + bh * c.R * kHeadDim, nrg, st, tid);
      __syncthreads();
    }
    bad = quantize_group<BITS, kQuantWaves>(reinterpret_cast<const half_t*>(c.k_res) + bh * c.R * kHeadDim, k_src + skip * kHeadDim,
                                            v_src + skip * kHeadDim, st, nrg, valid, L.q, img, wave, lane);
    const long long grp = (long long)(s.nq / kGroup) + j;
    uint4* rec = reinterpret_cast<uint4*>(c.groups + (bh * c.max_groups + grp) * R::kWords);
    for (int i = tid; i < R::kWords / 4; i += 64 * kQuantWaves) rec[i] = reinterpret_cast<const uint4*>(img)[i];
  } else if (rows_stored_early(SLIDING, s.nr, s.plan)) {
    bad = store_window<kQuantWaves, false>(c, bh, k_src, v_src, s.nr, s.n, s.plan, st, L.ok, wave, lane);
  } else {
    // only a look at the rows (they are stored by the next launch)
    bad = false;
    const RowLane rl = row_lane(lane);
    for (int u0 = max(s.plan.n_flush, s.nr) + 16 * wave; u0 < s.nr + s.n; u0 += 16 * kQuantWaves) {
      const int u = u0 + 4 * rl.rho + 2 * rl.ip + rl.b;
      if (u < s.nr + s.n) {
        Row kr, vr;
        load_row(kr, k_src + (long long)(u - s.nr) * kHeadDim, rl.q);
        load_row(vr, v_src + (long long)(u - s.nr) * kHeadDim, rl.q);
        half2_t h[16];
        row_pairs(vr, h);
        rotate_rows(h, rl.q);
#pragma unroll
        for (int m = 0; m < 4; ++m)
          bad |= nonfinite_pair(kr.p[m].x) || nonfinite_pair(kr.p[m].y) || nonfinite_pair(kr.p[m].z) || nonfinite_pair(kr.p[m].w);
#pragma unroll
        for (int i = 0; i < 16; ++i) bad |= nonfinite_pair(as_u32(h[i]));
      }
    }
  }
  if (__builtin_amdgcn_ballot_w64(bad) != 0 && lane == 0) atomicOr(c.split_done + (long long)b * c.H_kv, kScanFlag);
}

// ---- states (Eq. 5, Eq. 6) ----------------------------------------------------------------------------------------
// A workgroup of 8 waves owns one half of phi of a (sequence, kv head): the features 128 fp .. 128 fp + 127 of S and P (Eq. 6
// normalises each half by itself).  Per group of 128 tokens
//   logits[t][f] = sum_c (K - K_q)[t][c] W_k[c][f]   for the 128 features of the half,
//   phi = softmax over that half (Eq. 6),
//   S[f][c] += sum_t (phi s_t)[t][f] (code[t][c] - ctr) + sum_t phi[t][f] (z_t + ctr s_t),   P[f] += sum_t phi[t][f]   (Eq. 5)
// with V_q[t][c] = z_t + s_t code[t][c] and ctr = (2^BITS - 1) / 2 the centre of the code range, on
// v_mfma_f32_16x16x32_f16: products of binary16 operands are exact in it (the centred codes are multiples of 0.5, W_k is
// binary16, the key error and phi s are carried as two binary16 terms).  The instruction lines its 32 products and its
// addend up with the largest of them before it adds, so what it is given is kept small and of both signs: the two terms of
// the key error go to accumulators of their own, the products of every group start from a zero addend and are added to S
// by ordinary binary32 additions, and the codes are centred (the other part is the same for all channels of a row and is
// added once per call).
//
// Nothing but phi, W_k and the key scales passes through LDS: a lane reads the raw keys of its token and the tile words of its key codes
// straight into the layout of the A operand and forms the key error there; the value tile is the B operand of the S
// update as it lies in memory (the nibble hi|0|lo|1 is the FP4 number code - 1.5, one conversion gives two binary16
// numbers).  Tokens are dealt to the waves and to the rows of their tiles so that the four tokens a lane holds of a result
// are four neighbouring contraction positions of the S update:
//   wave w, row rho of its tile: token 16 (4 (w % 2) + rho % 4) + 4 (w / 2) + rho / 4;
//   phi in LDS: [feature][token % 16][token / 16];
//   S update: wave w owns the features 32 (w / 2) .. + 31 and the channels 64 (w % 2) .. + 63.
// Bound: the vector and the matrix instructions of a group one after the other (two waves per SIMD, all in the same phase):
// of the busy time 67 % vector, 37 % matrix, 10 % both at once; LDS 42 %.
// Measured, 16 prompts of 8192 tokens (8 kv heads): about 320 us of a call's 461 for the states, 370 to 440 single calls
// under a profiler as the clock goes (444 on average before the logits were laid out by hand, 407 now; 500 us before the terms were
// formed with mixed-precision fused multiply-adds, the four contractions chained and the loads freed of execution masks; 1742 us, quantization included,
// when the same workgroups also quantized the group in LDS, each half for itself).  Two teams of four waves, one at the
// logits and the softmax while the other is at the update, took 10 % longer: one wave of a kind per SIMD does not hide its own latencies.
struct StateLds {
  half_t Wt[kRank / 2][kRowH];        // W_k of the half, [feature][channel]
  half_t ph[2][kRank / 2][kRowH];     // high / low term of phi s of the group, [feature][8 (token % 16) + token / 16]
  float red[2][kWaves][kRank / 2];    // sums of phi and of phi (z + ctr s) over each wave's tokens
};

// Which channel a lane's column of tile ct is.  QUAD: four neighbouring channels per lane, so that a row of S moves in
// 16-byte pieces -- a flush, which loads and stores S for every group (a step of 144 sequences of 1280 tokens 82.2 -> 81.2 us).
// The other order reads the value tile in whole lines and adds to S in whole lines: the walk over many groups (one prompt of
// 131072 tokens 505 us, 559 us with QUAD).
struct StateAcc {
  float4_t acc[2][4];  // S[32 (w / 2) + 16 ft + 4 kq + r][channel 64 (w % 2) + ...], ... = 16 ct + l16, or 4 l16 + ct (QUAD)
  float P[8], Z[8];    // sums over this lane's tokens of phi and of phi (z + ctr s), feature 16 fo + l16
};

// What a wave reads of a group; requested one group ahead, each part as soon as the one before has been used.
template <int BITS>
struct KeyError {
  uint4 k[4];                // raw keys of the lane's token, channels 32 kk + 8 kq .. + 7
  uint32_t code[BITS / 2][4];  // the tile words that hold their codes
};
template <int BITS>
struct ValueCodes {
  uint2 v[BITS / 2][4];  // value tile: the two words of the lane's channel of tile ct, quarter kq
};
struct ValueScales {
  uint4 mine;   // (s, z) of the lane's four tokens
  uint2 all;    // (s, z) of two tokens: the 64 lanes hold all of them
};

__device__ __forceinline__ int state_row_token(int wave, int rho) { return 16 * (4 * (wave & 1) + (rho & 3)) + 4 * (wave >> 1) + (rho >> 2); }

template <int BITS>
__device__ __forceinline__ void load_key_codes(KeyError<BITS>& e, const uint32_t* rec, int t, int kq) {
#pragma unroll
  for (int pl = 0; pl < BITS / 2; ++pl)
#pragma unroll
    for (int kk = 0; kk < 4; ++kk)
      e.code[pl][kk] = rec[Rec<BITS>::kKeyTile + kPlaneWords * pl + ((t >> 5) * 64 + (t & 15) + 16 * kk) * 4 + 2 * ((t >> 4) & 1) + (kq >> 1)];
}
template <int BITS>
__device__ __forceinline__ void load_key_rows(KeyError<BITS>& e, const half_t* __restrict__ row, int kq) {
#pragma unroll
  for (int kk = 0; kk < 4; ++kk) e.k[kk] = *reinterpret_cast<const uint4*>(row + 32 * kk + 8 * kq);
}
template <int BITS, bool QUAD>
__device__ __forceinline__ void load_value_codes(ValueCodes<BITS>& r, const uint32_t* rec, int wave, int lane) {
#pragma unroll
  for (int pl = 0; pl < BITS / 2; ++pl) {
    const uint32_t* tile = rec + Rec<BITS>::kValueTile + kPlaneWords * pl;
    if constexpr (QUAD) {
#pragma unroll
      for (int ct = 0; ct < 4; ++ct)  // channel 16 n + j, n = 4 (w % 2) + l16 / 4, j = 4 (l16 % 4) + ct
        r.v[pl][ct] = *reinterpret_cast<const uint2*>(
            tile + ((2 * (wave & 1) + ((lane >> 3) & 1)) * 64 + 4 * (lane & 3) + ct + 16 * (lane >> 4)) * 4 + 2 * ((lane >> 2) & 1));
    } else {
#pragma unroll
      for (int m = 0; m < 2; ++m) {
        const uint4 t = reinterpret_cast<const uint4*>(tile)[(2 * (wave & 1) + m) * 64 + lane];
        r.v[pl][2 * m] = make_uint2(t.x, t.y);
        r.v[pl][2 * m + 1] = make_uint2(t.z, t.w);
      }
    }
  }
}
template <int BITS>
__device__ __forceinline__ void load_value_scales(ValueScales& r, const uint32_t* rec, int wave, int lane) {
  const uint32_t* sz = rec + Rec<BITS>::kValueSZ;
  r.mine = *reinterpret_cast<const uint4*>(sz + 8 * (4 * (wave >> 1) + (lane >> 4)) + 4 * (wave & 1));
  r.all = *reinterpret_cast<const uint2*>(sz + 2 * lane);
}

// FP4 numbers code - 1.5 from a tile word (see the record layout): the codes with p % 2 = 0; shifted left by one, p % 2 = 1.
// `pick` is 0xAAAAAAAA, opaque to constant folding (code_bits_mask): the form then is a single bit-field insert.
__device__ __forceinline__ uint32_t code_bits_mask() {
  uint32_t m = 0xAAAAAAAAu;
  asm volatile("" : "+s"(m));
  return m;
}
__device__ __forceinline__ uint32_t fp4_codes(uint32_t w, uint32_t pick) { return 0x11111111u ^ (pick & (w ^ 0x11111111u)); }

// 1.0f in a scalar register, opaque to constant folding: a fused multiply-add with it keeps the form that takes a binary16 operand
// as it is (v_fma_mix), where a plain subtraction would convert it first.  (As inline assembly the same instructions came with
// 75 idle ones a group, which the compiler puts between an assembly statement and the use of its result.)
__device__ __forceinline__ float opaque_one() {
  float one = 1.0f;
  asm("" : "+s"(one));
  return one;
}
typedef float float2_t __attribute__((ext_vector_type(2)));
// x0, x1 as two binary16 terms each, high terms in h, what they leave in l (the differences are exact).  (The conversion is
// of both numbers at once: one by one they would be fused into the operations that x0 and x1 come from, which rounds
// another number, and the low terms would belong to other high terms in rare near-tie cases: 2e-4 of the largest entry of S, ten
// times what the element-wise state tests let pass.  Making h opaque as well gives the same bits and costs 0.7 to 1.2 % of a prompt.)
__device__ __forceinline__ void two_terms(float x0, float x1, float one, uint32_t& h, uint32_t& l) {
  const half2_t t = __builtin_convertvector((float2_t{x0, x1}), half2_t);
  h = as_u32(t);
  l = as_u32(half2_t{(half_t)__builtin_fmaf(-(float)t[0], one, x0), (half_t)__builtin_fmaf(-(float)t[1], one, x1)});
}
// The same of the products a0 b0, a1 b1: the low terms are what the high ones leave of the exact products.
__device__ __forceinline__ void two_terms_of_products(float a0, float b0, float a1, float b1, uint32_t& h, uint32_t& l) {
  const half2_t t = __builtin_convertvector((float2_t{a0 * b0, a1 * b1}), half2_t);
  h = as_u32(t);
  l = as_u32(half2_t{(half_t)__builtin_fmaf(a0, b0, -(float)t[0]), (half_t)__builtin_fmaf(a1, b1, -(float)t[1])});
}
template <int BYTE>
__device__ __forceinline__ half2_t fp4_to_h2(uint32_t w, float scale) { return __builtin_amdgcn_cvt_scalef32_pk_f16_fp4(w, scale, BYTE); }

// Key scales s and mid-points z + ctr s of a group in binary32, channel by channel: formed once per group by 64 threads from
// the record's scales and zero-points, two channels each.
struct KeyAffine {
  float s[kHeadDim], mid[kHeadDim];
};
template <int BITS>
__device__ __forceinline__ void store_key_affine(KeyAffine& a, uint32_t scales, uint32_t zeros, int pair) {
  const half2_t s = as_h2(scales), z = as_h2(zeros);
  *reinterpret_cast<float2*>(&a.s[2 * pair]) = make_float2((float)s[0], (float)s[1]);
  *reinterpret_cast<float2*>(&a.mid[2 * pair]) = make_float2(__builtin_fmaf((float)s[0], Rec<BITS>::kCentre, (float)z[0]),
                                                             __builtin_fmaf((float)s[1], Rec<BITS>::kCentre, (float)z[1]));
}

// logits of the wave's 16 tokens: d[ft][r] = token row 4 kq + r, feature 16 ft + l16.  (All rows are finite: a token that does
// not exist is a copy of the last one, see states_item.)
template <int BITS>
__device__ __forceinline__ void state_logits(const KeyError<BITS>& e, const KeyAffine& ka, const StateLds& L, uint32_t pick, int lane, float4_t (&d)[8]) {
  const int l16 = lane & 15, kq = lane >> 4;
  const float one = opaque_one();
  float4_t lo[8];
#pragma unroll
  for (int ft = 0; ft < 8; ++ft) d[ft] = lo[ft] = float4_t{0.f, 0.f, 0.f, 0.f};
  // The key error of a step is formed between the products of the one before, and W_k is read two tiles ahead: laid out by hand, in
  // pieces that the compiler may not mix, because it puts every pair of products behind the read of its operand otherwise.  (16
  // prompts of 8192 tokens 540 -> 521 us, 32 ragged ones at 4 bits in three calls 403 -> 388, one of 700 tokens 61.6 -> 59.5, the
  // rest of the calls included.  Not for the update, whose operands a step ahead took 3 % longer; and the softmax of a group laid
  // between the products of the next, at 100 more lines, was no faster: beside a matrix instruction the vector unit issues at half
  // its rate.)
  uint32_t op[2][8];  // high terms, low terms
  float4_t s4, m4;
  auto read_affine = [&](int kk, int half) __attribute__((always_inline)) {
    s4 = *reinterpret_cast<const float4_t*>(&ka.s[32 * kk + 8 * kq + 4 * half]);
    m4 = *reinterpret_cast<const float4_t*>(&ka.mid[32 * kk + 8 * kq + 4 * half]);
  };
  auto key_error = [&](int kk, int half) __attribute__((always_inline)) {
    asm volatile("" : "+v"(s4));
    const uint32_t w2 = fp4_codes(e.code[0][kk] << (kq & 1), pick);
    constexpr float kStep = BITS == 2 ? 1.0f : 4.0f;
    float2_t c0, c1;
    if (half == 0) {
      c0 = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(w2, kStep, 0);
      c1 = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(w2, kStep, 1);
    } else {
      c0 = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(w2, kStep, 2);
      c1 = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(w2, kStep, 3);
    }
    if constexpr (BITS == 4) {  // code - 7.5 = 4 (high digit - 1.5) + (low digit - 1.5)
      const uint32_t wl = fp4_codes(e.code[1][kk] << (kq & 1), pick);
      float2_t a0, a1;
      if (half == 0) {
        a0 = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(wl, 1.0f, 0);
        a1 = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(wl, 1.0f, 1);
      } else {
        a0 = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(wl, 1.0f, 2);
        a1 = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(wl, 1.0f, 3);
      }
      c0[0] += a0[0]; c0[1] += a0[1]; c1[0] += a1[0]; c1[1] += a1[1];
    }
    const half2_t ka2 = as_h2(half == 0 ? e.k[kk].x : e.k[kk].z), kb2 = as_h2(half == 0 ? e.k[kk].y : e.k[kk].w);
    // K - (z + s code), the difference to the mid-point first
    two_terms(__builtin_fmaf(-s4.x, c0[0], __builtin_fmaf((float)ka2[0], one, -m4.x)),
              __builtin_fmaf(-s4.y, c0[1], __builtin_fmaf((float)ka2[1], one, -m4.y)), one, op[kk & 1][2 * half], op[kk & 1][4 + 2 * half]);
    two_terms(__builtin_fmaf(-s4.z, c1[0], __builtin_fmaf((float)kb2[0], one, -m4.z)),
              __builtin_fmaf(-s4.w, c1[1], __builtin_fmaf((float)kb2[1], one, -m4.w)), one, op[kk & 1][2 * half + 1], op[kk & 1][4 + 2 * half + 1]);
  };
  half8_t w[3];
  auto weights = [&](int i) { return *reinterpret_cast<const half8_t*>(&L.Wt[16 * (i & 7) + l16][32 * (i >> 3) + 8 * kq]); };
  w[0] = weights(0);
  w[1] = weights(1);
  read_affine(0, 0);
  key_error(0, 0);
  read_affine(0, 1);
  key_error(0, 1);
#pragma unroll
  for (int i = 0; i < 32; ++i) {
    const int kk = i >> 3, ft = i & 7;
    if (i + 2 < 32) w[(i + 2) % 3] = weights(i + 2);
    asm volatile("" : "+v"(w[i % 3]));
    const uint32_t* o = op[kk & 1];
    const half8_t ah = __builtin_bit_cast(half8_t, make_uint4(o[0], o[1], o[2], o[3]));
    const half8_t al = __builtin_bit_cast(half8_t, make_uint4(o[4], o[5], o[6], o[7]));
    lo[ft] = __builtin_amdgcn_mfma_f32_16x16x32_f16(al, w[i % 3], lo[ft], 0, 0, 0);
    d[ft] = __builtin_amdgcn_mfma_f32_16x16x32_f16(ah, w[i % 3], d[ft], 0, 0, 0);
    if (kk < 3) {
      if (ft == 1 || ft == 4) read_affine(kk + 1, ft == 4 ? 1 : 0);
      if (ft == 3 || ft == 6) key_error(kk + 1, ft == 6 ? 1 : 0);
    }
    __builtin_amdgcn_sched_barrier(0);
  }
#pragma unroll
  for (int ft = 0; ft < 8; ++ft) d[ft] += lo[ft];
}

// reductions over the 16 lanes of a row, result in every lane
// (four at once: each step is one instruction, and an instruction that reads another lane's register comes at least two
// instructions after the one that wrote it)
__device__ __forceinline__ void row16_max(float (&v)[4]) {
#define KVLINC_MAX_STEP(ror)                                              \
  "v_max_f32_dpp %0, %0, %0 row_ror:" #ror " row_mask:0xf bank_mask:0xf\n\t" \
  "v_max_f32_dpp %1, %1, %1 row_ror:" #ror " row_mask:0xf bank_mask:0xf\n\t" \
  "v_max_f32_dpp %2, %2, %2 row_ror:" #ror " row_mask:0xf bank_mask:0xf\n\t" \
  "v_max_f32_dpp %3, %3, %3 row_ror:" #ror " row_mask:0xf bank_mask:0xf\n\t"
  asm("s_nop 1\n\t" KVLINC_MAX_STEP(1) KVLINC_MAX_STEP(2) KVLINC_MAX_STEP(4) KVLINC_MAX_STEP(8)
      : "+v"(v[0]), "+v"(v[1]), "+v"(v[2]), "+v"(v[3]));
#undef KVLINC_MAX_STEP
}
__device__ __forceinline__ float row16_sum(float v) {
  v += dpp_f<kRowRor1>(v);
  v += dpp_f<kRowRor2>(v);
  v += dpp_f<kRowRor4>(v);
  return v + dpp_f<kRowRor8>(v);
}
__device__ __forceinline__ float rows_sum(float v) {  // over the lanes l, l ^ 16, l ^ 32, l ^ 48
  v += __shfl_xor(v, 16, 64);
  return v + __shfl_xor(v, 32, 64);
}

// A power of two F with max_t s_t F in [2^13, 2^14): phi s_t F then fills binary16's range from the top, and the two binary16
// terms it is carried in leave 2^-38 of the largest entry (rather than 2^-25 of one).
__device__ __forceinline__ float scale_factor(const ValueScales& sz, float& inv) {
  uint32_t m = max(sz.all.x & 0xffffu, sz.all.y & 0xffffu);  // (scales are not negative: their bit patterns order like they do)
  m = max(m, dpp_u<kRowRor1>(m));
  m = max(m, dpp_u<kRowRor2>(m));
  m = max(m, dpp_u<kRowRor4>(m));
  m = max(m, dpp_u<kRowRor8>(m));
  const auto a = __builtin_amdgcn_permlane16_swap(m, m, false, false);
  m = max(a[0], a[1]);
  const auto b = __builtin_amdgcn_permlane32_swap(m, m, false, false);
  const float top = (float)__builtin_bit_cast(half_t, (unsigned short)max(b[0], b[1]));
  const int e = (int)(__builtin_bit_cast(uint32_t, top) >> 23);  // biased
  const int k = top > 0.0f ? 13 - (e - 127) : 0;
  inv = __builtin_bit_cast(float, (uint32_t)(127 - k) << 23);
  return __builtin_bit_cast(float, (uint32_t)(127 + k) << 23);
}

// phi of the wave's tokens (softmax over the half) from the logits; its sums, and phi s F in two binary16 terms to LDS.
template <int BITS>
__device__ __forceinline__ void state_softmax(float4_t (&d)[8], const ValueScales& sz, float F, int valid, StateAcc& st, StateLds& L, int wave, int lane) {
  constexpr float kCentre = Rec<BITS>::kCentre, kLog2e = 1.4426950408889634f;
  const int l16 = lane & 15, kq = lane >> 4, jj = 4 * (wave >> 1) + kq;
  const uint32_t szw[4] = {sz.mine.x, sz.mine.y, sz.mine.z, sz.mine.w};
  float m[4], sum[4], inv[4], wz[4], ws[4];
#pragma unroll
  for (int r = 0; r < 4; ++r)
    m[r] = fmaxf(fmaxf(fmaxf(d[0][r], d[1][r]), fmaxf(d[2][r], d[3][r])), fmaxf(fmaxf(d[4][r], d[5][r]), fmaxf(d[6][r], d[7][r])));
  row16_max(m);
  // (The difference first: it is never positive, whatever its rounding.  fma(d, log2(e), -m log2(e)) saves an instruction per
  // element, 1 to 1.8 % of a prompt, but leaves the rounding of m log2(e) in the exponent, which passes what a power of two can
  // hold where adapters in the hundreds make logits of 1e9.)
#pragma unroll
  for (int ft = 0; ft < 8; ++ft)
#pragma unroll
    for (int r = 0; r < 4; ++r) d[ft][r] = __builtin_amdgcn_exp2f((d[ft][r] - m[r]) * kLog2e);
#pragma unroll
  for (int r = 0; r < 4; ++r) sum[r] = ((d[0][r] + d[1][r]) + (d[2][r] + d[3][r])) + ((d[4][r] + d[5][r]) + (d[6][r] + d[7][r]));
#pragma unroll
  for (int r = 0; r < 4; ++r) sum[r] = row16_sum(sum[r]);
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const half2_t t = as_h2(szw[r]);
    const bool live = 16 * (4 * (wave & 1) + r) + jj < valid;
    float rc = __builtin_amdgcn_rcpf(sum[r]);  // 1 <= sum <= 128: one Newton step gives the binary32 quotient
    rc = __builtin_fmaf(__builtin_fmaf(-sum[r], rc, 1.0f), rc, rc);
    inv[r] = live ? rc : 0.0f;
    wz[r] = inv[r] * __builtin_fmaf((float)t[0], kCentre, (float)t[1]);
    ws[r] = inv[r] * ((float)t[0] * F);
  }
#pragma unroll
  for (int fo = 0; fo < 8; ++fo) {
    const float4_t e = d[fo];
    uint2 h4, l4;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      st.P[fo] = __builtin_fmaf(e[r], inv[r], st.P[fo]);
      st.Z[fo] = __builtin_fmaf(e[r], wz[r], st.Z[fo]);
    }
    two_terms_of_products(e[0], ws[0], e[1], ws[1], h4.x, l4.x);
    two_terms_of_products(e[2], ws[2], e[3], ws[3], h4.y, l4.y);
    *reinterpret_cast<uint2*>(&L.ph[0][16 * fo + l16][8 * jj + 4 * (wave & 1)]) = h4;
    *reinterpret_cast<uint2*>(&L.ph[1][16 * fo + l16][8 * jj + 4 * (wave & 1)]) = l4;
  }
}

// eight centred codes of one channel as a B operand: tokens 16 i + tok, i = 0..7
__device__ __forceinline__ half8_t codes_operand(uint32_t w, float scale) {
  const half2_t a = fp4_to_h2<0>(w, scale), b = fp4_to_h2<1>(w, scale), c = fp4_to_h2<2>(w, scale), d = fp4_to_h2<3>(w, scale);
  return half8_t{a[0], a[1], b[0], b[1], c[0], c[1], d[0], d[1]};
}

// S += (phi s F)^T (code - ctr) / F over the group's tokens: four contractions of 32 tokens, summed in the matrix cores.  (Error
// of S against 64 bits over 300 to 20000 tokens 1.6e-7 to 2.1e-7; 1.8e-7 to 2.9e-7 when each contraction started from zero and
// was added to S by itself, which also took 96 more vector instructions per wave and group.)
template <int BITS>
__device__ __forceinline__ void state_update(const ValueCodes<BITS>& vc, float inv_F, StateAcc& st, const StateLds& L, uint32_t pick, int wave, int lane) {
  const int l16 = lane & 15, kq = lane >> 4, fw = 32 * (wave >> 1);
  float4_t dd[2][4];
#pragma unroll
  for (int wd = 0; wd < 2; ++wd) {
    const int tok0 = 4 * ((2 * kq + wd) & 3) + 2 * (kq >> 1);
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      const int step = 2 * wd + b;
      half8_t aH[2], aL[2];
#pragma unroll
      for (int ft = 0; ft < 2; ++ft) {
        aH[ft] = *reinterpret_cast<const half8_t*>(&L.ph[0][fw + 16 * ft + l16][8 * (tok0 + b)]);
        aL[ft] = *reinterpret_cast<const half8_t*>(&L.ph[1][fw + 16 * ft + l16][8 * (tok0 + b)]);
      }
#pragma unroll
      for (int ct = 0; ct < 4; ++ct) {
        half8_t op;
#pragma unroll
        for (int pl = 0; pl < BITS / 2; ++pl) {
          const uint32_t w = wd ? vc.v[pl][ct].y : vc.v[pl][ct].x;
          const half8_t o = codes_operand(fp4_codes(b ? w << 1 : w, pick), BITS == 4 && pl == 0 ? 4.0f : 1.0f);
          op = pl == 0 ? o : op + o;
        }
#pragma unroll
        for (int ft = 0; ft < 2; ++ft) {
          if (step == 0) dd[ft][ct] = float4_t{0.f, 0.f, 0.f, 0.f};
          dd[ft][ct] = __builtin_amdgcn_mfma_f32_16x16x32_f16(aL[ft], op, dd[ft][ct], 0, 0, 0);
          dd[ft][ct] = __builtin_amdgcn_mfma_f32_16x16x32_f16(aH[ft], op, dd[ft][ct], 0, 0, 0);
          if (step == 3) {
#pragma unroll
            for (int r = 0; r < 4; ++r) st.acc[ft][ct][r] = __builtin_fmaf(dd[ft][ct][r], inv_F, st.acc[ft][ct][r]);
          }
        }
      }
    }
  }
}

// W_k of the half goes to LDS transposed: a lane's B operand (8 channels of one feature) is then one 16-byte read.  Thread:
// two features (a wave reads whole rows of W_k), 16 channels.  Requested first, put down when it has arrived.
struct WkRegs {
  uint32_t x[16];
};
__device__ __forceinline__ void request_wk(WkRegs& w, const kvlinc_cache& c, int g, int fp, int tid) {
  const uint32_t* W0 = reinterpret_cast<const uint32_t*>(c.Wk) + ((long long)g * 2 + fp) * kHeadDim * (kRank / 4) +
                       (16 * (tid >> 6)) * (kRank / 4) + (tid & 63);
#pragma unroll
  for (int i = 0; i < 16; ++i) w.x[i] = W0[i * (kRank / 4)];
}
__device__ __forceinline__ void put_wk(const WkRegs& w, StateLds& L, int tid) {
  const int f = 2 * (tid & 63), c0 = 16 * (tid >> 6);
#pragma unroll
  for (int i = 0; i < 16; i += 8) {
    uint32_t lo[4], hi[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      lo[e] = __builtin_amdgcn_perm(w.x[i + 2 * e + 1], w.x[i + 2 * e], 0x05040100u);
      hi[e] = __builtin_amdgcn_perm(w.x[i + 2 * e + 1], w.x[i + 2 * e], 0x07060302u);
    }
    *reinterpret_cast<uint4*>(&L.Wt[f][c0 + i]) = make_uint4(lo[0], lo[1], lo[2], lo[3]);
    *reinterpret_cast<uint4*>(&L.Wt[f + 1][c0 + i]) = make_uint4(hi[0], hi[1], hi[2], hi[3]);
  }
}

template <bool QUAD>
__device__ __forceinline__ int state_channel(int wave, int l16, int ct) { return 64 * (wave & 1) + (QUAD ? 4 * l16 + ct : 16 * ct + l16); }
// The state rows of this wave into registers (fresh: a chunk that starts from zero).  P_old: P of feature tid (threads 0 .. 127).
template <bool QUAD>
__device__ __forceinline__ void load_states(const kvlinc_cache& c, long long bh, int fp, bool fresh, StateAcc& st, float& P_old, int wave, int lane) {
  const int tid = 64 * wave + lane, l16 = lane & 15, kq = lane >> 4;
#pragma unroll
  for (int fo = 0; fo < 8; ++fo) st.P[fo] = st.Z[fo] = 0.0f;
  const half_t* tiles = reinterpret_cast<const half_t*>(c.S16) + bh * kRank * kHeadDim;
#pragma unroll
  for (int ft = 0; ft < 2; ++ft) {
    const int frow = (kRank / 2) * fp + 32 * (wave >> 1) + 16 * ft + 4 * kq;  // first of the 4 rows of S this lane holds
    const int tile = ((frow >> 6) * 2 + (wave & 1)) * 16 + ((frow & 63) >> 2);
    if (fresh) {
#pragma unroll
      for (int ct = 0; ct < 4; ++ct) st.acc[ft][ct] = float4_t{0.f, 0.f, 0.f, 0.f};
    } else if (c.S != nullptr) {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float* row = c.S + (bh * kRank + frow + r) * kHeadDim;
        if constexpr (QUAD) {
          const float4 v = *reinterpret_cast<const float4*>(row + state_channel<true>(wave, l16, 0));
          st.acc[ft][0][r] = v.x; st.acc[ft][1][r] = v.y; st.acc[ft][2][r] = v.z; st.acc[ft][3][r] = v.w;
        } else {
#pragma unroll
          for (int ct = 0; ct < 4; ++ct) st.acc[ft][ct][r] = row[state_channel<false>(wave, l16, ct)];
        }
      }
    } else {
#pragma unroll
      for (int ct = 0; ct < 4; ++ct) {
        const half4_t t16 = *reinterpret_cast<const half4_t*>(tiles + ((long long)tile * 64 + (state_channel<QUAD>(wave, l16, ct) & 63)) * 4);
#pragma unroll
        for (int r = 0; r < 4; ++r) st.acc[ft][ct][r] = (float)t16[r];
      }
    }
  }
  P_old = 0.0f;
  if (tid < kRank / 2 && !fresh) P_old = c.P[bh * kRank + (kRank / 2) * fp + tid];
}

// End: the sums of phi over all waves -- P to memory, the term of the code centres into S -- and S to its fp32 master
// copy (if the cache keeps one), row-major, and to the binary16 tiles the decode kernel reads: tile (64-feature block, channel
// half hh, feature step fb) holds S[64 block + 4 fb + k][64 hh + l] at [l][k].  An entry beyond the binary16 range is stored as
// +-65504 and reported in the status word.  share: this is one chunk's share, added to the fp32 state with atomic additions.
// share_phi_sums first, then a barrier, then store_states.
__device__ __forceinline__ void share_phi_sums(StateLds& L, StateAcc& st, int wave, int lane) {
  const int l16 = lane & 15;
#pragma unroll
  for (int fo = 0; fo < 8; ++fo) {
    st.P[fo] = rows_sum(st.P[fo]);
    st.Z[fo] = rows_sum(st.Z[fo]);
  }
  if (lane < 16) {
#pragma unroll
    for (int fo = 0; fo < 8; ++fo) {
      L.red[0][wave][16 * fo + l16] = st.P[fo];
      L.red[1][wave][16 * fo + l16] = st.Z[fo];
    }
  }
}
template <bool QUAD>
__device__ __forceinline__ void store_states(const kvlinc_cache& c, long long bh, int fp, bool share, const StateLds& L, const StateAcc& st, float P_old, int wave, int lane) {
  const int tid = 64 * wave + lane, l16 = lane & 15, kq = lane >> 4;
  if (tid < kRank / 2) {
    float add = 0.0f;
#pragma unroll
    for (int w2 = 0; w2 < kWaves; ++w2) add += L.red[0][w2][tid];
    float* dst = c.P + bh * kRank + (kRank / 2) * fp + tid;
    if (share) __hip_atomic_fetch_add(dst, add, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    else *dst = P_old + add;
  }
  half_t* tiles = reinterpret_cast<half_t*>(c.S16) + bh * kRank * kHeadDim;
  bool out_of_range = false;
#pragma unroll
  for (int ft = 0; ft < 2; ++ft) {
    const int fl = 32 * (wave >> 1) + 16 * ft + 4 * kq, frow = (kRank / 2) * fp + fl;
    const int tile = ((frow >> 6) * 2 + (wave & 1)) * 16 + ((frow & 63) >> 2);
    float z[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w2 = 0; w2 < kWaves; ++w2) {
      const float4 zz = *reinterpret_cast<const float4*>(&L.red[1][w2][fl]);
      z[0] += zz.x; z[1] += zz.y; z[2] += zz.z; z[3] += zz.w;
    }
    half_t t16[4][4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      float* row = c.S + (bh * kRank + frow + r) * kHeadDim;
      float v[4];
#pragma unroll
      for (int ct = 0; ct < 4; ++ct) {
        v[ct] = st.acc[ft][ct][r] + z[r];
        out_of_range |= !(fabsf(v[ct]) <= 65504.0f);
        t16[ct][r] = (half_t)fminf(fmaxf(v[ct], -65504.0f), 65504.0f);
        if (share) __hip_atomic_fetch_add(row + state_channel<QUAD>(wave, l16, ct), v[ct], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        else if (!QUAD && c.S != nullptr) row[state_channel<QUAD>(wave, l16, ct)] = v[ct];
      }
      if (QUAD && c.S != nullptr) *reinterpret_cast<float4*>(row + state_channel<true>(wave, l16, 0)) = make_float4(v[0], v[1], v[2], v[3]);
    }
    if (!share) {
#pragma unroll
      for (int ct = 0; ct < 4; ++ct)  // (QUAD: neighbouring pieces, which the compiler joins)
        *reinterpret_cast<half4_t*>(tiles + ((long long)tile * 64 + (state_channel<QUAD>(wave, l16, ct) & 63)) * 4) =
            half4_t{t16[ct][0], t16[ct][1], t16[ct][2], t16[ct][3]};
    }
  }
  if (!share && __builtin_amdgcn_ballot_w64(out_of_range) != 0 && lane == 0) atomicOr(c.status, KVLINC_ST_STATE_RANGE);
}

// ---- an append of several rows: states, window, counters ------------------------------------------------------------
// Owners as in `arrive`.  Nobody votes here: the verdict is the flag that the quantizing launch has left.  The owners of a
// (sequence, kv head) also count themselves in at the pair's own entry (bits 20 .. 27; it shares the entry with the
// sequence's count for head 0): the last of them, when every part has read the old window's keys and every chunk has added
// its share, stores the pair's window rows and, after chunks, its binary16 tiles.
constexpr int kPairShift = 20;

struct StatesLds {
  StateLds st;
  KeyAffine ka[2];  // of a group (by group parity)
  __align__(16) int ok[kGroup];
  int heavy[kListCap];
  int n_heavy, last_flag;
};

template <bool SLIDING, int BITS>
__device__ void states_item(const kvlinc_cache& c, StatesLds& L, int item, const half_t* __restrict__ k_new,
                            const half_t* __restrict__ v_new, const int32_t* __restrict__ n_new, int T, int keep,
                            int n_chunks, int tid) {
  using R = Rec<BITS>;
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, kq = lane >> 4;
  const int ck = item % n_chunks, fp = (item / n_chunks) % kParts, p = item / (n_chunks * kParts);
  const int b = p / c.H_kv, g = p % c.H_kv;
  const long long bh = p;
  const Counters s = read_counters(c, b, n_new, T, keep);
  const AppendPlan plan = s.plan;
  // Chunks (few sequences, many groups): the groups of the call are shared out evenly among n_chunks owners per
  // part, each of which forms the sum of its groups' contributions to S and P and adds it to the fp32 state in memory
  // with atomic additions (the order of the additions, and with it the last bits of S, then differ from run to run).
  // A call with one chunk in use -- every cache without an fp32 state -- keeps S in registers from load to store.
  const int per_chunk = (plan.n_groups + n_chunks - 1) / n_chunks;
  const int j_first = ck * per_chunk, j_last = min(plan.n_groups, j_first + per_chunk);
  const bool chunked = plan.n_groups > per_chunk;  // more than one chunk has groups
  const bool has_work = c.S16 != nullptr && j_first < j_last;
  const half_t* k_res = reinterpret_cast<const half_t*>(c.k_res) + bh * c.R * kHeadDim;
  const half_t* k_src = k_new + bh * (long long)T * kHeadDim;
  const half_t* v_src = v_new + bh * (long long)T * kHeadDim;
  const uint32_t* rec0 = c.groups + (bh * c.max_groups + s.nq / kGroup) * (long long)R::kWords;
  if (has_work) {
    StateAcc acc;
    float P_old;
    KeyError<BITS> ke;
    ValueCodes<BITS> vc;
    ValueScales vs;
    uint32_t k_s = 0, k_z = 0;  // scales and zero-points of two channels (threads 0 .. 63)
    const uint32_t pick = code_bits_mask();
    const int my_t = state_row_token(wave, l16);
    // (Every lane requests: a load that only some lanes or waves issue makes the compiler wait for all loads at the next use of
    // any, a trip to memory per group.  A lane whose token does not exist takes the last one's key and codes, an ordinary
    // key error; its weight is 0.  The padding's own codes would not do: their distance from a key can leave binary16, and
    // a weight of 0 does not remove the NaN that comes of it.)
    auto request_keys = [&](int j) {
      const int u = min(j * kGroup + my_t, plan.n_flush - 1), t = u - j * kGroup;
      const half_t* row = u < s.nr ? k_res + (long long)u * kHeadDim : k_src + (long long)(u - s.nr) * kHeadDim;
      const uint32_t* rec = rec0 + (long long)j * R::kWords;
      load_key_rows<BITS>(ke, row, kq);
      load_key_codes<BITS>(ke, rec, t, kq);
      k_s = rec[R::kKeyScale + lane];
      k_z = rec[R::kKeyZero + lane];
    };
    request_keys(j_first);
    load_value_scales<BITS>(vs, rec0 + (long long)j_first * R::kWords, wave, lane);
    load_value_codes<BITS, false>(vc, rec0 + (long long)j_first * R::kWords, wave, lane);
    WkRegs wk;
    request_wk(wk, c, g, fp, tid);
    load_states<false>(c, bh, fp, chunked, acc, P_old, wave, lane);
    put_wk(wk, L.st, tid);
    if (tid < 64) store_key_affine<BITS>(L.ka[0], k_s, k_z, tid);
    lds_barrier();
    for (int j = j_first; j < j_last; ++j) {
      const int valid = min(kGroup, plan.n_flush - j * kGroup), par = (j - j_first) & 1;
      const int nxt = min(j + 1, j_last - 1);  // (past the last group: a request that hits the caches)
      float4_t d[8];
      state_logits<BITS>(ke, L.ka[par], L.st, pick, lane, d);
      float inv_F;
      const float F = scale_factor(vs, inv_F);
      request_keys(nxt);
      lds_barrier();  // every wave has read the phi of the group before
      state_softmax<BITS>(d, vs, F, valid, acc, L.st, wave, lane);
      load_value_scales<BITS>(vs, rec0 + (long long)nxt * R::kWords, wave, lane);
      if (tid < 64) store_key_affine<BITS>(L.ka[par ^ 1], k_s, k_z, tid);
      lds_barrier();
      state_update<BITS>(vc, inv_F, acc, L.st, pick, wave, lane);
      load_value_codes<BITS, false>(vc, rec0 + (long long)nxt * R::kWords, wave, lane);
    }
    share_phi_sums(L.st, acc, wave, lane);
    lds_barrier();
    store_states<false>(c, bh, fp, chunked, L.st, acc, P_old, wave, lane);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // (the additions of every wave are done before this owner counts itself in)
  }
  __syncthreads();
  const bool stored = rows_stored_early(SLIDING, s.nr, plan);
  const bool pair_work = !stored || (chunked && c.S16 != nullptr);
  if (pair_work) {
    if (tid == 0) {
      const int owners = kParts * n_chunks;
      const int before = __hip_atomic_fetch_add(c.split_done + bh, 1 << kPairShift, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
      L.last_flag = ((before >> kPairShift) & 255) == owners - 1 ? 1 : 0;
      if (L.last_flag != 0) __hip_atomic_fetch_add(c.split_done + bh, -(owners << kPairShift), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    }
    __syncthreads();
    if (L.last_flag != 0) {
      if (chunked && c.S16 != nullptr) {
        bool out_of_range = false;
        for (int i = tid; i < 128 * 64; i += kThreads) {
          const int t = i >> 6, l = i & 63;
          const int f0 = 64 * (t >> 5) + 4 * (t & 15), ch = 64 * ((t >> 4) & 1) + l;
          half4_t t16;
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            const float v = __hip_atomic_load(c.S + (bh * kRank + f0 + k) * kHeadDim + ch, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
            out_of_range |= !(fabsf(v) <= 65504.0f);
            t16[k] = (half_t)fminf(fmaxf(v, -65504.0f), 65504.0f);
          }
          *reinterpret_cast<half4_t*>(reinterpret_cast<half_t*>(c.S16) + bh * kRank * kHeadDim + ((long long)t * 64 + l) * 4) = t16;
        }
        if (__builtin_amdgcn_ballot_w64(out_of_range) != 0 && lane == 0) atomicOr(c.status, KVLINC_ST_STATE_RANGE);
      }
      if (!stored) store_window<kWaves, SLIDING>(c, bh, k_src, v_src, s.nr, s.n, plan, L.st.ph[0], L.ok, wave, lane);
    }
  }
  if (tid == 0 && arrive_unanimous(c, b, n_chunks)) finish(c, b, s.nq, s.n, plan, true);
}

// One launch serves every sequence: item it of the grid's list is part (it / 8) % kParts of the pair
// (it / (8 kParts)) * 8 + it % 8 of (sequence, kv head), and workgroup x owns the items x, x + G, x + 2 G, ...: the parts of a
// pair sit on one XCD (workgroups are dealt to the 8 XCDs in turn, and G is a multiple of 8), whose L2 then serves
// the keys and records that all of them read.
// SLIDING: the variant for caches with the sliding value window (KVLINC_FLAG_SLIDING_VALUES) is a kernel of its own;
// BITS: so is the one for caches with 4-bit codes.
template <bool SLIDING, int BITS>
__global__ __launch_bounds__(kThreads) void append_states_kernel(kvlinc_cache c, const half_t* __restrict__ k_new,
                                                                  const half_t* __restrict__ v_new,
                                                                  const int32_t* __restrict__ n_new, int T, int keep,
                                                                  int n_chunks) {
  extern __shared__ __align__(16) unsigned char lds_raw[];
  StatesLds& L = *reinterpret_cast<StatesLds*>(lds_raw);
  const int tid = threadIdx.x;
  const uint32_t n_pairs = (uint32_t)c.B * (uint32_t)c.H_kv;
  const uint32_t owners = kParts * n_chunks;  // per (sequence, kv head)
  const uint32_t n_items = owners * 8u * ((n_pairs + 7u) / 8u);
  const uint32_t G = gridDim.x;
  for (uint32_t k0 = 0; k0 * G < n_items; k0 += kListCap) {
    if (tid == 0) L.n_heavy = 0;
    __syncthreads();
    // every thread looks at one item: what needs the workgroup is listed, the rest is counted in at once
    const uint32_t it = (k0 + tid) * G + blockIdx.x;
    if (it < n_items) {
      const int own = (int)((it >> 3) % owners);  // (part, chunk): part = own / n_chunks, chunk = own % n_chunks
      const uint32_t p = (it / (8u * owners)) * 8u + (it & 7u);
      if (p < n_pairs) {
        const int b = (int)(p / (uint32_t)c.H_kv);
        const Counters s = read_counters(c, b, n_new, T, keep);
        const bool refused = s.plan.err == 0 && s.n > 0 && scan_flag(c, b);
        if (s.plan.err != 0 || s.n == 0 || refused || (s.plan.n_groups == 0 && rows_stored_early(SLIDING, s.nr, s.plan))) {
          const int fault = s.plan.err != 0 ? s.plan.err : refused ? KVLINC_ST_NONFINITE : 0;
          if (fault != 0 && own == 0) atomicOr(c.status, fault);
          bool clean;
          if (arrive(c, b, n_chunks, fault != 0, &clean)) finish(c, b, s.nq, s.n, s.plan, clean);
        } else {
          L.heavy[atomicAdd(&L.n_heavy, 1)] = (int)(p * owners) + own;
        }
      }
    }
    __syncthreads();
    const int n_heavy = L.n_heavy;
    for (int i = 0; i < n_heavy; ++i) {
      states_item<SLIDING, BITS>(c, L, L.heavy[i], k_new, v_new, n_new, T, keep, n_chunks, tid);
      __syncthreads();
    }
    __syncthreads();
  }
}

// ---- an append of one token, or of few ------------------------------------------------------------------------------
template <int BITS>
struct TokenLds {
  StateLds st;
  QuantLds<kWaves> q;
  __align__(16) uint32_t img[Rec<BITS>::kWords];
  __align__(16) KeyAffine ka;
  float row[kWaves][kHeadDim];  // new rows read ahead
  int light[kListCap], heavy[kListCap], heavy_nq[kListCap], heavy_nr[kListCap];  // (heavy_nr: n_res + 256 n)
  int n_light, n_heavy, last_flag;
  int refuse[kWaves];
  // the item that thread w looked at is a light one whose new row wave w has read ahead; the sequence's counters as that
  // thread read them
  int ahead[kWaves], ahead_nq[kWaves], ahead_nr[kWaves], ahead_n[kWaves];
};

// The window of one (sequence, kv head) is full, or the n new rows fill it: its 128 tokens become a group, the last 128 - nr of
// them from the new rows.  Two owners, one per half of phi; both quantize the group (the record feeds both halves of the state
// update), each writes half of the record.
// Bound: latency, a chain of loads and phases on a few compute units.  So everything is requested at once, in the order in
// which it is wanted; the verdict on the new rows, the staged values and the keys' minima share the first barrier; and the owner
// counts itself in as soon as it has read the window, so that the answer is there when the states are done.  Measured (144
// sequences of 1280 tokens, where nearly every launch has one that flushes): 16.3 us from the start of the launch, 20.5 us when
// the rows, the window and the states were requested one after the other and the count came last.
template <bool SLIDING, int BITS, int ROWS>
__device__ void flush_item(const kvlinc_cache& c, TokenLds<BITS>& L, int item, int nq, int nr, int n, const half_t* __restrict__ k_new,
                           const half_t* __restrict__ v_new, int T, int tid) {
  using R = Rec<BITS>;
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, kq = lane >> 4;
  const int fp = item % kParts, p = item / kParts;
  const int b = p / c.H_kv, g = p % c.H_kv;
  const long long bh = p;
  const AppendPlan plan = plan_append(nq, nr, n, c.R, 0, c.max_groups);
  const half_t* k_res = reinterpret_cast<const half_t*>(c.k_res) + bh * c.R * kHeadDim;
  auto key_row = [&](int t) {  // (one row: it only arrives at a full window)
    return ROWS == 1 || t < nr ? k_res + (long long)t * kHeadDim : k_new + (bh * T + t - nr) * kHeadDim;
  };
  const bool states_live = c.S16 != nullptr;
  // (Nothing is stored to global memory before the verdict on the new rows.)
  constexpr int kAhead = ROWS == 1 ? 1 : 4;
  NewRows<kAhead> rows;  // the first 8 (32) of the sequence's rows
  request_new_rows<ROWS>(rows, c, b, g, k_new, v_new, T, n, lane, wave, kWaves);
  KeyTile<kWaves> keys;
#pragma unroll
  for (int i = 0; i < 32 / kWaves; ++i)
    keys.raw[i] = *reinterpret_cast<const uint4*>(key_row(key_token<kWaves>(i, wave, lane)) + 8 * l16);
  StateAcc acc;
  float P_old = 0.0f;
  KeyError<BITS> ke;
  WkRegs wk;
  {
    WindowValues<kWaves> win;
    request_window_values<kWaves>(win, reinterpret_cast<const half_t*>(c.v_res) + bh * c.R * kHeadDim, kGroup, tid);
    if (states_live) {
      load_key_rows<BITS>(ke, key_row(state_row_token(wave, l16)), kq);
      request_wk(wk, c, g, fp, tid);
      load_states<true>(c, bh, fp, false, acc, P_old, wave, lane);
    }
    // A flush changes live state (S, P, the window's first slot) in every kv head: the new row of every kv head of this
    // sequence is looked at first; the verdict is the same in all workgroups of the sequence.
    bool bad = new_rows_bad(rows, lane);
    if (c.H_kv * n > kAhead * kWaves) bad |= new_rows_of_all_heads_bad<ROWS>(c, b, g, k_new, v_new, T, n, lane, wave + kAhead * kWaves, kWaves);
    const bool refuse = __builtin_amdgcn_ballot_w64(bad) != 0;
    if (lane == 0) L.refuse[wave] = refuse ? 1 : 0;
    key_minmax<kWaves>(keys, kGroup, L.q, wave, lane);
    put_window_values<kWaves>(win, kGroup, L.st.ph[0], tid);
  }
  lds_barrier();
  {
    int refused = 0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) refused |= L.refuse[w];
    if (refused != 0) {
      if (tid == 0) {
        if (fp == 0) atomicOr(c.status, KVLINC_ST_NONFINITE);
        bool clean;
        if (arrive(c, b, 1, true, &clean)) finish(c, b, nq, n, plan, false);
      }
      return;
    }
  }
  // the record (its image in LDS): key parameters by two waves, values by all, then the key codes
  if (tid < kGroup) {
    key_params<BITS, kWaves>(L.q, tid, L.img);
    const half_t* img16 = reinterpret_cast<const half_t*>(L.img);
    const float s = (float)img16[2 * R::kKeyScale + tid], z = (float)img16[2 * R::kKeyZero + tid];
    L.ka.s[tid] = s;
    L.ka.mid[tid] = __builtin_fmaf(s, R::kCentre, z);
  }
  {
    const RowLane rl = row_lane(lane);
    const int t = value_pass_token(wave, rl);
    Row w;
    load_row(w, L.st.ph[0][t], rl.q);
    half2_t h[16];
    row_pairs(w, h);
    if (ROWS > 1 && __builtin_amdgcn_ballot_w64(t >= nr) != 0) {  // (the slots from nr on hold something else)
#pragma unroll
      for (int m = 0; m < 4; ++m) w.p[m] = make_uint4(0, 0, 0, 0);
      if (t >= nr) load_row(w, v_new + (bh * T + t - nr) * kHeadDim, rl.q);
      half2_t fresh[16];
      row_pairs(w, fresh);
      rotate_rows(fresh, rl.q);
#pragma unroll
      for (int e = 0; e < 16; ++e) h[e] = t < nr ? h[e] : fresh[e];
    }
    quantize_value_pass<BITS>(h, wave, rl, lane, L.img);
  }
  lds_barrier();
  key_codes<BITS, kWaves>(keys, kGroup, L.q, wave, lane, L.img);
  if (states_live) {
    put_wk(wk, L.st, tid);
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) asm volatile("" : "+v"(ke.k[kk].x), "+v"(ke.k[kk].y), "+v"(ke.k[kk].z), "+v"(ke.k[kk].w));  // (they have arrived, too)
  }
  lds_barrier();
  // every wave has the window's rows: count this part in.  The arrival that completes the sequence stores the new rows -- raw key,
  // rotated value -- that stay in the window, from slot 0 on, for all its kv heads and commits.
  int before = 0;
  if (tid == 0) before = __hip_atomic_fetch_add(c.split_done + (long long)b * c.H_kv, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  {
    uint4* rec = reinterpret_cast<uint4*>(c.groups + (bh * c.max_groups + nq / kGroup) * R::kWords);
    constexpr int kHalf = R::kWords / 8;
    for (int i = kHalf * fp + tid; i < kHalf * (fp + 1); i += kThreads) rec[i] = reinterpret_cast<const uint4*>(L.img)[i];
  }
  ValueCodes<BITS> vc;
  float inv_F = 1.0f;
  const uint32_t pick = code_bits_mask();
  if (states_live) {
    ValueScales vs;
    load_key_codes<BITS>(ke, L.img, state_row_token(wave, l16), kq);
    load_value_scales<BITS>(vs, L.img, wave, lane);
    load_value_codes<BITS, true>(vc, L.img, wave, lane);
    const float F = scale_factor(vs, inv_F);
    float4_t d[8];
    state_logits<BITS>(ke, L.ka, L.st, pick, lane, d);
    state_softmax<BITS>(d, vs, F, kGroup, acc, L.st, wave, lane);
    share_phi_sums(L.st, acc, wave, lane);
  }
  if (tid == 0) L.last_flag = (before & (kFaultVote - 1)) == kParts * c.H_kv - 1 ? (before < kFaultVote ? 2 : 1) : 0;
  lds_barrier();
  const int flag = L.last_flag;
  if (states_live) {
    state_update<BITS>(vc, inv_F, acc, L.st, pick, wave, lane);
    store_states<true>(c, bh, fp, false, L.st, acc, P_old, wave, lane);
  }
  if (flag == 2) {
    for (int i = wave; i < c.H_kv * n; i += kWaves) {
      const int g2 = ROWS == 1 ? i : i / n, r = i - g2 * n, u = nr + r;
      // (Sliding value window: the values of the new rows that were quantized stay in their slots u; the key that is stored along
      // with them lands in a dead one.)
      if (ROWS > 1 && !SLIDING && u < kGroup) continue;
      const long long bh2 = (long long)b * c.H_kv + g2;
      store_window_row(reinterpret_cast<half_t*>(c.k_res) + bh2 * c.R * kHeadDim, reinterpret_cast<half_t*>(c.v_res) + bh2 * c.R * kHeadDim,
                       u % kGroup, k_new + (bh2 * T + r) * kHeadDim, v_new + (bh2 * T + r) * kHeadDim, lane);
    }
  }
  if (flag != 0 && tid == 0) finish(c, b, nq, n, plan, flag == 2);
}

// Items as in append_states_kernel, without chunks.
// ROWS: 1, or kFewRows for an append of 2 .. kFewRows rows (a kernel of its own, so that the generation step carries none of it).
// What the way to the counters and to the new rows takes stands first among the arguments, ahead of the cache that holds it too:
// the first 14 words are in scalar registers when a wave starts (kernarg preload, see build.py), the others a trip to memory away.
// (Here and in the decode kernel: a step of 1 sequence of 300 tokens 12.1 -> 11.75 us, 16 of 8k 25.2 -> 25.05, 144 of 1280 73.5 ->
// 73.0.)
template <bool SLIDING, int BITS, int ROWS>
__global__ __launch_bounds__(kThreads) void append_token_kernel(int32_t* n_quant, int32_t* n_res, const half_t* __restrict__ k_new,
                                                                 const half_t* __restrict__ v_new, const int32_t* __restrict__ n_new,
                                                                 int B, int H_kv, int R, int rows_T, kvlinc_cache cache) {
  kvlinc_cache c = cache;
  c.n_quant = n_quant; c.n_res = n_res; c.B = B; c.H_kv = H_kv; c.R = R;
  extern __shared__ __align__(16) unsigned char lds_raw[];
  TokenLds<BITS>& L = *reinterpret_cast<TokenLds<BITS>*>(lds_raw);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int T = ROWS == 1 ? 1 : rows_T;
  const uint32_t n_pairs = (uint32_t)c.B * (uint32_t)c.H_kv;  // at most 2^24
  const uint32_t n_items = kParts * 8u * ((n_pairs + 7u) / 8u);
  const uint32_t G = gridDim.x;

  for (uint32_t k0 = 0; k0 * G < n_items; k0 += kListCap) {
    if (tid == 0) {
      L.n_light = 0;
      L.n_heavy = 0;
    }
    if (tid < kWaves) L.ahead[tid] = 0;
    __syncthreads();
    // Wave w requests the new rows of the pair of the item that thread w looks at in the first round while the sequence's
    // counters are on their way (most such appends only store them into the window).  One row goes straight to LDS,
    // 4 bytes per lane.
    int pre_p = -1;
    NewRows<ROWS> pre;
    if (k0 == 0 && (uint32_t)wave * G + blockIdx.x < n_items) {
      const uint32_t it = (uint32_t)wave * G + blockIdx.x;
      const uint32_t p = (it >> 4) * 8u + (it & 7u);
      if (((it >> 3) & 1u) == 0u && p < n_pairs) {
        pre_p = (int)p;
        if constexpr (ROWS == 1) {
          __builtin_amdgcn_global_load_lds(k_new + (long long)p * kHeadDim + 2 * lane, &L.row[wave][0], 4, 0, 0);
          __builtin_amdgcn_global_load_lds(v_new + (long long)p * kHeadDim + 2 * lane, &L.row[wave][64], 4, 0, 0);
        } else {
          request_rows_of_pair(pre, (int)p, k_new, v_new, T, lane);
        }
      }
    }
    // every thread looks at one item: what needs a wave or the workgroup is listed, the rest is counted in at once
    const uint32_t it = (k0 + tid) * G + blockIdx.x;
    if (it < n_items) {
      const int own = (int)((it >> 3) % kParts);
      const uint32_t p = (it / (8u * kParts)) * 8u + (it & 7u);
      if (p < n_pairs) {
        const int b = (int)(p / (uint32_t)c.H_kv);
        const Counters s = read_counters(c, b, n_new, T, 0);
        if (s.plan.err || s.n == 0) {
          if (s.plan.err && own == 0) atomicOr(c.status, s.plan.err);
          bool clean;
          if (arrive(c, b, 1, s.plan.err != 0, &clean)) finish(c, b, s.nq, s.n, s.plan, clean);
        } else if (s.plan.n_groups == 0) {
          if (own == 0) {
            if (k0 == 0 && tid < kWaves) {  // wave `tid` holds the row
              L.ahead[tid] = 1;
              L.ahead_nq[tid] = s.nq;
              L.ahead_nr[tid] = s.nr;
              L.ahead_n[tid] = s.n;
            } else {
              L.light[atomicAdd(&L.n_light, 1)] = (int)p;
            }
          } else {
            bool clean;
            if (arrive(c, b, 1, false, &clean)) finish(c, b, s.nq, s.n, s.plan, clean);
          }
        } else {
          const int at = atomicAdd(&L.n_heavy, 1);
          L.heavy[at] = (int)(p * kParts) + own;
          L.heavy_nq[at] = s.nq;
          L.heavy_nr[at] = s.nr + 256 * s.n;
        }
      }
    }
    __syncthreads();
    const int n_light = L.n_light, n_heavy = L.n_heavy;
    if (L.ahead[wave] != 0) {  // (the barrier has waited for the row)
      Counters s;
      s.nq = L.ahead_nq[wave];
      s.nr = L.ahead_nr[wave];
      s.n = L.ahead_n[wave];
      s.plan = plan_append(s.nq, s.nr, s.n, c.R, 0, c.max_groups);
      if constexpr (ROWS == 1) {
        pre.k[0] = __builtin_bit_cast(uint32_t, L.row[wave][lane]);
        pre.v[0] = __builtin_bit_cast(uint32_t, L.row[wave][64 + lane]);
      }
      light_item<SLIDING, ROWS>(c, pre_p, k_new, v_new, n_new, T, lane, &s, pre);
    }
    for (int i = wave; i < n_light; i += kThreads / 64) light_item<SLIDING, ROWS>(c, L.light[i], k_new, v_new, n_new, T, lane, nullptr, pre);
    for (int i = 0; i < n_heavy; ++i) {
      // (the thread index is made opaque here so that none of the flush's address arithmetic is hoisted to the top of
      // the kernel, where every launch -- most of them flush nothing -- would pay for it)
      int tid_here = tid;
      asm volatile("" : "+v"(tid_here));
      flush_item<SLIDING && (ROWS > 1), BITS, ROWS>(c, L, L.heavy[i], L.heavy_nq[i], L.heavy_nr[i] & 255, ROWS == 1 ? 1 : L.heavy_nr[i] >> 8,
                                                    k_new, v_new, T, tid_here);
      __syncthreads();
    }
    __syncthreads();
  }
}

template <typename F>
int launch_with_lds(F kernel, size_t lds) {
  // per device and cheap: set on every call rather than remembered in process state
  return hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) == hipSuccess
             ? KVLINC_OK : KVLINC_EHIP;
}

}  // namespace

int launch_append(const kvlinc_cache& c, const kvlinc_half* k_new, const kvlinc_half* v_new, const int32_t* n_new,
                  int T, int keep, hipStream_t stream) {
  static_assert(sizeof(TokenLds<2>) <= 160 * 1024 && sizeof(TokenLds<4>) <= 160 * 1024 && sizeof(StatesLds) <= 160 * 1024,
                "LDS budget of one CU");
  const bool sliding = (c.flags & KVLINC_FLAG_SLIDING_VALUES) != 0;
  const half_t* kk = reinterpret_cast<const half_t*>(k_new);
  const half_t* vv = reinterpret_cast<const half_t*>(v_new);
  const long long pairs = (long long)c.B * c.H_kv;
  if (keep == 0 && (T == 1 || (T <= kFewRows && T * (long long)c.H_kv <= kFewRowsOfAllHeads))) {
    const long long n_items = (long long)kParts * 8 * ((pairs + 7) / 8);
    // one workgroup per compute unit at most (the LDS of a flush fills most of one); items beyond that are taken
    // in further rounds by the same workgroups
    const int grid = (int)(n_items < 256 ? n_items : 256);
    typedef void (*kernel_t)(int32_t*, int32_t*, const half_t*, const half_t*, const int32_t*, int, int, int, int, kvlinc_cache);
    const kernel_t one = c.bits == 4 ? (sliding ? append_token_kernel<true, 4, 1> : append_token_kernel<false, 4, 1>)
                                     : (sliding ? append_token_kernel<true, 2, 1> : append_token_kernel<false, 2, 1>);
    const kernel_t few = c.bits == 4 ? (sliding ? append_token_kernel<true, 4, kFewRows> : append_token_kernel<false, 4, kFewRows>)
                                     : (sliding ? append_token_kernel<true, 2, kFewRows> : append_token_kernel<false, 2, kFewRows>);
    const kernel_t kernel = T == 1 ? one : few;
    const size_t lds = c.bits == 4 ? sizeof(TokenLds<4>) : sizeof(TokenLds<2>);
    if (launch_with_lds(kernel, lds) != KVLINC_OK) return KVLINC_EHIP;
    hipLaunchKernelGGL(kernel, dim3(grid), dim3(kThreads), lds, stream, c.n_quant, c.n_res, kk, vv, n_new, c.B, c.H_kv, c.R, T, c);
    return hipGetLastError() == hipSuccess ? KVLINC_OK : KVLINC_EHIP;
  }
  const long long groups_most = ((long long)T + c.R + kGroup - 1) / kGroup;
  // A bulk append of few sequences and many groups (a long prompt) would leave most of the chip idle with two
  // workgroups per (sequence, kv head): from 64 groups on, its groups are shared out in chunks of at least 16, about one
  // owner per compute unit.  The chunks add their shares of S and P to the fp32 state with atomic additions -- S and P
  // are then reproducible up to the rounding order only -- so this needs a cache that keeps the fp32 state (or has no
  // correction at all).
  int n_chunks = 1;
  if (pairs * kParts < 128 && (c.S != nullptr || c.S16 == nullptr)) {
    long long want = 256 / (pairs * kParts);
    if (want > groups_most / 16) want = groups_most / 16;
    if (want > 64) want = 64;
    if (groups_most >= 64 && want > 1) n_chunks = (int)want;
  }
  void (*quantize)(kvlinc_cache, const half_t*, const half_t*, const int32_t*, int, int, int, int) =
      c.bits == 4 ? (sliding ? append_quantize_kernel<true, 4> : append_quantize_kernel<false, 4>)
                  : (sliding ? append_quantize_kernel<true, 2> : append_quantize_kernel<false, 2>);
  void (*states)(kvlinc_cache, const half_t*, const half_t*, const int32_t*, int, int, int) =
      c.bits == 4 ? (sliding ? append_states_kernel<true, 4> : append_states_kernel<false, 4>)
                  : (sliding ? append_states_kernel<true, 2> : append_states_kernel<false, 2>);
  if (launch_with_lds(states, sizeof(StatesLds)) != KVLINC_OK) return KVLINC_EHIP;
  int per_pair = (int)groups_most + 1;  // groups of a pair at most, and the rows that stay in the window
  // A launch has to stay below 2^32 threads (8.4 million pairs, if none takes more than one group).  The states may only be
  // launched behind records that are there: a failed launch ends the call.
  constexpr int kQuantThreads = 64 * kQuantWaves;
  const int pairs_most = (int)(((1ll << 32) - 1) / kQuantThreads / per_pair);
  kvlinc_cache cache = c;
  for (long long first = 0; first < pairs; first += pairs_most) {
    int first_pair = (int)first;
    const long long n_pairs = pairs - first < pairs_most ? pairs - first : pairs_most;
    void* args[] = {&cache, &kk, &vv, &n_new, &T, &keep, &per_pair, &first_pair};
    if (hipLaunchKernel(reinterpret_cast<const void*>(quantize), dim3((unsigned)(n_pairs * per_pair)), dim3(kQuantThreads), args, 0, stream) != hipSuccess)
      return KVLINC_EHIP;
  }
  const long long n_items = (long long)kParts * n_chunks * 8 * ((pairs + 7) / 8);
  const int grid = (int)(n_items < 256 ? n_items : 256);
  hipLaunchKernelGGL(states, dim3(grid), dim3(kThreads), sizeof(StatesLds), stream, c, kk, vv, n_new, T, keep, n_chunks);
  return hipGetLastError() == hipSuccess ? KVLINC_OK : KVLINC_EHIP;
}

}  // namespace kvlinc
