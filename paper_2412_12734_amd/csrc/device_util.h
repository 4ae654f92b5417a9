// Device helpers for gfx950: float-pair ("double-float") arithmetic, wave64 reductions via
// DPP, ballot helpers and bfloat16 decoding.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace gbb {

// ---- unevaluated float pairs (hi + lo), error-free transformations ---------------------
// Knuth's TwoSum and the FMA-based TwoProduct; contraction is switched off so that the
// compiler cannot fuse the error terms away.
struct f2 {
  float hi, lo;
};

__device__ __forceinline__ f2 two_sum(float a, float b) {
#pragma clang fp contract(off)
  float s = a + b;
  float bb = s - a;
  float e = (a - (s - bb)) + (b - bb);
  return {s, e};
}

__device__ __forceinline__ f2 fast_two_sum(float a, float b) {
#pragma clang fp contract(off)
  float s = a + b;
  float e = b - (s - a);
  return {s, e};
}

__device__ __forceinline__ f2 two_prod(float a, float b) {
#pragma clang fp contract(off)
  float p = a * b;
  float e = __builtin_fmaf(a, b, -p);
  return {p, e};
}

__device__ __forceinline__ f2 f2_add(f2 a, f2 b) {
#pragma clang fp contract(off)
  f2 s = two_sum(a.hi, b.hi);
  float lo = s.lo + (a.lo + b.lo);
  return fast_two_sum(s.hi, lo);
}

__device__ __forceinline__ f2 f2_add(f2 a, float b) {
#pragma clang fp contract(off)
  f2 s = two_sum(a.hi, b);
  float lo = s.lo + a.lo;
  return fast_two_sum(s.hi, lo);
}

__device__ __forceinline__ f2 f2_mul(f2 a, float b) {
#pragma clang fp contract(off)
  f2 p = two_prod(a.hi, b);
  float lo = __builtin_fmaf(a.lo, b, p.lo);
  return fast_two_sum(p.hi, lo);
}

__device__ __forceinline__ f2 f2_neg(f2 a) { return {-a.hi, -a.lo}; }

__device__ __forceinline__ f2 f2_sub(f2 a, f2 b) { return f2_add(a, f2_neg(b)); }

__device__ __forceinline__ f2 f2_mul(f2 a, f2 b) {
#pragma clang fp contract(off)
  f2 p = two_prod(a.hi, b.hi);
  float lo = __builtin_fmaf(a.hi, b.lo, __builtin_fmaf(a.lo, b.hi, p.lo));
  return fast_two_sum(p.hi, lo);
}

__device__ __forceinline__ f2 f2_of(float a) { return {a, 0.0f}; }

__device__ __forceinline__ float f2_round(f2 a) { return a.hi + a.lo; }

__device__ __forceinline__ f2 f2_div(f2 a, f2 b) {
#pragma clang fp contract(off)
  float q1 = a.hi / b.hi;
  // r = a - q1 * b, exactly enough: q1*b.hi as a pair, then the small terms
  f2 p = two_prod(q1, b.hi);
  float r = ((a.hi - p.hi) - p.lo) + (a.lo - q1 * b.lo);
  float q2 = r / b.hi;
  return fast_two_sum(q1, q2);
}

// ---- wave64 helpers ------------------------------------------------------------------
// The lanes (of the active ones) where p holds. The compiler builtin takes the condition as
// a lane mask in scalar registers; HIP's __ballot(int) widened it to an integer first and
// compared that again (two vector instructions per vote in the blend loops).
__device__ __forceinline__ uint64_t ballot(bool p) { return __builtin_amdgcn_ballot_w64(p); }

__device__ __forceinline__ uint32_t popc64(uint64_t m) { return (uint32_t)__popcll(m); }

// Number of set bits of m below this lane.
__device__ __forceinline__ uint32_t mbcnt(uint64_t m) {
  return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32),
                                   __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

template <int CTRL, int ROW_MASK = 0xf, int BANK_MASK = 0xf, bool BOUND_CTRL = true>
__device__ __forceinline__ float dpp_f(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, ROW_MASK,
                                                    BANK_MASK, BOUND_CTRL));
}

// Sum over the 64 lanes of a wave; every lane must be active. The total lands in lane 63.
__device__ __forceinline__ float wave_sum_to_lane63(float v) {
  v += dpp_f<0xB1>(v);             // quad_perm [1,0,3,2]
  v += dpp_f<0x4E>(v);             // quad_perm [2,3,0,1]
  v += dpp_f<0x124>(v);            // row_ror:4
  v += dpp_f<0x128>(v);            // row_ror:8   -> every lane holds its row's sum
  v += dpp_f<0x142, 0xa, 0xf, false>(v);  // row_bcast:15 into rows 1 and 3
  v += dpp_f<0x143, 0xc, 0xf, false>(v);  // row_bcast:31 into rows 2 and 3
  return v;
}

// Sums of K values over the 64 lanes, every lane receiving the totals. The K reductions are
// interleaved step by step so that independent DPP operations fill the VALU-to-DPP wait
// states. Within each row of 16 lanes: xor 1 and xor 2 (quad permutes), rotate by 4 and by 8;
// across rows: swap with the neighbouring row (permlane16) and with the other half of the
// wave (permlane32), each followed by an add.
template <int K>
__device__ __forceinline__ void wave_sum_all(float (&v)[K]) {
#pragma unroll
  for (int k = 0; k < K; ++k) v[k] += dpp_f<0xB1>(v[k]);
#pragma unroll
  for (int k = 0; k < K; ++k) v[k] += dpp_f<0x4E>(v[k]);
#pragma unroll
  for (int k = 0; k < K; ++k) v[k] += dpp_f<0x124>(v[k]);
#pragma unroll
  for (int k = 0; k < K; ++k) v[k] += dpp_f<0x128>(v[k]);
#pragma unroll
  for (int k = 0; k < K; ++k) {
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v[k]), __float_as_uint(v[k]),
                                                    false, false);
    v[k] = __uint_as_float(r[0]) + __uint_as_float(r[1]);
  }
#pragma unroll
  for (int k = 0; k < K; ++k) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v[k]), __float_as_uint(v[k]),
                                                    false, false);
    v[k] = __uint_as_float(r[0]) + __uint_as_float(r[1]);
  }
}

// Sums of K values over each row of 16 lanes (every lane receives its row's totals),
// interleaved like wave_sum_all.
template <int K>
__device__ __forceinline__ void row_sum_all(float (&v)[K]) {
#pragma unroll
  for (int k = 0; k < K; ++k) v[k] += dpp_f<0xB1>(v[k]);
#pragma unroll
  for (int k = 0; k < K; ++k) v[k] += dpp_f<0x4E>(v[k]);
#pragma unroll
  for (int k = 0; k < K; ++k) v[k] += dpp_f<0x124>(v[k]);
#pragma unroll
  for (int k = 0; k < K; ++k) v[k] += dpp_f<0x128>(v[k]);
}

// One swap step across lane groups: v_permlane32_swap pairs each lane of the wave's lower half
// with one of the upper half, v_permlane16_swap each lane of an even row with one of the next
// row. Swapping a value pair (a, b) and adding the two results leaves one side of every lane
// pair with a summed over the pair and the other side with b summed: a transposing step at one
// swap and one add per pair. A value without a pair is summed on both sides.
template <bool HALVES>
__device__ __forceinline__ float swap_sum(float a, float b) {
  if constexpr (HALVES) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b),
                                                    false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
  } else {
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b),
                                                    false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
  }
}

template <bool HALVES, int KI>
__device__ __forceinline__ void swap_step(const float (&in)[KI], float (&out)[(KI + 1) / 2]) {
#pragma unroll
  for (int i = 0; i < KI / 2; ++i) out[i] = swap_sum<HALVES>(in[2 * i], in[2 * i + 1]);
  if (KI & 1) out[KI / 2] = swap_sum<HALVES>(in[KI - 1], in[KI - 1]);
}

// The side of each swap step a lane is on: true where it receives the second value of a pair.
// Taken from the swap itself once per kernel, so that the slot mapping holds whichever way
// the hardware orders the exchange.
struct SwapSides {
  bool halves, rows;
};

__device__ __forceinline__ SwapSides swap_sides() {
  return {swap_sum<true>(0.f, 1.f) != 0.f, swap_sum<false>(0.f, 1.f) != 0.f};
}

// ---- row sums by masked DPP adds ---------------------------------------------------------------
// Sums of K = 12, 6 or 3 values over each row of 16 lanes (all lanes active). A pair (a, b) is
// halved by two DPP adds: a + mirrored a into every lane, then b + mirrored b into the half of
// the lanes that the bank mask names (banks are four lanes of a row), so that one lane of each
// mirrored pair goes on with a and the other with b. That is two instructions a pair, against
// three for selects and an add, and three issue slots for a lane swap (which takes two) and an
// add; the bank masks reach lane bits 3 and 2, the last two steps (inside groups of four lanes)
// select. A value without a partner is left as partial sums in both halves where its row_slot
// entry has an owner in each. The four rows are not summed with each other: each owner lane adds
// its row's total to the LDS, where the four adds to one address cost less than two more
// swaps. Written as assembly because the compiler does not form masked DPP adds; the s_nop are
// the wait states a DPP read needs after a write of its source. Outputs are written before all inputs
// are read ("+&": no input, not even an equal one, may have an output's register).
#define GBB_PAIR(A, B, OP, MASK)                                    \
  "v_add_f32_dpp " A ", " A ", " A " " OP " row_mask:0xf bank_mask:0xf\n\t" \
  "v_add_f32_dpp " A ", " B ", " B " " OP " row_mask:0xf bank_mask:" MASK "\n\t"

template <int K>
__device__ __forceinline__ float row_sums(float (&v)[K]) {
  static_assert(K == 12 || K == 6 || K == 3, "built for 12, 6 and 3 values");
  const bool b1 = (threadIdx.x & 2) != 0, b0 = (threadIdx.x & 1) != 0;
  if constexpr (K == 12) {
    __asm__ volatile("s_nop 1\n\t"
                     GBB_PAIR("%0", "%6", "row_mirror", "0xc")
                     GBB_PAIR("%1", "%7", "row_mirror", "0xc")
                     GBB_PAIR("%2", "%8", "row_mirror", "0xc")
                     GBB_PAIR("%3", "%9", "row_mirror", "0xc")
                     GBB_PAIR("%4", "%10", "row_mirror", "0xc")
                     GBB_PAIR("%5", "%11", "row_mirror", "0xc")
                     GBB_PAIR("%0", "%1", "row_half_mirror", "0xa")
                     GBB_PAIR("%2", "%3", "row_half_mirror", "0xa")
                     GBB_PAIR("%4", "%5", "row_half_mirror", "0xa")
                     "s_nop 1"
                     : "+&v"(v[0]), "+&v"(v[2]), "+&v"(v[4]), "+&v"(v[6]), "+&v"(v[8]), "+&v"(v[10])
                     : "v"(v[1]), "v"(v[3]), "v"(v[5]), "v"(v[7]), "v"(v[9]), "v"(v[11]));
    const float x = (b1 ? v[4] : v[0]) + dpp_f<0x4E>(b1 ? v[0] : v[4]);
    const float y = v[8] + dpp_f<0x4E>(v[8]);
    return (b0 ? y : x) + dpp_f<0xB1>(b0 ? x : y);
  } else if constexpr (K == 6) {
    __asm__ volatile("s_nop 1\n\t"
                     GBB_PAIR("%0", "%3", "row_mirror", "0xc")
                     GBB_PAIR("%1", "%4", "row_mirror", "0xc")
                     GBB_PAIR("%2", "%5", "row_mirror", "0xc")
                     GBB_PAIR("%0", "%1", "row_half_mirror", "0xa")
                     "s_nop 1"
                     : "+&v"(v[0]), "+&v"(v[2]), "+&v"(v[4])
                     : "v"(v[1]), "v"(v[3]), "v"(v[5]));
    const float x = (b1 ? v[4] : v[0]) + dpp_f<0x4E>(b1 ? v[0] : v[4]);
    return x + dpp_f<0xB1>(x);
  } else {
    __asm__ volatile("s_nop 1\n\t"
                     GBB_PAIR("%0", "%1", "row_mirror", "0xc")
                     "s_nop 1\n\t"
                     GBB_PAIR("%0", "%2", "row_half_mirror", "0xa")
                     "s_nop 1"
                     : "+&v"(v[0])
                     : "v"(v[1]), "v"(v[2]));
    const float x = v[0] + dpp_f<0x4E>(v[0]);
    return x + dpp_f<0xB1>(x);
  }
}

// Wave sums of ten values, added in the order lane ^ 32, ^ 16, ^ 15, ^ 7, ^ 3, ^ 1: two swap steps,
// then the row steps above.
__device__ __forceinline__ float record_sums(const float (&v)[10]) {
  float a[5], b[3];
  swap_step<true>(v, a);
  swap_step<false>(a, b);
  __asm__ volatile("s_nop 1\n\t"
                   GBB_PAIR("%0", "%1", "row_mirror", "0xc")
                   "v_add_f32_dpp %2, %2, %2 row_mirror row_mask:0xf bank_mask:0xf\n\t"
                   "s_nop 1\n\t"
                   GBB_PAIR("%0", "%2", "row_half_mirror", "0xa")
                   "s_nop 1\n\t"
                   "v_add_f32_dpp %0, %0, %0 quad_perm:[3,2,1,0] row_mask:0xf bank_mask:0xf\n\t"
                   "s_nop 1\n\t"
                   "v_add_f32_dpp %0, %0, %0 quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf\n\t"
                   "s_nop 1"
                   : "+v"(b[0]), "+v"(b[1]), "+v"(b[2]));
  return b[0];
}
#undef GBB_PAIR

// The value that record_sums leaves in a lane of row position l, -1 where it leaves a copy of
// another lane's. With h and r the sides of the swaps and b3..b0 the bits of l: 4 b3 + 2 r + h for
// b2 = 0, 8 + h for b2 = 1 (held for both r and both b3); b1 and b0 hold copies.
__device__ __forceinline__ int record_slot(SwapSides s, int l) {
  if ((l & 3) != 0) return -1;
  if ((l & 4) != 0) return s.rows || (l & 8) != 0 ? -1 : 8 + (s.halves ? 1 : 0);
  return 4 * (l >> 3) + (s.rows ? 2 : 0) + (s.halves ? 1 : 0);
}

// The value whose (partial) sum row_sums<K> leaves in row position l (0..15), -1 in a position
// that holds a copy of another's. With b3..b0 the bits of l:
//   12: 4 j + 2 b2 + b3 with j = b1 for b0 = 0; j = 2 for b0 = 1, held twice (b1)
//    6: 2 i + b3 with i = b2 for b1 = 0; i = 2 for b1 = 1, in two parts (b2); b0 holds copies
//    3: b3 for b2 = 0; 2 for b2 = 1, in two parts (b3); b1 and b0 hold copies
__host__ __device__ constexpr int row_slot(int K, int l) {
  const int b3 = l >> 3 & 1, b2 = l >> 2 & 1, b1 = l >> 1 & 1, b0 = l & 1;
  if (K == 12) return b0 ? (b1 ? -1 : 8 + 2 * b2 + b3) : 4 * b1 + 2 * b2 + b3;
  if (K == 6) return b0 ? -1 : 2 * (b1 ? 2 : b2) + b3;
  return b1 || b0 ? -1 : (b2 ? 2 : b3);
}

// The lanes of a wave whose row position owns a value, as a lane mask.
__host__ __device__ constexpr uint64_t row_owners(int K) {
  uint64_t m = 0;
  for (int l = 0; l < 64; ++l)
    if (row_slot(K, l & 15) >= 0) m |= 1ull << l;
  return m;
}

__device__ __forceinline__ float bf16_to_f32(uint16_t b) {
  return __uint_as_float(((uint32_t)b) << 16);
}

}  // namespace gbb
