// Device code of the 2:4 minimum-variance unbiased estimator (paper Sec. 5.1) and its counter-based
// random draw.  The rule is stated in full in include/sste.h (sste_mvue_materialize).  Every float
// operation below is a single IEEE float32 operation in the order written; the translation unit is
// compiled with -ffp-contract=off so that tau1 = tau0 + h is not fused with tau0 = u * h.
#pragma once
#include "common.h"

namespace sste {

// 32-bit draw for a group id: three-round multiply-xorshift hash keyed by (k0, k1).  draw_u32_mixed takes it from
// x = (low word ^ k0) + high word * 0x9E3779B9, which callers that walk consecutive ids form themselves; draw_u32_folded from x ^ (x >> 17).
__device__ __forceinline__ uint32_t draw_u32_folded(uint32_t x, uint32_t k1) {
  x *= 0xED5AD4BBu;
  x += k1;
  x ^= x >> 11;
  x *= 0xAC4C1B51u;
  x ^= x >> 15;
  x *= 0x31848BABu;
  x ^= x >> 14;
  return x;
}
__device__ __forceinline__ uint32_t draw_u32_mixed(uint32_t x, uint32_t k1) { return draw_u32_folded(x ^ (x >> 17), k1); }
__device__ __forceinline__ uint32_t draw_u32(uint32_t k0, uint32_t k1, uint32_t gid_lo, uint32_t gid_hi) {
  return draw_u32_mixed((gid_lo ^ k0) + gid_hi * 0x9E3779B9u, k1);
}

// What the rule below costs decides how fast the estimator's kernels run, so the forms are chosen by the measured issue time of the
// vector instructions (clocks per wave on a full SIMD): 32-bit add, subtract, and, or, xor, right shift, float add and multiply,
// bitop3 about 3; minima, maxima, compares, left shifts, byte permutes, three-operand integer forms and 32-bit multiplies about 5;
// a select right behind its compare 2.4; a conversion of two 8-bit codes 4.6 (as much as one of a single code), back 8.7.
struct Sel {
  float h;        // common magnitude of recorded elements that are not kept as they are
  // recorded positions pos0 = 2 - n0 < pos1 = 3 - n1; sign bits: n0 >= 1, n0 >= 2, n1 >= 1, n1 >= 2
  uint32_t n0_1, n0_2, n1_1, n1_2;
};

// Steps 1-4 of the rule on the four magnitudes m0..m3 (all >= 0, finite) and the 32-bit draw x.
// Non-negative floats order like their bit patterns, so minima, maxima and comparisons are taken on
// the bits as unsigned integers (same results, and no NaN canonicalisation instructions); sums and
// products are float32 operations.
// A NaN pattern is the greatest magnitude and so stays out of the sum of the three smaller ones: where one of these is not zero, the NaN is recorded.
// EXACT: the magnitudes are e4m3's, whole multiples of 2^-9 up to 448, so that no sum of them rounds and the three may be added in any order:
// the least and the median of three, and the lesser of their greatest and the fourth.  One dear instruction less (e4m3 32768 x 5120 64.6 -> 62.0 us);
// the instructions are named because the compiler makes two of each from the shared parts.  The sum of all less the largest takes as long, but is
// NaN with the largest, and such NaNs were lost ahead of one non-zero element and two zeros.
__device__ __forceinline__ uint32_t min3_u32(uint32_t a, uint32_t b, uint32_t c) {
  uint32_t r;
  asm("v_min3_u32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
  return r;
}
__device__ __forceinline__ uint32_t max3_u32(uint32_t a, uint32_t b, uint32_t c) {
  uint32_t r;
  asm("v_max3_u32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
  return r;
}
template <bool EXACT>
__device__ __forceinline__ Sel mvue_select(float m0f, float m1f, float m2f, float m3f, uint32_t x) {
  uint32_t m0 = f2u(m0f), m1 = f2u(m1f), m2 = f2u(m2f), m3 = f2u(m3f);
  uint32_t a = max(m0, m1), b = min(m0, m1);
  float Lo;
  if (EXACT) {
    const uint32_t median = max(min(a, m2), b);
    Lo = (u2f(min3_u32(m0, m1, m2)) + u2f(median)) + u2f(min(max3_u32(m0, m1, m2), m3));
  } else {
    uint32_t cc = max(m2, m3), d = min(m2, m3);
    uint32_t mid = min(a, cc);
    Lo = (u2f(b) + u2f(d)) + u2f(mid);
  }
  // Lo is a sum of non-negative terms: +0 or positive.  Where it is 0 the rule clamps to the largest magnitude, which clamps nothing.
  uint32_t clampv = (f2u(Lo) == 0u) ? 0xFFFFFFFFu : f2u(Lo);
  float l0 = u2f(min(m0, clampv)), l1 = u2f(min(m1, clampv)), l2 = u2f(min(m2, clampv)), l3 = u2f(min(m3, clampv));
  float P0 = l0;
  float P1 = P0 + l1;
  float P2 = P1 + l2;
  float L = P2 + l3;
  float h = 0.5f * L;
  float u = (float)(x & 0xFFFFFF00u) * 0x1p-32f;     // (x >> 8) 2^-24: exact, a 24-bit integer times a power of two
  float tau0 = u * h;
  float tau1 = tau0 + h;
  uint32_t p0 = f2u(P0), p1 = f2u(P1), p2 = f2u(P2), t0 = f2u(tau0), t1 = f2u(tau1);
  // pos0 = min(#{k : P_k <= tau0}, 2): the prefix sums never decrease, so P2 <= tau0 implies the other
  // two and the count capped at 2 is the count over P0 and P1 alone.  pos1 = min(3, max(i1, pos0 + 1))
  // with i1 = #{k <= 2 : P_k <= tau1} <= 3 and pos0 <= 2: the outer min never acts.  Counted are the prefix
  // sums ABOVE the thresholds, as sign bits of differences of patterns below 2^31:
  // pos0 = 2 - n0, i1 = 3 - #{k : P_k > tau1}, pos1 = 3 - n1, n1 = min(#{k : P_k > tau1}, n0).  As the sums never decrease, a count is
  // at least 1 where the last of its sums is above and at least 2 where the one before is; P0 > tau1 would be a third, which n0 <= 2 cuts off.
  Sel s;
  s.h = h;
  s.n0_1 = t0 - p1;
  s.n0_2 = t0 - p0;
  s.n1_1 = (t1 - p2) & s.n0_1;
  s.n1_2 = (t1 - p1) & s.n0_2;
  return s;
}

// bf16 group {hi:lo} = (g0 | g1 << 16, g2 | g3 << 16).  Returns the two recorded bf16 values packed
// (pos0's value in the low half); nn = n0 + 4 n1, the metadata nibble pos0 | pos1 << 2 being 14 - nn.
__device__ __forceinline__ uint32_t mvue_group_bf16(uint32_t lo, uint32_t hi, uint32_t x, uint32_t& nn) {
  float m0 = u2f((lo << 16) & 0x7FFFFFFFu), m1 = u2f(lo & 0x7FFF0000u);
  float m2 = u2f((hi << 16) & 0x7FFFFFFFu), m3 = u2f(hi & 0x7FFF0000u);
  const Sel s = mvue_select<false>(m0, m1, m2, m3, x);
  const uint32_t n0 = (s.n0_1 >> 31) + (s.n0_2 >> 31), n1 = (s.n1_1 >> 31) + (s.n1_2 >> 31);
  // Both recorded elements at once, as a pair of 16-bit patterns (pos0's in the low half): one byte
  // permute of {hi:lo} with selector bytes (2 pos0, 2 pos0 + 1, 2 pos1, 2 pos1 + 1).
  typedef __attribute__((__vector_size__(2 * sizeof(uint16_t)))) uint16_t u16x2;
  const uint32_t sel = 0x07060504u - 0x0202u * (n0 + (n1 << 16));
  const uint32_t g = __builtin_amdgcn_perm(hi, lo, sel);
  // An element keeps its own pattern when m_p > h or m_p == 0.  On the 15-bit magnitude fields (the low
  // 16 bits of a bf16's float32 pattern are zero): field > bits(h) >> 16, or field == 0; both at once as
  // (field - 1) mod 2^16 >= bits(h) >> 16, evaluated for the pair with packed 16-bit arithmetic:
  // the saturating difference hh - (field - 1) is zero exactly for the elements that keep their pattern.
  const uint32_t hh = f2u(s.h) >> 16;
  u16x2 field, one = {1, 1}, hh2 = {(uint16_t)hh, (uint16_t)hh};
  const uint32_t gm = g & 0x7FFF7FFFu;
  __builtin_memcpy(&field, &gm, 4);
  u16x2 d = __builtin_elementwise_sub_sat(hh2, (u16x2)(field - one));
  u16x2 common_mask = (u16x2){0, 0} - __builtin_elementwise_min(d, one);        // 0xFFFF where sign | RNE(h) is stored
  uint32_t cm;
  __builtin_memcpy(&cm, &common_mask, 4);
  const uint32_t hq = bf16_rne(s.h);
  const uint32_t common = (g & 0x80008000u) | (hq | (hq << 16));
  nn = n0 + (n1 << 2);
  return (common & cm) | (g & ~cm);
}

// Two 8-bit groups (e4m3, or e5m2 when BF8), ga and gb: the four codes of a group in one dword (g0 in byte 0).  Returns the recorded
// codes of theta / 2, group ga's in the low half (pos0's in its low byte), and the metadata byte of the pair.  In pairs because the
// byte permute that gathers the recorded codes, the conversion of two of them and the signs serve two groups at once.
template <bool BF8>
__device__ __forceinline__ uint32_t mvue_pair_f8(uint32_t ga, uint32_t gb, uint32_t xa, uint32_t xb, uint32_t& meta) {
  typedef __attribute__((__vector_size__(2 * sizeof(float)))) float f32x2;
  typedef __attribute__((__vector_size__(2 * sizeof(short)))) short i16x2;
#define MVUE_CVT2(w, hi) (BF8 ? __builtin_amdgcn_cvt_pk_f32_bf8((int)(w), hi) : __builtin_amdgcn_cvt_pk_f32_fp8((int)(w), hi))
  const uint32_t maga = ga & 0x7F7F7F7Fu, magb = gb & 0x7F7F7F7Fu;
  const f32x2 a01 = MVUE_CVT2(maga, false), a23 = MVUE_CVT2(maga, true), b01 = MVUE_CVT2(magb, false), b23 = MVUE_CVT2(magb, true);
  const Sel sa = mvue_select<!BF8>(a01[0], a01[1], a23[0], a23[1], xa), sb = mvue_select<!BF8>(b01[0], b01[1], b23[0], b23[1], xb);
  // recorded codes: bytes 2 - n0, 3 - n1 of ga (bytes 0 .. 3 of the permute's source) and of gb (bytes 4 .. 7).  The four counts of the
  // pair, n0 and n1 of ga in the low half, by byte permutes that spread sign bits (selector 9: the low operand's, 11: the high one's)
  const uint32_t one = __builtin_amdgcn_perm(sa.n1_1, sa.n0_1, 0x0C0C0B09u) | __builtin_amdgcn_perm(sb.n1_1, sb.n0_1, 0x0B090C0Cu);
  const uint32_t two = __builtin_amdgcn_perm(sa.n1_2, sa.n0_2, 0x0C0C0B09u) | __builtin_amdgcn_perm(sb.n1_2, sb.n0_2, 0x0B090C0Cu);
  const uint32_t n = (one & 0x01010101u) + (two & 0x01010101u);
  const uint32_t rec = __builtin_amdgcn_perm(gb, ga, 0x07060302u - n);
  meta = 0xEEu - __builtin_amdgcn_udot4(n, 0x40100401u, 0u, false);       // nibbles 14 - n0 - 4 n1
  const uint32_t mag = rec & 0x7F7F7F7Fu;
  const f32x2 ra = MVUE_CVT2(mag, false), rb = MVUE_CVT2(mag, true);
#undef MVUE_CVT2
  // stored magnitude: half of m_p where m_p > h or m_p = 0 (then 0), else half of h: the median of m_p, h and 2^40 m_p (in either
  // format 2^40 times the least positive magnitude is above every h); halved by the conversion, within the format's range
  auto stored = [](float m, float h) {
    const uint32_t x = f2u(m), y = f2u(h), z = f2u(m * 0x1p40f);
    return u2f(max(min(max(x, y), z), min(x, y)));
  };
  i16x2 q;
  asm volatile("" : "=v"(q));                         // both halves are written: nothing to clear first
  if (BF8) {
    q = __builtin_amdgcn_cvt_scalef32_pk_bf8_f32(q, stored(ra[0], sa.h), stored(ra[1], sa.h), 2.0f, false);
    q = __builtin_amdgcn_cvt_scalef32_pk_bf8_f32(q, stored(rb[0], sb.h), stored(rb[1], sb.h), 2.0f, true);
  } else {
    q = __builtin_amdgcn_cvt_scalef32_pk_fp8_f32(q, stored(ra[0], sa.h), stored(ra[1], sa.h), 2.0f, false);
    q = __builtin_amdgcn_cvt_scalef32_pk_fp8_f32(q, stored(rb[0], sb.h), stored(rb[1], sb.h), 2.0f, true);
  }
  uint32_t codes;
  __builtin_memcpy(&codes, &q, 4);
  return codes | (rec & 0x80808080u);
}

}  // namespace sste
