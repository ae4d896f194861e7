// The activation's derivative by table, for the epilogues that evaluate it on whole tiles.
//
// The pre-activation is a bf16 value: between 2^-21 and 8 there are 24 binades of 128 values and two signs, so the derivative of
// GELU (tanh form, common.h) over that range is 6144 float32 values, 24 KiB.  Below it is 1/2 to within 4e-7, above 1 or 0 to within 1e-19, for
// every finite value; of infinities and NaN comes NaN.
// A lookup takes four vector instructions and an LDS read per element where the formula takes nine, an exp2 and a reciprocal.  The values
// are rounded from float64: over all bf16 patterns the largest error is 3.8e-7 (just below 2^-21), the formula's 1.9e-6.  Only beyond the table's
// ends is the formula the closer one, below 2^-21 (6e-8) and below -8 (where the derivative is smaller than 1e-19).  Input gradient with it, 256 x 256 tiles, against the formula (us):
// 32768 x 1280 x 5120 e4m3 309 -> 293 (253 without activation), 16384 x 1024 x 4096 bf16 156 -> 152; single rounds of tiles (3072 x 1280 x 5120)
// 36.8 -> 35.7 and 53.5 -> 52.6.  What is left above the plain product is less than H takes to be read.
// The forward product's epilogue, bound by its two stores, gains nothing from a table of its own (215 against 217, 105 against 104).
#pragma once
#include "common.h"

namespace sste {

constexpr int GELU_BINADES = 24, GELU_ENTRIES = 128 * GELU_BINADES, GELU_FIRST = (127 - 21) << 7;   // values per sign; bf16 pattern of 2^-21
constexpr int GELU_TABLE_BYTES = 2 * GELU_ENTRIES * 4;
struct GeluTable {
  float v[2 * GELU_ENTRIES];             // [2 c + sign], c = pattern of |h| - GELU_FIRST, at least 0 and below GELU_ENTRIES
};

constexpr double exp_host(double x) {    // for x >= 0: 2^-10 of it by the series, squared ten times
  const double y = x / 1024.0;
  double t = 1.0, sum = 0.0;             // exp(y) - 1, which keeps its digits: (1 + s)^2 - 1 = s (2 + s)
  for (int k = 1; k < 10; k++) {
    t *= y / k;
    sum += t;
  }
  for (int k = 0; k < 10; k++) sum = sum * (2.0 + sum);
  return 1.0 + sum;
}
constexpr GeluTable gelu_grad_table() {
  GeluTable g{};
  for (int c = 0; c < GELU_ENTRIES; c++) {
    double x = c ? 1.0 + (c & 127) / 128.0 : 0.0;                      // entry 0 stands for everything below, zero among it
    for (int b = c >> 7; b < 21; b++) x *= 0.5;
    for (int b = 21; b < c >> 7; b++) x *= 2.0;
    const double k = 0.79788456080286535588, x2 = x * x;               // sqrt(2 / pi)
    const double e = 1.0 / exp_host(2.0 * k * x * (1.0 + 0.044715 * x2));   // s(x) = 1 / (1 + e), s(-x) = e / (1 + e)
    const double p = 2.0 * k * x * (1.0 + 3.0 * 0.044715 * x2) * e / ((1.0 + e) * (1.0 + e));
    g.v[2 * c] = (float)(1.0 / (1.0 + e) + p);
    g.v[2 * c + 1] = (float)(e / (1.0 + e) - p);
  }
  return g;
}

// The table into LDS by NW waves: its loads are only issued, the caller waits for them.
template <int NW>
__device__ __forceinline__ void gelu_table_load(uint8_t* tab, const GeluTable& table, int wave, int lane) {
  const i32x4 rsrc = rsrc_words(&table, GELU_TABLE_BYTES);
  constexpr int N = GELU_TABLE_BYTES / 1024;
  static_assert(N % NW == 0, "whole loads per wave");
#pragma unroll
  for (int i = 0; i < N / NW; i++) {
    const int n = N / NW * wave + i;
    dma_b128(rsrc, (uint32_t)(uintptr_t)(lds_u8*)tab + n * 1024, (uint32_t)(n * 1024 + lane * 16), 0u);
  }
}

// The table's values for eight bf16 patterns.
__device__ __forceinline__ void gelu_lookup8(const uint8_t* tab, const uint32_t (&w)[4], float (&d)[8]) {
  typedef __attribute__((__vector_size__(2 * sizeof(uint16_t)))) uint16_t u16x2;
  const u16x2 first = {GELU_FIRST, GELU_FIRST}, last = {GELU_ENTRIES - 1, GELU_ENTRIES - 1};
#pragma unroll
  for (int e = 0; e < 4; e++) {
    const uint32_t mag = w[e] & 0x7FFF7FFFu;
    u16x2 c;
    __builtin_memcpy(&c, &mag, 4);
    c = __builtin_elementwise_min(__builtin_elementwise_sub_sat(c, first), last) << 3;
    uint32_t at;
    __builtin_memcpy(&at, &c, 4);
    at |= (w[e] >> 13) & 0x00040004u;
    d[2 * e] = *(const float*)(tab + (at & 0xFFFFu));
    d[2 * e + 1] = *(const float*)(tab + (at >> 16));
  }
}
// Whether an infinity or a NaN is among the eight, and NaN in the place of those, as the formula gives it; the others keep their values.
__device__ __forceinline__ bool gelu_not_in_table(const uint32_t (&w)[4]) {
  typedef __attribute__((__vector_size__(2 * sizeof(uint16_t)))) uint16_t u16x2;
  u16x2 m = {0, 0};
#pragma unroll
  for (int e = 0; e < 4; e++) {
    const uint32_t mag = w[e] & 0x7FFF7FFFu;
    u16x2 c;
    __builtin_memcpy(&c, &mag, 4);
    m = __builtin_elementwise_max(m, c);
  }
  uint32_t b;
  __builtin_memcpy(&b, &m, 4);
  return ((b + 0x00800080u) & 0x80008000u) != 0;
}
__device__ __forceinline__ void gelu_mark_nan8(const uint32_t (&w)[4], float (&d)[8]) {
#pragma unroll
  for (int e = 0; e < 4; e++) {
    if ((w[e] & 0x7F80u) == 0x7F80u) d[2 * e] = __builtin_nanf("");
    if ((w[e] & 0x7F800000u) == 0x7F800000u) d[2 * e + 1] = __builtin_nanf("");
  }
}

}  // namespace sste
