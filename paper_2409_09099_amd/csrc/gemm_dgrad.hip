// Input gradient of the S-STE linear layer (paper Sec. 5.1): grad_X = grad_Z S(W).  The paper keeps this
// product dense (only grad_Z is sparsified, and only for the weight gradient), so it runs on the dense
// matrix instruction; what it shares with the forward pass is the packed weight, which is decoded to
// dense-with-zeros on its way into the matrix operand instead of being kept a second time in memory.
//
// MFMA mapping: grad_X^T = S(W)^T grad_Z^T.  Rows = input features i, columns = tokens t, contraction
// k = output channels o.  Any assignment of channels to the bytes of a lane's fragment is right as long as both
// operands use the same one.  The grad_Z tile lies in LDS as token rows of 128 bytes of channels (64 bf16 / 128
// 8-bit), 16-byte piece c of row r at position c ^ ((r / 2) % 8), so that 16 rows x one piece hit 16 different bank
// groups; it arrives by direct-to-LDS loads.
//
// The packed operand runs along features, the contraction along channels: decoding it means transposing it.  The sparse matrix
// instruction does both: S_block x identity (v_smfmac_f32_32x32x32_bf16 / 32x32x64_fp8_fp8 with the packed slots as operand A, exactly as
// they lie in memory) leaves in lane (n, hh) sixteen channels of feature n as float32, exactly (one term per sum).  With the packed
// rows assigned to the instruction's rows in the order rho(m) = 16 (m / 4 % 2) + 4 (m / 8) + m % 4 the sixteen channels are
// consecutive: converted back they ARE the operand fragments of the product (of 32 x 32 instructions; for 16 x 16 ones after a swap of
// 16-lane rows), and S(W) never passes through the LDS in dense form.  Each wave owns 32 features and ALL tokens of its workgroup's tile,
// so no block is decoded twice in a workgroup: one expansion per 16 (bf16) or 8 (8-bit) equal shares of matrix time in the 256-token
// tiles.  The price is that every wave reads the whole grad_Z tile from LDS (256 KiB per k-step of 256 x 256, 43 % of
// its clocks at the measured 128 KiB in 567).
//
// What bounds it.  The large tiles run at the clock that the power limit leaves, 1.6 ... 1.8 GHz: a k-step of 256 x 256 takes 2650 (bf16) /
// 2670 (8-bit) clocks, of which the matrix pipe needs 2176 / 2304.  Before (decode by two waves each, or by byte
// permutes through the LDS) it took 2990 / 3740 clocks at 1.75 / 1.99 GHz; so of 11 / 29 % fewer clocks 10 / 14 % of time are left, and what
// counts is work per result: the 16 x 16 instructions of bf16 sustain 1.87 ... 2.04 PFLOP/s on random operands in registers against 1.76 of the
// 32 x 32 ones (hence the former in the large bf16 tiles, with the two operands exchanged in turn: 4 % faster; 8-bit tiles lose 4 % to
// the narrower fragments' extra instructions, small ones 6 %, being bound by latencies).  Two waves of 64 features x 128 tokens (half
// the LDS reads, twice the decoding) are equal in bf16 and 15 % slower in 8 bits; four waves of 64 features each would need
// accumulators beyond the vector registers (1.4 x slower, moves between the two files).
// Small tiles: with KG > 1 the workgroup's waves form KG groups that take the k-steps in turn, each with its own LDS slots, and add
// their sums at the end: a problem with few tiles is bound by the time a k-step's loads take to arrive, not by any rate, and KG times the
// k-steps in flight divide that.
// Measured (us before -> after, T x O x I): bf16 2112 x 1544 x 832 16.7 -> 12.9, 4096 x 3072 x 768 31.0 -> 23.5, 8192 x 3072 x 768 56 -> 50,
// 16384 x 4096 x 1024 123 -> 111, 16384 x 5120 x 1280 205 -> 183, 16384 x 1280 x 5120 201 -> 179; e5m2 3200 x 1552 x 896 15.8 -> 12.2,
// 32768 x 1280 x 5120 249 -> 223, 32768 x 5120 x 1280 214 -> 191; e4m3 2048 x 4096 x 1024 20.3 -> 17.9.  One and two k-steps, which
// a wave decodes and multiplies in a longer serial chain: within 3 % of before.
// The identity product is exact for finite values; an infinite or NaN packed value (the interface rules them out) makes NaN of the 32
// features it is expanded with.  Asking every packed slot for one, with a second look in a branch, was measured: 2.1 % of a four-layer
// training step in bf16 (1668 -> 1704 us), 1.8 % of an 8-bit layer of small tiles, so it is not asked.
// Which tile runs is decided by a time model fitted to a sweep (dgrad_choice).
// Epilogue as in the forward GEMM: transposed through LDS, 16-byte streaming stores of bf16 rows.
#include "common.h"
#include "gelu_table.h"
#include "tile_order.h"

#include <stdio.h>

#include <type_traits>
#include <utility>

namespace sste {

__device__ constexpr GeluTable kGeluGrad = gelu_grad_table();

namespace {
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;
// f(0), f(1), ... f(N - 1) with the numbers as constants: a loop that is unrolled whatever its size
template <class F, int... K>
__device__ __forceinline__ void static_for_seq(F&& f, std::integer_sequence<int, K...>) {
  (f(std::integral_constant<int, K>{}), ...);
}
template <int N, class F>
__device__ __forceinline__ void static_for(F&& f) {
  static_for_seq(f, std::make_integer_sequence<int, N>{});
}
struct DgradArgs {
  const uint8_t* dY;
  int64_t T, O, lddy_bytes;
  const uint8_t* vals;
  const uint8_t* meta;
  int64_t I;
  int isteps;              // packed column steps (64 bf16 / 128 e4m3 features)
  float scale;
  uint16_t* dX;
  int64_t lddx;
  const uint16_t* H;       // stored pre-activation, or null
  int64_t ldh;
};
}  // namespace

// grad_Z loads.  A row's bytes past its last channel belong to somebody else (the next token's row, padding of any content): S(W) has
// zeros there, but zero times a NaN pattern is NaN, so the 16-byte pieces past the last channel are pushed out of range and arrive as zeros.
// `live` bytes of a row are left at this k-step (O x element size - 128 x step), `piece` = 16 x the piece's number inside the k-step.
constexpr uint32_t NO_PIECE = 0x80000000u;
__device__ __forceinline__ uint32_t dy_offset(uint32_t off, int piece, int live) { return piece < live ? off : NO_PIECE; }
// the piece a lane fetches in load number wl of a tile (8 rows x 128 bytes per load, row r's piece c at position c ^ ((r / 2) % 8)), times 16
__device__ __forceinline__ int dy_piece(int lane, int wl) { return 16 * ((lane & 7) ^ ((4 * (wl & 1) + (lane >> 4)) & 7)); }

// Two of the sixteen accumulator registers of an expansion set to zero (the compiler otherwise builds a zero vector and copies it).  Only
// where no matrix instruction that writes them is in flight, and two wait states ahead of one that reads them, which settle() holds: the
// compiler does not know the assembly for a vector instruction and counts none itself.
__device__ __forceinline__ void zero_pair(f32x16& v, int r) {
  typedef __attribute__((__vector_size__(2 * sizeof(float)))) float f32x2;
  f32x2 z;
  asm volatile("v_mov_b64 %0, 0" : "=v"(z));
  v[2 * r] = z[0];
  v[2 * r + 1] = z[1];
}
// The wait states between the zeroing of v and the matrix instruction that adds to it.  v is an operand: without one the compiler may
// issue the matrix instruction ahead of the wait.
__device__ __forceinline__ void settle(f32x16& v) { asm volatile("s_nop 1" : "+v"(v)); }

// Which tiles take the activation's derivative from the table (gelu_table.h): those whose lookups are worth the table's 24 KiB.
template <int WF, int NT>
constexpr bool dgrad_table() { return WF * NT >= 16; }

// Backward of the activation that produced this layer's input: grad_H = grad_A * GELU'(H), on 16 bytes of the bf16 gradient just formed and
// of the stored pre-activation.
template <bool TABLE>
__device__ __forceinline__ uint4 dgrad_act_piece(const uint8_t* tab, const uint4& v, const uint4& hv) {
  const uint32_t g[4] = {v.x, v.y, v.z, v.w}, hw[4] = {hv.x, hv.y, hv.z, hv.w};
  float d[8];
  if (TABLE) {
    gelu_lookup8(tab, hw, d);
    if (gelu_not_in_table(hw)) gelu_mark_nan8(hw, d);
  } else {
#pragma unroll
    for (int e = 0; e < 4; e++) {
      d[2 * e] = gelu_tanh_grad(bf16lo_f32(hw[e]));
      d[2 * e + 1] = gelu_tanh_grad(bf16hi_f32(hw[e]));
    }
  }
  uint32_t r[4];
#pragma unroll
  for (int e = 0; e < 4; e++) r[e] = bf16_rne_pack(bf16lo_f32(g[e]) * d[2 * e], bf16hi_f32(g[e]) * d[2 * e + 1]);
  return make_uint4(r[0], r[1], r[2], r[3]);
}

// Accumulators of a wave's 32 features x 32 NT tokens: 16 x 16 or 32 x 32 blocks of the matrix instruction.  Register 4 g + r of lane l
// holds feature 8 g + 4 (l / TB) + r (16 x 16: one g) of token l % TB.
template <bool M16, int NT>
struct DgradAcc {
  static constexpr int TB = M16 ? 16 : 32, MB = 32 / TB, NB = 32 * NT / TB, G = M16 ? 1 : 4;
  typedef std::conditional_t<M16, f32x4, f32x16> block;
  block v[MB][NB];
};

// Output stage: accumulators -> LDS (row = token, the tile's 32 WF features contiguous) -> 16-byte stores of whole rows.  Chunk c of
// token row t sits at c ^ key(t), and with 32 x 32 blocks rows with bit 4 set have the 8-byte halves of their chunks swapped: every write
// and read then covers all banks.
template <bool M16, int WF, int NT, int KG>
__device__ __forceinline__ void dgrad_store(uint8_t* smem, const DgradArgs& a, const DgradAcc<M16, NT>& acc, int kg, int wave, int lane,
                                            int64_t i0, int64_t t0) {
  constexpr int CH = 4 * WF, ROWS = 32 * NT / (WF * KG), NIT = ROWS * CH / 64;   // 16-byte chunks per token row; rows of a wave, chunks of a lane
  static_assert(ROWS * WF * KG == 32 * NT && NIT * 64 == ROWS * CH, "whole rows per wave");
  typedef DgradAcc<M16, NT> A;
  const int n = lane % A::TB, hq = lane / A::TB;
  const float scale = a.scale;
  auto key = [](int row) { return CH >= 16 ? (row & 15) : (row / (16 / (CH < 16 ? CH : 16))) % CH; };
  auto flip = [](int row) { return M16 ? 0 : (row >> 4) & 1; };
  // Activation: the table's loads and the first of H's go ahead of the staging writes.  H is requested AHEAD chunks in advance: asked for one by
  // one, each between its bounds check and its use, the loads cost a memory latency each (32768 x 1280 x 5120 e5m2: 380 -> 338 us,
  // 277 without the activation; 16384 x 1024 x 4096 bf16: 181 -> 164; 8192 x 768 x 3072 e4m3: 49 -> 44).
  constexpr bool TABLE = dgrad_table<WF, NT>();
  constexpr int AHEAD = NIT < 8 ? NIT : 8;
  uint8_t* const tab = smem + 32 * NT * 64 * WF;
  const int r0 = ROWS * (KG > 1 ? kg * WF + wave : wave);
  // The plain product, the more frequent one, falls through: with this block in its way the small tiles took 1 % longer.
  int live_rows = 0, live_cols = 0;
  uint4 h[AHEAD];
  auto fetch = [&](int it) {                        // a lane outside the matrix reads the tile's first chunk
    const int c = 64 * it + lane, row = c / CH, chunk = c % CH;
    const bool live = row < live_rows && 8 * chunk < live_cols;
    const i32x4 v = __builtin_nontemporal_load((const i32x4*)(a.H + (t0 + (live ? r0 + row : 0)) * a.ldh + i0 + (live ? 8 * chunk : 0)));
    return make_uint4((uint32_t)v[0], (uint32_t)v[1], (uint32_t)v[2], (uint32_t)v[3]);
  };
  if (__builtin_expect(a.H != nullptr, 0)) {
    live_rows = (int)(a.T - t0 < 32 * NT ? a.T - t0 : 32 * NT) - r0;
    live_cols = (int)(a.I - i0 < 8 * CH ? a.I - i0 : 8 * CH);
    if (TABLE) gelu_table_load<WF * KG>(tab, kGeluGrad, KG > 1 ? kg * WF + wave : wave, lane);
#pragma unroll
    for (int it = 0; it < AHEAD; it++) h[it] = fetch(it);
    __builtin_amdgcn_sched_barrier(0);
  }
  if (KG == 1 || kg == 0) {                       // group 0 holds the sums
#pragma unroll
    for (int t = 0; t < A::NB; t++)
#pragma unroll
      for (int m = 0; m < A::MB; m++)
#pragma unroll
        for (int g = 0; g < A::G; g++) {
          uint2 v;
          v.x = bf16_rne_pack(acc.v[m][t][4 * g] * scale, acc.v[m][t][4 * g + 1] * scale);
          v.y = bf16_rne_pack(acc.v[m][t][4 * g + 2] * scale, acc.v[m][t][4 * g + 3] * scale);
          const int row = A::TB * t + n, half = (8 * g + 4 * hq) / 4;         // 8-byte half chunk inside the block
          const int chunk = (32 * wave + A::TB * m) / 8 + (half >> 1);
          *(uint2*)(smem + row * (16 * CH) + ((chunk ^ key(row)) * 16) + 8 * ((half & 1) ^ flip(row))) = v;
        }
  }
  if (TABLE && a.H) wait_vmcnt<0>();
  __syncthreads();
  auto piece = [&](int row, int chunk) {
    const uint4 v = *(const uint4*)(smem + (r0 + row) * (16 * CH) + ((chunk ^ key(r0 + row)) * 16));
    return flip(r0 + row) ? make_uint4(v.z, v.w, v.x, v.y) : v;
  };
  if (__builtin_expect(a.H != nullptr, 0)) {
#pragma unroll
    for (int it = 0; it < NIT; it++) {
      const int c = 64 * it + lane, row = c / CH, chunk = c % CH;
      const uint4 v = piece(row, chunk), hv = h[it % AHEAD];
      if (it + AHEAD < NIT) h[it % AHEAD] = fetch(it + AHEAD);
      const uint4 r = dgrad_act_piece<TABLE>(tab, v, hv);
      if (row < live_rows && 8 * chunk < live_cols) store_stream_b128(a.dX + (t0 + r0 + row) * a.lddx + i0 + 8 * chunk, r);
    }
    return;
  }
#pragma unroll
  for (int it = 0; it < NIT; it++) {
    const int c = 64 * it + lane, row = c / CH, chunk = c % CH;
    const uint4 v = piece(row, chunk);
    const int64_t t = t0 + r0 + row, i = i0 + 8 * chunk;
    if (t < a.T && i < a.I) store_stream_b128(a.dX + t * a.lddx + i, v);
  }
}

// LDS bytes of one tile: KG k-groups, NS slots of both operands each; reused by the sums of the k-groups and the epilogue.
template <bool FP8, int WF, int NT, int KG, int NS>
constexpr int dgrad_smem() {
  constexpr int RING = KG * NS * (32 * WF * (64 + (FP8 ? 16 : 8)) + 32 * NT * 128);
  constexpr int EPI = 32 * NT * 64 * WF + (dgrad_table<WF, NT>() ? GELU_TABLE_BYTES : 0);
  constexpr int RED = (KG - 1) * WF * NT * 4096;
  constexpr int M1 = RING > EPI ? RING : EPI;
  return M1 > RED ? M1 : RED;
}

// One tile: features [32 WF tm, + 32 WF) x tokens [t0, t0 + 32 NT) by KG groups of WF waves; a wave owns 32 features and all tokens, so
// that no block of the weight is decoded twice in a group.  Group kg takes the k-steps kg, kg + KG, ... and the groups' sums are added
// at the end.
template <bool FP8, bool BF8, bool M16, int WF, int NT, int KG, int NS>
__device__ __forceinline__ void dgrad_tile(uint8_t* smem, const DgradArgs& a, int tm, int64_t t0) {
  constexpr int EB = FP8 ? 1 : 2;
  constexpr int KC = FP8 ? 128 : 64;                // channels per k-step (128 bytes of a grad_Z row)
  constexpr int RBK = KC / 16;                      // packed row blocks per k-step
  constexpr int MBLK = FP8 ? 256 : 128;             // metadata bytes per packed block
  constexpr int SM = MBLK / 64;                     // ... per slot
  constexpr int BM = 32 * WF, BN = 32 * NT;
  constexpr int QT = BM / (FP8 ? 32 : 16);          // quarters of packed blocks (16 slots) along the tile's features
  constexpr int P_BYTES = BM * 64, M_BYTES = RBK * QT * 16 * SM, PSLOT = P_BYTES + M_BYTES, SLOT = PSLOT + BN * 128;
  constexpr int LP = 2, LM = M_BYTES / 256 / WF, LB = BN / 8 / WF, LPW = LP + LM + LB;   // loads per wave and k-step: packed slots, position bits, grad_Z
  static_assert(P_BYTES == LP * WF * 1024 && M_BYTES == LM * WF * 256 && LM >= 1 && LB >= 1 && LB * WF * 8 == BN && NS >= 3, "loads per wave");
  static_assert(!(FP8 && M16), "16 x 16 instructions: bf16");
  typedef DgradAcc<M16, NT> Acc;
  constexpr int MB = Acc::MB, NB = Acc::NB;
  constexpr int SUB = FP8 || M16 ? 1 : 2;           // fragments per half k-step and NB block of tokens
  constexpr int NF = 2 * SUB * NB;                  // grad_Z fragments per k-step, each for MB matrix instructions
  constexpr int FP = FP8 ? 2 : 1;                   // 16-byte pieces per fragment
  constexpr int D = FP8 ? 2 : 4;                    // fragments read ahead
  constexpr int NH = NF / 2;
  // The last k-step by itself, without the waiting, loading and decoding for a next one, and no loads of k-steps past the last ahead of the
  // first: in the small tiles, whose problems may have one or two k-steps (geometric mean over random problems of one / two k-steps: 8-bit 9 /
  // 6 % faster, bf16 6 / 2 %; the 64 x 64 tiles over all lengths 3 ... 10 %).  Long contractions gain little: the bf16 tiles of 128
  // features measured 0 ... 1 % slower and keep the plain loop, as the large tiles do.
  constexpr bool PEEL = WF == 2 || (FP8 && WF == 4);
  // The loads of a k-step are issued behind its barrier, every second fragment one where there are enough: in one burst they fill the queue
  // and stop the wave (5120 x 1280 weights, 32768 tokens, e4m3: 204 -> 196 us).  load_at(l): the fragment, counted from the barrier, with
  // which load l goes; the first L1 loads go in the k-step of the barrier, the others in the next one.
  constexpr auto load_at = [](int l) constexpr { return 2 * LPW <= NF ? 2 * l : l * NF / LPW; };
  constexpr int L1 = []() constexpr {
    int c = 0;
    for (int l = 0; l < LPW; l++) c += (2 * LPW <= NF ? 2 * l : l * NF / LPW) < D;
    return c;
  }();

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave_all = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int kg = KG > 1 ? wave_all / WF : 0, wave = KG > 1 ? wave_all % WF : wave_all;
  const int n = lane & 31, hh = lane >> 5;
  const int nsteps = (int)((a.O + KC - 1) / KC);
  const int nloc = KG > 1 ? (nsteps + KG - 1) / KG : nsteps;
  const int rbn = (int)((a.O + 15) / 16);
  uint8_t* const ring = smem + kg * NS * SLOT;
  const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_u8*)ring;

  const int rows_b = (int)((a.T - t0) < BN ? (a.T - t0) : BN);
  const i32x4 bb = rsrc_words(a.dY + t0 * a.lddy_bytes, (uint32_t)((rows_b - 1) * a.lddy_bytes + a.O * EB));
  const i32x4 bp = rsrc_words(a.vals, (uint32_t)((int64_t)rbn * a.isteps * 1024)), bm = rsrc_words(a.meta, (uint32_t)((int64_t)rbn * a.isteps * MBLK));
  const int row_bytes = (int)a.O * EB;
  constexpr uint32_t DEAD = 0x80000000u;            // offset past every descriptor: zeros arrive
  uint32_t offb[LB], offp[LP], offm[LM];
#pragma unroll
  for (int i = 0; i < LB; i++) {
    const int r = 8 * (LB * wave + i) + (lane >> 3);
    offb[i] = (uint32_t)(r * a.lddy_bytes + dy_piece(lane, LB * wave + i));
  }
  // packed slots of a k-step in LDS: [row block][quarter][row]; the row block of slot number d, and its offset in memory
  auto slot_rb = [](int d) { return d / (16 * QT); };
  auto slot_off = [&](int d, uint32_t slot_bytes) {
    const int gq = QT * tm + (d / 16) % QT;
    return (gq >> 2) < a.isteps ? (uint32_t)((slot_rb(d) * a.isteps + (gq >> 2)) * 64 + 16 * (gq & 3) + d % 16) * slot_bytes : DEAD;
  };
#pragma unroll
  for (int i = 0; i < LP; i++) offp[i] = slot_off(64 * (LP * wave + i) + lane, 16u);
#pragma unroll
  for (int i = 0; i < LM; i++) {
    const int d = 64 * (LM * wave + i) + lane;      // dword; bf16: two slots each
    offm[i] = FP8 ? slot_off(d, 4u) : slot_off(2 * d, 2u);
  }
  // Row blocks past the last one fetch nothing: asked per load, and per lane where a load covers two of them (the narrowest tile).
  constexpr bool ONE_RB = QT % 4 == 0, ONE_RBM = QT % (FP8 ? 4 : 8) == 0;
  // load number i (0 .. LPW - 1: packed slots, position bits, grad_Z) of k-step ls
  auto load = [&](int i, int ls, int slot) {
    const int st = KG > 1 ? ls * KG + kg : ls;
    const uint32_t base = lds0 + (uint32_t)(slot * SLOT);
    const uint32_t sv = (uint32_t)st * (uint32_t)(RBK * a.isteps);
    const int left = rbn - RBK * st;                // row blocks left at this k-step
    if (i < LP) {
      const int d = 64 * (LP * wave + i);
      if (ONE_RB) dma_b128(bp, base + (LP * wave + i) * 1024, offp[i < LP ? i : 0], slot_rb(d) < left ? sv * 1024u : DEAD);
      else dma_b128(bp, base + (LP * wave + i) * 1024, slot_rb(d + lane) < left ? offp[i < LP ? i : 0] : DEAD, left > 0 ? sv * 1024u : 0u);
    } else if (i < LP + LM) {
      const int m = LM * wave + (i - LP), d = 64 * m * (FP8 ? 1 : 2);
      const uint32_t om = offm[i >= LP && i < LP + LM ? i - LP : 0];
      if (ONE_RBM) dma_b32(bm, base + P_BYTES + m * 256, om, slot_rb(d) < left ? sv * (uint32_t)MBLK : DEAD);
      else dma_b32(bm, base + P_BYTES + m * 256, slot_rb(d + (FP8 ? lane : 2 * lane)) < left ? om : DEAD, left > 0 ? sv * (uint32_t)MBLK : 0u);
    } else {
      const int w = LB * wave + (i - LP - LM);
      dma_b128(bb, base + PSLOT + w * 1024, dy_offset(offb[i >= LP + LM ? i - LP - LM : 0], dy_piece(lane, w), row_bytes - 128 * st), (uint32_t)st * 128u);
    }
  };

  // Decoding: the lane's packed slot, the identity operand and the result.
  const int rho = 16 * ((n >> 2) & 1) + 4 * (n >> 3) + (n & 3);
  const int sl = FP8 ? ((2 * hh + (rho >> 4)) * QT + wave) * 16 + (rho & 15) : ((rho >> 4) * QT + 2 * wave + hh) * 16 + (rho & 15);
  constexpr int HSL = (FP8 ? 4 : 2) * QT * 16;      // slots of half a k-step
  i32x8 id0, id1;
#pragma unroll
  for (int d = 0; d < 8; d++) {
    if (FP8) {
      // bytes 0..15 of lane (n, hh) are k = 16 hh + e, bytes 16..31 k = 32 + 16 hh + e
      const int rel = n - 16 * hh - 4 * (d & 3);
      const int v = (rel >= 0 && rel < 4) ? (0x38 << (8 * rel)) : 0;
      id0[d] = d < 4 ? v : 0;
      id1[d] = d < 4 ? 0 : v;
    } else {
      // elements 0..7 are k = 8 hh + e, elements 8..15 k = 16 + 8 hh + e
      const int rel = n - (d < 4 ? 8 * hh : 16 + 8 * hh) - 2 * (d & 3);
      id0[d] = rel == 0 ? 0x3F80 : (rel == 1 ? 0x3F800000 : 0);
      id1[d] = 0;
    }
  }
  // expansion u of a half k-step (8-bit: two, of 32 channels each)
  constexpr int NU = FP8 ? 2 : 1;
  i32x4 pk;
  int pm;
  f32x16 ex;
  int fa[2][8];                                     // A fragments of the current / next half k-step
  auto slot_read = [&](int half, const uint8_t* slot) {
    pk = *(const i32x4*)(slot + (sl + half * HSL) * 16);
    if (FP8) pm = *(const int*)(slot + P_BYTES + (sl + half * HSL) * SM);
    else pm = *(const uint16_t*)(slot + P_BYTES + (sl + half * HSL) * SM);
  };
  auto unit_mma = [&](int u) {
    settle(ex);
    if (FP8) {
      ex = __builtin_amdgcn_smfmac_f32_32x32x64_fp8_fp8(pk, u ? id1 : id0, ex, pm, 0, 0);
    } else {
      bf16x8 av;
      bf16x16 bv;
      __builtin_memcpy(&av, &pk, 16);
      __builtin_memcpy(&bv, &id0, 32);
      ex = __builtin_amdgcn_smfmac_f32_32x32x32_bf16(av, bv, ex, pm, 0, 0);
    }
  };
  auto unit_cvt = [&](int u, int half, int e) {     // eighth e of the results: two values
    if (FP8) {
      int& w = fa[half][4 * u + (e >> 1)];
      if (!(e & 1)) asm("" : "=v"(w));              // both halves are written: nothing to clear first
      w = e & 1 ? __builtin_amdgcn_cvt_pk_fp8_f32(ex[2 * e], ex[2 * e + 1], w, true) : __builtin_amdgcn_cvt_pk_fp8_f32(ex[2 * e], ex[2 * e + 1], w, false);
    } else if (M16) {
      // lane (j, q) is to hold channels 8 q .. 8 q + 7 of features j and 16 + j instead of channels 16 hh .. of feature n: swapping 16-lane
      // rows between the first and the second eight channels does that
      if (e & 1) return;
      const int d = e >> 1;
      const auto sw = __builtin_amdgcn_permlane16_swap(bf16_rne_pack(ex[2 * d], ex[2 * d + 1]), bf16_rne_pack(ex[2 * d + 8], ex[2 * d + 9]), false, false);
      fa[half][d] = (int)sw[0];
      fa[half][4 + d] = (int)sw[1];
    } else {
      fa[half][e] = (int)bf16_rne_pack(ex[2 * e], ex[2 * e + 1]);
    }
  };
  // An expansion's share of the half k-step is UW matrix instructions of the product: the expansion goes with the first, the conversions
  // with the second and third quarter, zeroing for the next one with the last.  What a wave issues in one go stops its matrix instructions.
  constexpr int NHM = NH * MB, UW = NHM / NU;
  static_assert(UW * NU == NHM, "expansions of a half k-step");
  constexpr auto cvt_at = [](int e) constexpr { return UW == 1 ? 0 : UW / 4 + e * UW / 16 > 1 ? UW / 4 + e * UW / 16 : 1; };
  constexpr auto zero_at = [](int r) constexpr { return UW < 4 ? UW - 1 : 3 * UW / 4 + r * UW / 32; };

  Acc acc;
#pragma unroll
  for (int m = 0; m < MB; m++)
#pragma unroll
    for (int t = 0; t < NB; t++)
#pragma unroll
      for (int r = 0; r < 4 * Acc::G; r++) acc.v[m][t][r] = 0.f;

  // Fragment f of a k-step: half f / NH, tokens of block f % NB.  8-bit: pieces 4 half + hh and 4 half + 2 + hh of a lane's token row; bf16:
  // piece 4 half + 2 hh + sub, with 16 x 16 instructions 4 half + q.
  uint4 fb[D][FP];
  const int fn = lane % Acc::TB, fp = FP8 || M16 ? lane / Acc::TB : 2 * (lane / Acc::TB);
  const uint32_t fr = (uint32_t)(PSLOT + fn * 128 + ((fp ^ ((fn >> 1) & 7)) * 16));
  auto read_b = [&](int f, const uint8_t* slot) {
    const int half = f / NH, sub = (f / NB) % SUB, t = f % NB;
    fb[f % D][0] = *(const uint4*)(slot + (fr ^ (uint32_t)(64 * half + 16 * sub)) + t * (128 * Acc::TB));
    if (FP8) fb[f % D][FP - 1] = *(const uint4*)(slot + (fr ^ (uint32_t)(64 * half + 32)) + t * (128 * Acc::TB));
  };
  auto mma = [&](int f, int m) {
    const int half = f / NH, sub = (f / NB) % SUB, t = f % NB;
    if constexpr (FP8) {
      i32x8 av, bv;
      __builtin_memcpy(&av, &fa[half][0], 32);
      __builtin_memcpy(&bv, &fb[f % D][0], 32);
      // format arguments: A (expanded weight) e4m3; B (grad_Z) e4m3, or e5m2 when BF8; zero scales: the unscaled form
      acc.v[m][t] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(av, bv, acc.v[m][t], 0, BF8 ? 1 : 0, 0, 0, 0, 0);
    } else {
      bf16x8 av, bv;
      __builtin_memcpy(&bv, &fb[f % D][0], 16);
      if constexpr (M16) {
        __builtin_memcpy(&av, &fa[half][4 * m], 16);
        acc.v[m][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, bv, acc.v[m][t], 0, 0, 0);
      } else {
        __builtin_memcpy(&av, &fa[half][4 * sub], 16);
        acc.v[m][t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av, bv, acc.v[m][t], 0, 0, 0);
      }
    }
  };

  // prologue
  if (nloc > 0) {
#pragma unroll
    for (int k = 0; k < NS; k++) {
      if (PEEL && k >= nloc) break;             // k-steps past the last one are never multiplied
#pragma unroll
      for (int l = 0; l < LPW; l++)
        if (k < NS - 1 || l < L1) load(l, k, k);
    }
    if (PEEL && nloc < NS) wait_vmcnt<0>();     // everything; the waits of the k-steps count on loads that were not issued
    else wait_vmcnt<LB + (NS - 3) * LPW + L1>();   // packed slots of k-steps 0 and 1, grad_Z tile 0
    __syncthreads();
#pragma unroll
    for (int r = 0; r < 8; r++) zero_pair(ex, r);
#pragma unroll
    for (int u = 0; u < NU; u++) {
      if (u == 0) slot_read(0, ring);
      unit_mma(u);
#pragma unroll
      for (int e = 0; e < 8; e++) unit_cvt(u, 0, e);
#pragma unroll
      for (int r = 0; r < 8; r++) zero_pair(ex, r);
    }
#pragma unroll
    for (int f = 0; f < D; f++) read_b(f, ring);
    slot_read(1, ring);
  }

  int s = 0, slot = 0, slot1 = 1, slotp = NS - 1;
  // k-step s; behind the last one (small tiles) there is nothing to wait for, to load and to decode
  auto step = [&](auto last_) __attribute__((always_inline)) {
    constexpr bool LAST = decltype(last_)::value;
    const uint8_t* const p0 = ring + slot * SLOT;
    const uint8_t* const p1 = ring + slot1 * SLOT;
    static_for<2 * NHM>([&](auto kc) __attribute__((always_inline)) {
      constexpr int k = decltype(kc)::value, half = k / NHM, f = k / MB, mi = k % MB, m = f & 1 ? MB - 1 - mi : mi, u = k % NHM / UW, w = k % UW;
      constexpr bool DECODE = !LAST || half == 0;
      if (!LAST && f == NF - D && mi == 0) {
        // grad_Z tile s + 1 and the packed slots of s + 2 have landed (grad_Z s + 2 and what is newer may be in flight) ...
        wait_vmcnt<LB + (NS - 3) * LPW>();
        __syncthreads();                 // ... for every wave; the slot of s has been read
      }
      // decoding for the next half k-step: (s, 1) during half 0, (s + 1, 0) during half 1
      if (DECODE && w == 0) unit_mma(u);
      __builtin_amdgcn_sched_barrier(0);
      mma(f, m);
      __builtin_amdgcn_sched_barrier(0);
      if (mi == MB - 1) {
        if (f + D < NF) read_b(f + D, p0);
        else if (!LAST) read_b(f + D - NF, p1);
      }
      // k-step s + NS, into the slot that the barrier freed; not in one burst, which fills the queue and stops the wave
      if (!LAST && mi == 0) {
#pragma unroll
        for (int l = 0; l < LPW; l++) {
          if (NF - D + load_at(l) == f) load(l, s + NS, slot);
          if (load_at(l) - D == f) load(l, s + NS - 1, slotp);
        }
      }
      if (!LAST && w == 0 && u == NU - 1) slot_read(half, p1);      // the packed slot of the half after the next one
#pragma unroll
      for (int e = 0; e < 8; e++)
        if (DECODE && cvt_at(e) == w) unit_cvt(u, 1 - half, e);
#pragma unroll
      for (int r = 0; r < 8; r++)
        if (DECODE && zero_at(r) == w && !(LAST && u == NU - 1)) zero_pair(ex, r);
      __builtin_amdgcn_sched_barrier(0);
    });
    slotp = slot;
    slot = slot1;
    slot1 = slot1 == NS - 1 ? 0 : slot1 + 1;
  };
  for (; s < (PEEL ? nloc - 1 : nloc); s++) step(std::false_type());
  if (PEEL && nloc > 0) step(std::true_type());
  wait_vmcnt<0>();
  __syncthreads();
  if (KG > 1) {
    // sums of the k-groups: groups 1 .. KG - 1 leave theirs in LDS, lane for lane
    if (kg > 0) {
#pragma unroll
      for (int m = 0; m < MB; m++)
#pragma unroll
        for (int t = 0; t < NB; t++)
#pragma unroll
          for (int g = 0; g < Acc::G; g++)
            *(float4*)(smem + (((((kg - 1) * WF + wave) * MB + m) * NB + t) * Acc::G + g) * 1024 + lane * 16) =
                make_float4(acc.v[m][t][4 * g], acc.v[m][t][4 * g + 1], acc.v[m][t][4 * g + 2], acc.v[m][t][4 * g + 3]);
    }
    __syncthreads();
    if (kg == 0) {
#pragma unroll
      for (int k = 0; k < KG - 1; k++)
#pragma unroll
        for (int m = 0; m < MB; m++)
#pragma unroll
          for (int t = 0; t < NB; t++)
#pragma unroll
            for (int g = 0; g < Acc::G; g++) {
              const float4 v = *(const float4*)(smem + ((((k * WF + wave) * MB + m) * NB + t) * Acc::G + g) * 1024 + lane * 16);
              acc.v[m][t][4 * g] += v.x;
              acc.v[m][t][4 * g + 1] += v.y;
              acc.v[m][t][4 * g + 2] += v.z;
              acc.v[m][t][4 * g + 3] += v.w;
            }
    }
    __syncthreads();
  }
  dgrad_store<M16, WF, NT, KG>(smem, a, acc, kg, wave, lane, (int64_t)tm * BM, t0);
}

// ---------------------------------------------------------------------------------------------------------
// kernels: one tile shape for the whole grid; or 256 x 256 tiles (workgroups 0 .. n_big - 1: all of them, or whole rounds followed by the tiles of
// the last, partial round as twice as many 256 x 128 tiles, so that the round takes half a tile time on twice the CUs)
template <bool FP8, bool BF8, bool M16, int WF, int NT, int KG, int NS>
__global__ void __launch_bounds__(64 * WF * KG, 2)
k_linear_dgrad(DgradArgs a, int m_tiles) {
  __shared__ __align__(1024) uint8_t smem[dgrad_smem<FP8, WF, NT, KG, NS>()];
  const int logical = xcd_contiguous(blockIdx.x, gridDim.x);
  dgrad_tile<FP8, BF8, M16, WF, NT, KG, NS>(smem, a, logical % m_tiles, (int64_t)(logical / m_tiles) * (32 * NT));
}

template <bool FP8, bool BF8>
__global__ void __launch_bounds__(512, 2)
k_linear_dgrad_dual(DgradArgs a, TileOrder order, int n_big) {
  __shared__ __align__(1024) uint8_t smem[dgrad_smem<FP8, 8, 8, 1, 3>()];
  static_assert(dgrad_smem<FP8, 8, 4, 1, 4>() <= dgrad_smem<FP8, 8, 8, 1, 3>(), "the half tile fits in the full tile's LDS");
  const int bid = blockIdx.x;
  if (bid < n_big) {
    const int logical = xcd_contiguous(bid, n_big);
    int tm, tn;
    tile_at(order, logical, tm, tn);
    dgrad_tile<FP8, BF8, !FP8, 8, 8, 1, 3>(smem, a, tm, (int64_t)tn * 256);
  } else {
    const int h = xcd_contiguous(bid - n_big, (int)gridDim.x - n_big);      // half-tile number
    const int tile = n_big + (h >> 1);
    int tm, tn;
    tile_at(order, tile, tm, tn);
    const int64_t t0 = (int64_t)tn * 256 + 128 * (h & 1);
    if (t0 >= a.T) return;                     // second half of a ragged last token tile: nothing to do
    dgrad_tile<FP8, BF8, !FP8, 8, 4, 1, 4>(smem, a, tm, t0);
  }
}

// The same with 128 x 128 tiles, two of which fit a CU, and 128 x 64 halves (dgrad_halves says when and why).
template <bool FP8>
constexpr int dgrad_dual128_smem() {
  constexpr int BIG = dgrad_smem<FP8, 4, 4, 1, 3>(), HALF = dgrad_smem<FP8, 4, 2, 1, 4>();
  return BIG > HALF ? BIG : HALF;
}
template <bool FP8, bool BF8>
__global__ void __launch_bounds__(256, 2)
k_linear_dgrad_dual128(DgradArgs a, int m_tiles, int n_big) {
  __shared__ __align__(1024) uint8_t smem[dgrad_dual128_smem<FP8>()];
  static_assert(2 * dgrad_dual128_smem<FP8>() <= 160 * 1024, "two workgroups per CU");
  const int bid = blockIdx.x;
  if (bid < n_big) {
    const int logical = xcd_contiguous(bid, n_big);
    dgrad_tile<FP8, BF8, false, 4, 4, 1, 3>(smem, a, logical % m_tiles, (int64_t)(logical / m_tiles) * 128);
  } else {
    const int h = xcd_contiguous(bid - n_big, (int)gridDim.x - n_big);
    const int tile = n_big + (h >> 1);
    const int64_t t0 = (int64_t)(tile / m_tiles) * 128 + 64 * (h & 1);
    if (t0 >= a.T) return;
    dgrad_tile<FP8, BF8, false, 4, 2, 1, 4>(smem, a, tile % m_tiles, t0);
  }
}

bool linear_dgrad_supported(int64_t T, int64_t O, int64_t lddy, int64_t I, int dtype) {
  const int eb = dtype != SSTE_BF16 ? 1 : 2;
  if (product_reaches(lddy, 256 * eb, 1ll << 30)) return false;           // 32-bit offsets inside a grad_Z tile
  if (product_reaches(O / 16 * 16 + 16, I, 1ll << 31)) return false;      // packed operand addressed with 32-bit offsets
  if (product_reaches(I / 256 + 1, T / 128 + 1, 0x80000000ll)) return false;
  return true;
}

// ---------------------------------------------------------------------------------------------------------
// Choice of the tile.  Form of a time model in microseconds: a workgroup costs F + nk * step, nk = its k-steps (each k-group of a workgroup takes
// a KG-th of them) and step = max(lat, r * thr) with r workgroups sharing a CU: lat is the time one k-step's loads, barrier and
// MFMAs take end to end, thr what a CU needs per workgroup and k-step when its pipes are shared; R workgroups fit a CU (LDS), and what
// does not fit runs in further rounds; base + store * (output bytes at 5 TB/s) on top.  The two-shape grid has a row of its own.  Two sets
// of rows:
// Weights up to 5120 wide and up to 32768 tokens: the rows rank the tiles and are no times (the two-shape grid's step is 0.05 us in bf16,
// where a k-step takes 1.6); what they say ends with that range.  They are chosen for what the choice costs on 1220 random problems (64 ...
// 32768 tokens, 64 ... 5120 channels and features, a third of them layers of the GPT-2 workloads), timed in every shape: 1.4 % (bf16) / 1.3 %
// (8-bit) slower than the best shape on the geometric mean, 0.8 / 0.6 % on the GPT-2 layers, 12 / 11 % of the problems by more than 5 %,
// 28 / 24 % at worst.
// Wider weights or more tokens: rows fitted to the times themselves, no step below the matrix pipe's, so that they hold beyond what was
// timed.  2600 random problems up to 65536 wide (1 ... 262144 tokens), on one set of buffers and on sets that rotate through 600 MB: 0.2 /
// 0.1 % slower than the best shape on the geometric mean, 12 % at worst; on 1500 others 0.3 / 0.1 %, 20 / 8 %.  The first set of rows loses
// 3.6 / 3.4 % there, up to 72 % (70 x 26616 x 23872 bf16: 331 against 193 us).
struct DgradShape {
  int bm, bn, kg, r, threads;
};
struct DgradCost {
  double f, lat, thr, base, store;
};
enum { DG_256, DG_256x128, DG_128_KG1, DG_128_KG2, DG_128x64_KG2, DG_64_KG1, DG_64_KG2, DG_64_KG4, DG_SHAPES, DG_DUAL = DG_SHAPES, DG_DUAL128 };
static const DgradShape kDgrad[DG_SHAPES] = {
  {256, 256, 1, 1, 512},
  {256, 128, 1, 1, 512},
  {128, 128, 1, 2, 256},
  {128, 128, 2, 1, 512},
  {128, 64, 2, 1, 512},
  {64, 64, 1, 4, 128},
  {64, 64, 2, 2, 256},
  {64, 64, 4, 1, 512},
};
static const DgradCost kDgradCost16[DG_SHAPES] = {
  {7.215, 0.006, 0.570, 0.289, 0.007},
  {3.800, 0.533, 0.205, 0.856, 0.374},
  {1.419, 0.409, 0.267, 3.920, 0.006},
  {4.335, 0.000, 0.741, 0.013, 0.537},
  {3.600, 0.004, 0.465, 0.428, 0.064},
  {0.004, 0.823, 0.380, 1.571, 0.684},
  {1.091, 0.002, 0.287, 2.359, 2.681},
  {1.829, 0.000, 0.420, 1.904, 3.960},
};
static const DgradCost kDgradCost8[DG_SHAPES] = {
  {1.805, 0.489, 1.112, 2.327, 0.910},
  {2.388, 0.008, 0.734, 0.929, 1.177},
  {1.731, 0.084, 0.391, 3.411, 0.270},
  {2.832, 0.009, 0.805, 0.758, 1.178},
  {1.530, 0.631, 0.007, 2.535, 0.015},
  {0.002, 0.893, 0.319, 2.579, 0.799},
  {0.948, 0.146, 0.521, 2.326, 1.694},
  {2.415, 0.010, 0.829, 1.028, 8.210},
};
static const DgradCost kDgradWide16[DG_SHAPES] = {
  {9.678, 0.954, 0.954, 0.179, 0.206},
  {7.414, 0.571, 0.476, 0.115, 0.219},
  {2.873, 0.488, 0.399, 2.017, 0.220},
  {4.000, 0.804, 0.311, 0.109, 0.313},
  {3.656, 0.592, 0.161, 0.122, 0.201},
  {0.330, 0.608, 0.131, 0.154, 2.239},
  {1.614, 0.602, 0.131, 0.125, 5.994},
  {3.363, 0.701, 0.105, 0.114, 5.935},
};
static const DgradCost kDgradWide8[DG_SHAPES] = {
  {7.059, 1.139, 1.139, 0.167, 0.206},
  {4.915, 0.761, 0.585, 0.102, 0.733},
  {1.322, 0.542, 0.447, 2.774, 0.586},
  {5.048, 0.874, 0.311, 0.147, 0.720},
  {2.456, 0.893, 0.161, 1.806, 1.666},
  {0.364, 0.792, 0.173, 1.047, 3.150},
  {1.625, 0.775, 0.131, 0.126, 3.269},
  {4.510, 0.864, 0.105, 0.141, 5.854},
};
// the two-shape grid: F and step of a round of 256 x 256 tiles, of the last one of 256 x 128 tiles, base, store
struct DgradDual {
  double f, step, f_half, step_half, base, store;
};
static const DgradDual kDgradDual16 = {0.049, 0.050, 0.115, 1.037, 1.285, 1.183}, kDgradDual8 = {0.003, 0.132, 0.004, 1.789, 0.846, 1.294};
static const DgradDual kDgradWideDual16 = {9.864, 0.871, 8.078, 0.447, 4.760, 0.207}, kDgradWideDual8 = {8.835, 0.884, 0.984, 1.225, 3.051, 0.203};

// 128 x 128 tiles that are more than one per CU and at most one and a half: the excess runs as twice as many 128 x 64 halves, so that every CU gets
// one tile and at most one half instead of some of them two tiles.  On 220 + 180 random problems of that kind (weights up to 5120 wide; wider ones
// and more tokens), against the shape that the rows below choose: bf16 11 / 9 % faster on the geometric mean, 8-bit 10 / 7 % up to 20 k-steps and
// 2 ... 7 % slower beyond 23, where the 256 x 128 tiles' fewer expansions win.  Shorter contractions are left to the plain tiles, which the tests hold
// to them in this range; that costs 8 bits 2 ... 33 % (one to four k-steps, 16 problems) and bf16 13 ... 30 % at four and five (9 problems), and bf16
// between -17 and +26 % at one and two.
// Not taken where it lost: features that fill less than three quarters of their tiles (64 of them: 0 ... 13 % slower than 64 x 64 tiles, 3 % faster at
// best), and below 512 tokens, where the last token tile may be mostly padding.
// The gain depends on grad_Z being in the cache, as it is behind the kernel that wrote it.  Read from memory (285 problems on buffers of 700 MB), the
// halves are 0 ... 33 % faster too where grad_Z's rows are whole 128-byte lines (one problem 6 % slower) and wherever the other choice is 128 x 128 tiles;
// against 256 x 128 tiles, which read grad_Z half as often, rows that end inside a line cost up to 640 features 2 ... 16 % (17239 x 4008 x 192: 55.8
// against 65.3 us, from the cache 50.0 against 43.1), from about 1000 channels on; shorter contractions gain.  (8192 x 3072 x 768 bf16: 44.6 -> 41.0 us.)
static bool dgrad_halves(bool fp8, int64_t T, int64_t steps, int64_t I) {
  const int64_t mt = (I + 127) / 128, tiles = mt * ((T + 127) / 128);
  return T >= 512 && 4 * I >= 3 * 128 * mt && tiles > 256 && tiles <= 384 && (fp8 ? steps >= 5 && steps <= 20 : steps >= 6);
}

static int dgrad_choice(bool fp8, int64_t T, int64_t O, int64_t I) {
  const bool wide = O > 5120 || I > 5120 || T > 32768;
  const DgradCost* cost = wide ? (fp8 ? kDgradWide8 : kDgradWide16) : (fp8 ? kDgradCost8 : kDgradCost16);
  const DgradDual& dual = wide ? (fp8 ? kDgradWideDual8 : kDgradWideDual16) : (fp8 ? kDgradDual8 : kDgradDual16);
  const int64_t steps = (O + (fp8 ? 127 : 63)) / (fp8 ? 128 : 64);
  if (dgrad_halves(fp8, T, steps, I)) return DG_DUAL128;
  const double out_us = (double)T * (double)I * 2.0 / 5e6;
  int best = DG_256;
  double best_t = 1e30;
  for (int c = 0; c < DG_SHAPES; c++) {
    const DgradShape& g = kDgrad[c];
    const DgradCost& s = cost[c];
    const int64_t wgs = ((I + g.bm - 1) / g.bm) * ((T + g.bn - 1) / g.bn);
    if (c != DG_256 && wgs > 0x7FFFFFFFll) continue;                                  // grid size
    const double nk = (double)((steps + g.kg - 1) / g.kg);
    const int64_t n = (wgs + 255) / 256, full = n / g.r, rem = n % g.r;      // workgroups on the busiest CU: full rounds of r, and a rest
    double t = s.base + s.store * out_us + (double)full * (s.f + nk * (s.lat > g.r * s.thr ? s.lat : g.r * s.thr));
    if (rem) t += s.f + nk * (s.lat > rem * s.thr ? s.lat : rem * s.thr);
    if (t < best_t) {
      best_t = t;
      best = c;
    }
    // 256 x 256 tiles whose last round is at most half full: that round as 256 x 128 tiles
    if (c == DG_256 && wgs > 256 && wgs % 256 != 0 && wgs % 256 <= 128) {
      const double td = dual.base + dual.store * out_us + (double)(wgs / 256) * (dual.f + nk * dual.step) + dual.f_half + nk * dual.step_half;
      if (td < best_t) {
        best_t = td;
        best = DG_DUAL;
      }
    }
  }
  return best;
}

void describe_dgrad(int64_t T, int64_t O, int64_t I, int dtype, char* text, size_t n) {
  const int cfg = dgrad_choice(dtype != SSTE_BF16, T, O, I);
  if (cfg == DG_DUAL) {
    const int64_t big = ((I + 255) / 256) * ((T + 255) / 256);
    snprintf(text, n, "256x256+256x128 kg 1 r 1 grid %lld block 512", (long long)(big + big % 256));
    return;
  }
  if (cfg == DG_DUAL128) {
    const int64_t tiles = ((I + 127) / 128) * ((T + 127) / 128);
    snprintf(text, n, "128x128+128x64 kg 1 r 2 grid %lld block 256", (long long)(2 * tiles - 256));
    return;
  }
  const DgradShape& s = kDgrad[cfg];
  snprintf(text, n, "%dx%d kg %d r %d grid %lld block %d", s.bm, s.bn, s.kg, s.r, (long long)(((I + s.bm - 1) / s.bm) * ((T + s.bn - 1) / s.bn)), s.threads);
}

template <bool FP8, bool BF8>
static void launch_dgrad_type(const DgradArgs& a, hipStream_t s) {
  const int m256 = (int)((a.I + 255) / 256);
  const int cfg = dgrad_choice(FP8, a.T, a.O, a.I);
  auto tile = [&](auto kernel, int bm, int bn, int threads) {
    const int mt = (int)((a.I + bm - 1) / bm);
    SSTE_LAUNCH(SSTE_K_DGRAD, kernel, dim3((unsigned)(mt * ((a.T + bn - 1) / bn))), dim3(threads), s, a, mt);
  };
  switch (cfg) {
    case DG_256:
    case DG_DUAL: {
      const int64_t big = (int64_t)m256 * ((a.T + 255) / 256), rem = cfg == DG_DUAL ? big % 256 : 0;
      SSTE_LAUNCH(SSTE_K_DGRAD, (k_linear_dgrad_dual<FP8, BF8>), dim3((unsigned)(big + rem)), dim3(512), s, a, tile_order(m256, (a.T + 255) / 256), (int)(big - rem));
      break;
    }
    case DG_DUAL128: {
      const int m128 = (int)((a.I + 127) / 128), tiles = m128 * (int)((a.T + 127) / 128);
      SSTE_LAUNCH(SSTE_K_DGRAD, (k_linear_dgrad_dual128<FP8, BF8>), dim3((unsigned)(2 * tiles - 256)), dim3(256), s, a, m128, 256);
      break;
    }
    case DG_256x128: tile(k_linear_dgrad<FP8, BF8, !FP8, 8, 4, 1, 4>, 256, 128, 512); break;
    case DG_128_KG1: tile(k_linear_dgrad<FP8, BF8, false, 4, 4, 1, 3>, 128, 128, 256); break;
    case DG_128_KG2: tile(k_linear_dgrad<FP8, BF8, false, 4, 4, 2, 3>, 128, 128, 512); break;
    case DG_128x64_KG2: tile(k_linear_dgrad<FP8, BF8, false, 4, 2, 2, 3>, 128, 64, 512); break;
    case DG_64_KG1: tile(k_linear_dgrad<FP8, BF8, false, 2, 2, 1, 3>, 64, 64, 128); break;
    case DG_64_KG2: tile(k_linear_dgrad<FP8, BF8, false, 2, 2, 2, 3>, 64, 64, 256); break;
    default: tile(k_linear_dgrad<FP8, BF8, false, 2, 2, 4, 3>, 64, 64, 512); break;
  }
}

hipError_t launch_linear_dgrad(const void* dY, int64_t T, int64_t O, int64_t lddy, int dtype, float scale, const void* vals,
                               const void* meta, int64_t I, void* dX, int64_t lddx, const void* H, int64_t ldh, hipStream_t s) {
  if (T == 0 || I == 0) return hipSuccess;
  const bool fp8 = dtype != SSTE_BF16;
  DgradArgs a;
  a.dY = (const uint8_t*)dY;
  a.T = T;
  a.O = O;
  a.lddy_bytes = lddy * (fp8 ? 1 : 2);
  a.vals = (const uint8_t*)vals;
  a.meta = (const uint8_t*)meta;
  a.I = I;
  a.isteps = (int)(I / (fp8 ? 128 : 64));
  a.scale = scale;
  a.dX = (uint16_t*)dX;
  a.lddx = lddx;
  a.H = (const uint16_t*)H;
  a.ldh = ldh;
  if (dtype == SSTE_F8E5M2) launch_dgrad_type<true, true>(a, s);
  else if (fp8) launch_dgrad_type<true, false>(a, s);
  else launch_dgrad_type<false, false>(a, s);
  return hipGetLastError();
}

}  // namespace sste
