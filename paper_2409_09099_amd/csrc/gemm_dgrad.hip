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
// The packed operand runs along features, the contraction along channels: decoding it means transposing it.  Three
// ways of doing that, each kept where it measured best:
//   dgrad_direct_tile  bf16, 256 features x 256 or 128 tokens.  The sparse matrix instruction itself decodes and
//       transposes: S_block x identity (v_smfmac_f32_32x32x32_bf16 with the packed slots as operand A, exactly as they
//       lie in memory) leaves in lane (n, hh) sixteen channels of feature n as float32, exactly (one term per sum).
//       With the packed rows assigned to the instruction's rows in the order rho(m) = 16 (m / 4 % 2) + 4 (m / 8) + m % 4
//       the sixteen channels are consecutive: converted to bf16 they ARE the operand fragments of two
//       v_mfma_f32_32x32x16_bf16, and S(W) never passes through the LDS in dense form.  Costs one matrix instruction per
//       eight of the product, 24 vector instructions and no LDS writes per 32 x 32 block (LDS writes run at 76 B/clk per
//       CU, reads at 233; shifting the values to their places took 130 vector instructions).
//   dgrad8_tile        8-bit, the same tile sizes: a group expands with one byte permute and is written to LDS as
//       dense channel rows, read back with the transposing load.  (There the identity costs two 32x32x64 instructions per
//       block, a quarter of the product's matrix time in the direct form.)
//   dgrad_tile         both types, 128 x 128 and 64 x 64 tiles: S_block x identity, the result written to LDS as
//       feature rows of channels (the form of the grad_Z tile), once per workgroup.  With KG > 1 the workgroup's waves
//       form KG groups that take the k-steps in turn, each with its own LDS slots, and add their sums at the end: a
//       problem with few tiles is bound by the time a k-step's loads take to arrive (about 1 us with one k-step in
//       flight), not by any rate, and KG k-steps in flight divide that.
// The identity product is exact for finite values; an infinite or NaN packed value (the interface rules them out) makes NaN of the 32
// features it is expanded with.  Asking every packed slot for one, with a second look in a branch, was measured: 2.1 % of a four-layer
// training step in bf16 (1668 -> 1704 us), 1.8 % of an 8-bit layer of small tiles, so it is not asked.
// Which tile runs is decided by a time model fitted to a sweep (dgrad_choice).
// Measured (us before -> after; start: 256-token tiles or their halves only): bf16 512 x 256 x 1024 (T, O, I)
// 8.2 -> 4.1, 1024^3 20.9 -> 7.8, 2048 x 4096 x 1024 72 -> 33, 4096 x 3072 x 768 54 -> 32, 8192 x 3072 x 768 57 -> 49,
// 16384 x 1280 x 5120 206 -> 195; e4m3 2048 x 4096 x 1024 36 -> 21.
// Epilogue as in the forward GEMM: transposed through LDS, 16-byte streaming stores of bf16 rows.
#include "common.h"

#include <stdio.h>

namespace sste {

namespace {
typedef __attribute__((address_space(3))) i32x2 lds_i32x2;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;
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

// One group of a packed e4m3 operand -> its four dense bytes: w holds value0 at byte b0 and value1 at byte b0 + 1, nib =
// pos0 | pos1 << 2.  A byte permute with a computed selector: selector bytes 0..3 pick from the zero operand, 4..7 from w.
__device__ __forceinline__ uint32_t expand_group8(uint32_t w, uint32_t b0, uint32_t nib) {
  const uint32_t sel = ((4u + b0) << (((nib & 3u) << 3) & 31u)) | ((5u + b0) << (((nib & 12u) << 1) & 31u));
  return __builtin_amdgcn_perm(w, 0u, sel);
}
}  // namespace

// grad_Z loads.  A row's bytes past its last channel belong to somebody else (the next token's row, padding of any content): S(W) has
// zeros there, but zero times a NaN pattern is NaN, so the 16-byte pieces past the last channel are pushed out of range and arrive as zeros.
// `live` bytes of a row are left at this k-step (O x element size - 128 x step), `piece` = 16 x the piece's number inside the k-step.
constexpr uint32_t NO_PIECE = 0x80000000u;
__device__ __forceinline__ uint32_t dy_offset(uint32_t off, int piece, int live) { return piece < live ? off : NO_PIECE; }
// the piece a lane fetches in load number wl of a tile (8 rows x 128 bytes per load, row r's piece c at position c ^ ((r / 2) % 8)), times 16
__device__ __forceinline__ int dy_piece(int lane, int wl) { return 16 * ((lane & 7) ^ ((4 * (wl & 1) + (lane >> 4)) & 7)); }

// sixteen accumulator registers set to zero by sixteen moves (the compiler otherwise builds a zero vector and copies it).  Only where no
// matrix instruction that writes them is in flight: the compiler does not order what it cannot see inside the assembly.
__device__ __forceinline__ void zero16(f32x16& v) {
#pragma unroll
  for (int r = 0; r < 16; r++) {
    float z;
    asm("v_mov_b32 %0, 0" : "=v"(z));
    v[r] = z;
  }
}

// Stores a wave's tile with the backward of the activation that produced this layer's input: grad_H = grad_A * GELU'(H), on the bf16
// gradient just formed (`piece(row, chunk)`: 16 bytes of it) and the stored pre-activation.  The tile's corner is (t0, i0), `rows` tokens
// of `ch` 16-byte chunks, NIT chunks per lane.  H is requested AHEAD chunks in advance: asked for one by one, each between its bounds
// check and its use, the loads cost a memory latency each (32768 x 1280 x 5120 e5m2: 380 -> 338 us, 277 without the activation;
// 16384 x 1024 x 4096 bf16: 181 -> 164; 8192 x 768 x 3072 e4m3: 49 -> 44).
template <int NIT, class Piece>
__device__ __forceinline__ void dgrad_store_act(const DgradArgs& a, int64_t t0, int64_t i0, int rows, int ch, int lane, Piece piece) {
  if (t0 >= a.T || i0 >= a.I) return;
  constexpr int AHEAD = NIT < 8 ? NIT : 8;
  const int live_rows = (int)(a.T - t0 < rows ? a.T - t0 : rows), live_cols = (int)(a.I - i0 < 8 * ch ? a.I - i0 : 8 * ch);
  uint4 h[AHEAD];
  auto fetch = [&](int it) {                        // a lane outside the matrix reads the tile's first chunk
    const int c = 64 * it + lane, row = c / ch, chunk = c % ch;
    const bool live = row < live_rows && 8 * chunk < live_cols;
    const i32x4 v = __builtin_nontemporal_load((const i32x4*)(a.H + (t0 + (live ? row : 0)) * a.ldh + i0 + (live ? 8 * chunk : 0)));
    return make_uint4((uint32_t)v[0], (uint32_t)v[1], (uint32_t)v[2], (uint32_t)v[3]);
  };
#pragma unroll
  for (int it = 0; it < AHEAD; it++) h[it] = fetch(it);
#pragma unroll
  for (int it = 0; it < NIT; it++) {
    const int c = 64 * it + lane, row = c / ch, chunk = c % ch;
    const uint4 v = piece(row, chunk), hv = h[it % AHEAD];
    if (it + AHEAD < NIT) h[it % AHEAD] = fetch(it + AHEAD);
    const uint32_t g[4] = {v.x, v.y, v.z, v.w}, hw[4] = {hv.x, hv.y, hv.z, hv.w};
    uint32_t r[4];
#pragma unroll
    for (int e = 0; e < 4; e++)
      r[e] = bf16_rne_pack(bf16lo_f32(g[e]) * gelu_tanh_grad(bf16lo_f32(hw[e])), bf16hi_f32(g[e]) * gelu_tanh_grad(bf16hi_f32(hw[e])));
    if (row < live_rows && 8 * chunk < live_cols) store_stream_b128(a.dX + (t0 + row) * a.lddx + i0 + 8 * chunk, make_uint4(r[0], r[1], r[2], r[3]));
  }
}

// Output stage of one wave: accumulators -> LDS (row = token, the wave's 32 MT features contiguous) -> 16-byte stores.  Chunk c
// of token row t sits at c ^ key(t), and rows with bit 4 set have the 8-byte halves of their chunks swapped: every write and read
// then covers all banks.
template <int WM, int WN, int MT, int NT>
__device__ __forceinline__ void dgrad_store(uint8_t* smem, const DgradArgs& a, const f32x16 (&acc)[MT][NT], int wave, int lane, int64_t i0,
                                            int64_t t0) {
  constexpr int CH = 4 * MT, NIT = 32 * NT * CH / 64;   // 16-byte chunks per token row of the wave; chunks per lane
  const int wm = wave / WN, wn = wave % WN;
  const int n = lane & 31, hh = lane >> 5;
  uint8_t* const eb = smem + wave * (32 * NT) * (64 * MT);
  const float scale = a.scale;
  auto key = [](int row) { return CH >= 16 ? (row & 15) : (row / (16 / CH)) % CH; };
#pragma unroll
  for (int t = 0; t < NT; t++)
#pragma unroll
    for (int m = 0; m < MT; m++)
#pragma unroll
      for (int g = 0; g < 4; g++) {
        uint2 v;
        v.x = bf16_rne_pack(acc[m][t][4 * g] * scale, acc[m][t][4 * g + 1] * scale);
        v.y = bf16_rne_pack(acc[m][t][4 * g + 2] * scale, acc[m][t][4 * g + 3] * scale);
        const int row = 32 * t + n;
        *(uint2*)(eb + row * (64 * MT) + (((4 * m + g) ^ key(row)) * 16) + 8 * (hh ^ (n >> 4))) = v;
      }
  if (a.H) {
    dgrad_store_act<NIT>(a, t0 + 32 * NT * wn, i0 + 32 * MT * wm, 32 * NT, CH, lane, [&](int row, int chunk) {
      const uint4 v = *(const uint4*)(eb + row * (64 * MT) + ((chunk ^ key(row)) * 16));
      return ((row >> 4) & 1) ? make_uint4(v.z, v.w, v.x, v.y) : v;
    });
    return;
  }
#pragma unroll
  for (int it = 0; it < NIT; it++) {
    const int c = 64 * it + lane, row = c / CH, chunk = c % CH;
    uint4 v = *(const uint4*)(eb + row * (64 * MT) + ((chunk ^ key(row)) * 16));
    if ((row >> 4) & 1) v = make_uint4(v.z, v.w, v.x, v.y);
    const int64_t t = t0 + 32 * NT * wn + row, i = i0 + 32 * MT * wm + 8 * chunk;
    if (t < a.T && i < a.I) store_stream_b128(a.dX + t * a.lddx + i, v);
  }
}

// ---------------------------------------------------------------------------------------------------------
// Tiles with the decoded weight in LDS.  A k-step is cut into stages (one k-slice of the MFMA tiles each); the fragments of the
// next stage are read while the MFMAs of the current one run.  The only barrier of a k-step stands before its LAST stage, whose
// fragments are in registers by then: behind it the slots of this k-step are free, the tiles of the next one are complete, and its
// first fragments can be read under the last stage's MFMAs.
// LDS bytes of one tile: KG k-groups, each two slots of both operands; reused by the epilogue.
template <int WM, int WN, int MT, int NT, int KG, int NSB>
constexpr int dgrad_smem() {
  constexpr int RING = KG * 128 * 32 * (2 * WM * MT + NSB * WN * NT);
  constexpr int EPI = WM * WN * (32 * NT) * (64 * MT);
  constexpr int RED = (KG - 1) * WM * WN * MT * NT * 4096;
  constexpr int M1 = RING > EPI ? RING : EPI;
  return M1 > RED ? M1 : RED;
}

// One tile: features [i0, i0 + 32 WM MT) x tokens [t0, t0 + 32 WN NT) by KG groups of WM x WN waves; wave (wm, wn) of a group
// owns 32 MT features x 32 NT tokens.  Group kg takes the k-steps kg, kg + KG, ... and the groups' sums are added at the end.
template <bool FP8, bool BF8, int WM, int WN, int MT, int NT, int KG, int NSB>
__device__ __forceinline__ void dgrad_tile(uint8_t* smem, const DgradArgs& a, int64_t i0, int64_t t0) {
  constexpr int NWG = WM * WN;
  constexpr int EB = FP8 ? 1 : 2;
  constexpr int KC = FP8 ? 128 : 64;                // channels per k-step (128 bytes of a grad_Z row)
  constexpr int RBK = KC / 16;                      // packed row blocks per k-step
  constexpr int MBLK = FP8 ? 256 : 128;             // metadata bytes per packed block
  constexpr int BM = 32 * WM * MT, BN = 32 * WN * NT;
  constexpr int ASLOT = BM * 128, BSLOT = BN * 128;
  constexpr int LB = BN / 8 / NWG;                  // direct-to-LDS loads (8 token rows, 1 KiB) per wave and k-step
  constexpr int EBK = BM / 16 / NWG;                // packed blocks per wave and k-step: 32 channels x 32 (bf16) / 64 (8-bit) features
  constexpr int NU = FP8 ? 2 * EBK : EBK;           // expansion instructions per wave and k-step
  constexpr int NU0 = NU > 2 ? NU / 2 : (FP8 ? 1 : NU);            // ... of which in the last stage (the rest in the next k-step's first)
  constexpr int PPF = FP8 ? 2 : 1;                  // 16-byte pieces per fragment
  constexpr int NSTG = FP8 ? 2 : 4;                 // stages per k-step: k-slices of the MFMA tiles
  static_assert(LB >= 1 && EBK >= 1, "tile too small for this many waves");

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave_all = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int kg = KG > 1 ? wave_all / NWG : 0, wave = KG > 1 ? wave_all % NWG : wave_all;
  const int wm = wave / WN, wn = wave % WN;
  const int n = lane & 31, hh = lane >> 5;
  const int nsteps = (int)((a.O + KC - 1) / KC);
  const int nloc = KG > 1 ? (nsteps + KG - 1) / KG : nsteps;
  const int64_t rbn = (a.O + 15) / 16;
  uint8_t* const smemA = smem + kg * (2 * ASLOT + NSB * BSLOT);
  uint8_t* const smemB = smemA + 2 * ASLOT;

  // grad_Z tile
  const int rows_b = (int)((a.T - t0) < BN ? (a.T - t0) : BN);
  const i32x4 bb = rsrc_words(a.dY + t0 * a.lddy_bytes, (uint32_t)((rows_b - 1) * a.lddy_bytes + a.O * EB));
  const int row_bytes = (int)a.O * EB;
  uint32_t offb[LB];
#pragma unroll
  for (int i = 0; i < LB; i++) {
    const int r = 8 * (LB * wave + i) + (lane >> 3);
    offb[i] = (uint32_t)(r * a.lddy_bytes + dy_piece(lane, LB * wave + i));
  }
  const uint32_t ldsB = (uint32_t)(uintptr_t)(lds_u8*)smemB;

  // packed S(W)
  const int rho = 16 * ((n >> 2) & 1) + 4 * (n >> 3) + (n & 3);
  constexpr int CB = FP8 ? 4 : 2;                   // 32-channel blocks per k-step
  // block e of a wave: channel block (first + e) % CB of feature block (first + e) / CB, first = EBK * wave
  static_assert(EBK == 1 || EBK == 2 || EBK == 4, "blocks of a wave: consecutive channel blocks, then the next features");
  const int fbk = EBK * wave / CB, cbk = EBK * wave % CB;
  const int fblk = (int)(i0 / (FP8 ? 64 : 32)) + fbk;
  const int rb_loc = 2 * cbk + (rho >> 4);
  const uint32_t pv_off = (uint32_t)(rb_loc * a.isteps + (fblk >> 1)) * 1024u + (uint32_t)(16 * (2 * (fblk & 1) + hh) + (rho & 15)) * 16u;
  const bool f_live = (fblk >> 1) < a.isteps;       // column steps past the last feature have nothing to fetch
  const uint32_t wr_off = (uint32_t)(((FP8 ? 64 : 32) * fbk + n) * 128 + (((FP8 ? 2 * cbk + hh : 4 * cbk + 2 * hh) ^ ((n >> 1) & 7)) * 16));
  static_assert(EBK <= CB || !FP8, "8-bit: a wave's blocks share their features");
  // operand B of the expansion: the identity (bf16), the two halves of one (8-bit)
  i32x8 sel0, sel1;
#pragma unroll
  for (int d = 0; d < 8; d++) {
    if (FP8) {
      // bytes 0..15 of lane (n, hh) are k = 16 hh + e, bytes 16..31 k = 32 + 16 hh + e
      const int rel = n - 16 * hh - 4 * (d & 3);
      const int v = (rel >= 0 && rel < 4) ? (0x38 << (8 * rel)) : 0;
      sel0[d] = d < 4 ? v : 0;
      sel1[d] = d < 4 ? 0 : v;
    } else {
      // elements 0..7 are k = 8 hh + e, elements 8..15 k = 16 + 8 hh + e
      const int rel = n - (d < 4 ? 8 * hh : 16 + 8 * hh) - 2 * (d & 3);
      sel0[d] = rel == 0 ? 0x3F80 : (rel == 1 ? 0x3F800000 : 0);
      sel1[d] = 0;
    }
  }

  i32x4 pk[EBK];
  int pm[EBK];
  const BufferRsrc rv = make_rsrc(a.vals, (uint32_t)(rbn * a.isteps * 1024)), rm = make_rsrc(a.meta, (uint32_t)(rbn * a.isteps * MBLK));
  auto load_packed = [&](int step) {
    const uint32_t sv = (uint32_t)step * (uint32_t)RBK * (uint32_t)a.isteps;
#pragma unroll
    for (int e = 0; e < EBK; e++) {
      // row blocks past the last one read as zeros; a slot's position bits lie at its offset times MBLK / 1024
      const int ec = e % CB, ef = e / CB;           // further channel blocks / 32 features (bf16 only: half a packed block)
      const bool live = f_live && RBK * step + 2 * ec + rb_loc < (int)rbn;
      const uint32_t off = live ? pv_off + 512u * ef : 0x80000000u;
      const uint32_t offm = live ? (pv_off + 512u * ef) / (1024 / MBLK) : 0x80000000u;
      const uint32_t se = RBK * step + 2 * ec < (int)rbn ? sv + (uint32_t)(2 * ec * a.isteps) : 0u;
      pk[e] = __builtin_amdgcn_raw_buffer_load_b128(rv, (int)off, (int)(se * 1024u), 0);
      pm[e] = FP8 ? (int)__builtin_amdgcn_raw_buffer_load_b32(rm, (int)offm, (int)(se * (uint32_t)MBLK), 0)
                  : (int)__builtin_amdgcn_raw_buffer_load_b16(rm, (int)offm, (int)(se * (uint32_t)MBLK), 0);
    }
  };
  f32x16 ex;
  auto expand_mma = [&](int u) {
    const int e = FP8 ? u >> 1 : u;
    zero16(ex);
    if (FP8) {
      ex = __builtin_amdgcn_smfmac_f32_32x32x64_fp8_fp8(pk[e], (u & 1) ? sel1 : sel0, ex, pm[e], 0, 0);
    } else {
      bf16x8 av;
      bf16x16 bv;
      __builtin_memcpy(&av, &pk[e], 16);
      __builtin_memcpy(&bv, &sel0, 32);
      ex = __builtin_amdgcn_smfmac_f32_32x32x32_bf16(av, bv, ex, pm[e], 0, 0);
    }
  };
  auto expand_store = [&](int u, uint8_t* slot) {
    const int e = FP8 ? u >> 1 : u;
    if (FP8) {
      int w[4];
#pragma unroll
      for (int d = 0; d < 4; d++) {
        w[d] = __builtin_amdgcn_cvt_pk_fp8_f32(ex[4 * d], ex[4 * d + 1], 0, false);
        w[d] = __builtin_amdgcn_cvt_pk_fp8_f32(ex[4 * d + 2], ex[4 * d + 3], w[d], true);
      }
      *(uint4*)(slot + (wr_off ^ (uint32_t)(32 * e)) + (u & 1) * 4096) = make_uint4((uint32_t)w[0], (uint32_t)w[1], (uint32_t)w[2], (uint32_t)w[3]);
    } else {
      uint32_t w[8];
#pragma unroll
      for (int d = 0; d < 8; d++) w[d] = bf16_rne_pack(ex[2 * d], ex[2 * d + 1]);
      *(uint4*)(slot + (wr_off ^ (uint32_t)(64 * (e % CB))) + 4096 * (e / CB)) = make_uint4(w[0], w[1], w[2], w[3]);
      *(uint4*)(slot + (wr_off ^ (uint32_t)(64 * (e % CB) + 16)) + 4096 * (e / CB)) = make_uint4(w[4], w[5], w[6], w[7]);
    }
  };
  auto dma_b = [&](int i, int step, int slot) {
    // a k-step past the last one (of a k-group) has no live piece: zeros against the zeros of its S(W) tile
    dma_b128(bb, ldsB + (uint32_t)(slot * BSLOT + (LB * wave + i) * 1024), dy_offset(offb[i], dy_piece(lane, LB * wave + i), row_bytes - 128 * step),
             (uint32_t)step * 128u);
  };
  auto gstep = [&](int ls) { return KG > 1 ? ls * KG + kg : ls; };

  f32x16 acc[MT][NT];
#pragma unroll
  for (int m = 0; m < MT; m++)
#pragma unroll
    for (int t = 0; t < NT; t++)
#pragma unroll
      for (int r = 0; r < 16; r++) acc[m][t][r] = 0.f;

  // fragment addresses: piece 2 kk + hh of the lane's row
  uint32_t fr[4];
#pragma unroll
  for (int kk = 0; kk < 4; kk++) fr[kk] = (uint32_t)(n * 128 + (((2 * kk + hh) ^ ((n >> 1) & 7)) * 16));
  const uint32_t fa_base = (uint32_t)(wm * MT * 4096), fb_base = (uint32_t)(wn * NT * 4096);

  uint4 fa[2][MT][PPF], fb[2][NT][PPF];
  // fragment read number k of stage st: first A's, then B's
  constexpr int NRA = MT * PPF, NRB = NT * PPF;
  auto read_frag = [&](int st, int k, const uint8_t* sa, const uint8_t* sb) {
    if (k < NRA) {
      const int m = k / PPF, p = k % PPF;
      fa[st & 1][m][p] = *(const uint4*)(sa + fa_base + m * 4096 + fr[PPF * st + p]);
    } else {
      const int t = (k - NRA) / PPF, p = (k - NRA) % PPF;
      fb[st & 1][t][p] = *(const uint4*)(sb + fb_base + t * 4096 + fr[PPF * st + p]);
    }
  };
  auto mma = [&](int st, int k) {                   // MFMA k of stage st
    const int m = k / NT, t = k % NT;
    f32x16& c = acc[m][t];
    if (FP8) {
      i32x8 av, bv;
      __builtin_memcpy(&av, &fa[st & 1][m][0], 32);
      __builtin_memcpy(&bv, &fb[st & 1][t][0], 32);
      // format arguments: A (expanded weight) e4m3; B (grad_Z) e4m3, or e5m2 when BF8; zero scales: the unscaled form
      c = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(av, bv, c, 0, BF8 ? 1 : 0, 0, 0, 0, 0);
    } else {
      bf16x8 av, bv;
      __builtin_memcpy(&av, &fa[st & 1][m][0], 16);
      __builtin_memcpy(&bv, &fb[st & 1][t][0], 16);
      c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av, bv, c, 0, 0, 0);
    }
  };
  constexpr int NM = MT * NT;                      // MFMAs per stage
  constexpr int RDW = NM > 4 ? NM / 2 : 1;          // ... of which the first RDW have the next stage's fragment reads between them
  // The MFMAs of stage st; between them the fragment reads of stage st_n (slots na, nb), expansion units u0 .. u0 + nu - 1 (if on;
  // an expansion's result is only converted after further MFMAs) and, behind the last of them, the requests of k-step `lstep`'s
  // packed blocks (if lon) and then of grad_Z tile `dstep` (if don): in this order, since loads complete in order and a barrier
  // waits for packed blocks while a newer grad_Z tile may still be in flight.
  auto stage = [&](int st, int st_n, const uint8_t* na, const uint8_t* nb, int u0, int nu, bool on, uint8_t* slot, bool loads, bool lon,
                   int lstep, bool don, int dstep, int dslot) {
    const int kl = nu ? (nu - 1) * NM / nu : 0;      // MFMA in front of which the last expansion is issued
#pragma unroll
    for (int k = 0; k < NM; k++) {
#pragma unroll
      for (int r = 0; r < NRA + NRB; r++)
        if (r * RDW / (NRA + NRB) == k) read_frag(st_n, r, na, nb);
#pragma unroll
      for (int u = 0; u < nu; u++)
        if (u * NM / nu == k && on) expand_mma(u0 + u);
      __builtin_amdgcn_sched_barrier(0);
      mma(st, k);
      __builtin_amdgcn_sched_barrier(0);
      if (loads && k == kl) {
        if (lon) load_packed(lstep);
        if (don) {
#pragma unroll
          for (int i = 0; i < LB; i++) dma_b(i, dstep, dslot);
        }
      }
#pragma unroll
      for (int u = 0; u < nu; u++)
        if ((u + 1) * NM / nu - 1 == k && on) expand_store(u0 + u, slot);
    }
    __builtin_amdgcn_sched_barrier(0);
  };

  // prologue: grad_Z tiles 0 .. NSB - 2 (and NSB - 1 where the loads go with the last stage), S(W) tiles 0 and (first units) 1
  constexpr bool LATE = NU0 == NU;                   // all units of a k-step fit in its last stage: the next loads follow there
  if (nloc > 0) {
    load_packed(gstep(0));
#pragma unroll
    for (int k = 0; k < NSB - 1; k++)
      if (k < nloc)
#pragma unroll
        for (int i = 0; i < LB; i++) dma_b(i, gstep(k), k);
    wait_vmcnt<0>();
#pragma unroll
    for (int u = 0; u < NU; u++) {
      expand_mma(u);
      expand_store(u, smemA);
    }
    if (nloc > 1) {
      load_packed(gstep(1));
      wait_vmcnt<0>();
#pragma unroll
      for (int u = 0; u < NU0; u++) {
        expand_mma(u);
        expand_store(u, smemA + ASLOT);
      }
      if (LATE && nloc > 2) load_packed(gstep(2));
    }
    if (LATE && NSB - 1 < nloc)
#pragma unroll
      for (int i = 0; i < LB; i++) dma_b(i, gstep(NSB - 1), NSB - 1);
    __syncthreads();
#pragma unroll
    for (int r = 0; r < NRA + NRB; r++) read_frag(0, r, smemA, smemB);
  }

  int sb0 = 0, sb1 = 1;                              // grad_Z slots of k-steps s and s + 1
  for (int s = 0; s < nloc; s++) {
    uint8_t* const a0 = smemA + (s & 1) * ASLOT;
    uint8_t* const a1 = smemA + ((s & 1) ^ 1) * ASLOT;
    const uint8_t* const b0 = smemB + sb0 * BSLOT;
    const uint8_t* const b1 = smemB + sb1 * BSLOT;
    const int sbp = sb0 == 0 ? NSB - 1 : sb0 - 1;    // slot of k-step s - 1: free
#pragma unroll
    for (int st = 0; st < NSTG; st++) {
      if (st == NSTG - 1) {
        // grad_Z tile s + 1 and the packed blocks of s + 2 have arrived (the newest grad_Z tile may be in flight) ...
        if (NSB > 2 && s + NSB - 1 < nloc) wait_vmcnt<LB>();
        else wait_vmcnt<0>();
        __syncthreads();               // ... everybody's, S(W) tile s + 1 is written and the slots of s have been read
        stage(st, 0, a1, b1, 0, NU0, s + 2 < nloc, a0, LATE, s + 3 < nloc, gstep(s + 3), s + NSB < nloc, gstep(s + NSB), sb0);
      } else if (st == 0) {
        stage(st, 1, a0, b0, NU0, NU - NU0, s + 1 < nloc, a1, !LATE, s + 2 < nloc, gstep(s + 2), s + NSB - 1 < nloc, gstep(s + NSB - 1), sbp);
      } else {
        stage(st, st + 1, a0, b0, 0, 0, false, nullptr, false, false, 0, false, 0, 0);
      }
    }
    sb0 = sb1;
    sb1 = sb1 == NSB - 1 ? 0 : sb1 + 1;
  }

  __syncthreads();
  if (KG > 1) {
    // sums of the k-groups: groups 1 .. KG - 1 leave theirs in LDS, lane for lane
    if (kg > 0) {
#pragma unroll
      for (int m = 0; m < MT; m++)
#pragma unroll
        for (int t = 0; t < NT; t++)
#pragma unroll
          for (int g = 0; g < 4; g++)
            *(float4*)(smem + (((kg - 1) * NWG + wave) * MT * NT + m * NT + t) * 4096 + g * 1024 + lane * 16) =
                make_float4(acc[m][t][4 * g], acc[m][t][4 * g + 1], acc[m][t][4 * g + 2], acc[m][t][4 * g + 3]);
    }
    __syncthreads();
    if (kg == 0) {
#pragma unroll
      for (int k = 0; k < KG - 1; k++)
#pragma unroll
        for (int m = 0; m < MT; m++)
#pragma unroll
          for (int t = 0; t < NT; t++)
#pragma unroll
            for (int g = 0; g < 4; g++) {
              const float4 v = *(const float4*)(smem + ((k * NWG + wave) * MT * NT + m * NT + t) * 4096 + g * 1024 + lane * 16);
              acc[m][t][4 * g] += v.x;
              acc[m][t][4 * g + 1] += v.y;
              acc[m][t][4 * g + 2] += v.z;
              acc[m][t][4 * g + 3] += v.w;
            }
    }
    __syncthreads();
    if (kg > 0) return;
  }
  dgrad_store<WM, WN, MT, NT>(smem, a, acc, wave, lane, i0, t0);
}

// ---------------------------------------------------------------------------------------------------------
// bf16, large problems: 256 features x 64 NT tokens by 8 waves (4 x 2), each 64 features x 32 NT tokens.  The waves decode the
// packed weight straight into their operand registers (each block by the two waves that share its features).  Three slots per
// operand in LDS; the packed tile of a k-step has to be there half a k-step before its grad_Z tile, because the fragments of a
// half k-step (32 channels) are decoded during the half before it.  The one barrier of a k-step stands before its last quarter:
// behind it the slots of this k-step are free.
// 5120 x 5120 weights at 16384 tokens: 694 us (start: 716, dense vendor GEMM 623); with an all-zero gradient 553 (676, 495): the
// chip lowers its clock under this load.  The 12 % that stay with a zero gradient are the decode, one matrix instruction in eight beside
// the product's.
template <int NT>
constexpr int dgrad_direct_smem() {
  constexpr int RING = 3 * (16 * 1024 + 2048 + 64 * NT * 128);
  constexpr int EPI = 64 * NT * 512;
  return RING > EPI ? RING : EPI;
}

template <int NT>
__device__ __forceinline__ void dgrad_direct_tile(uint8_t* smem, const DgradArgs& a, int tm, int64_t t0) {
  constexpr int WN = 2, MT = 2;
  constexpr int EB = 2, KC = 64, RBK = KC / 16, MBLK = 128;
  constexpr int FST = 4;                            // packed column steps of the tile's 256 features
  constexpr int BN = 64 * NT;
  constexpr int P_BYTES = 16 * 1024, PSLOT = P_BYTES + 16 * MBLK, BSLOT = BN * 128;
  constexpr int LP = 2, LM = 1, LB = BN / 64;       // loads per wave and k-step: packed blocks, position bits, grad_Z
  constexpr int NM = 2 * NT;                        // MFMAs per quarter k-step (16 channels)

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / WN, wn = wave % WN;
  const int n = lane & 31, hh = lane >> 5;
  const int nsteps = (int)((a.O + KC - 1) / KC);
  const int64_t rbn = (a.O + 15) / 16;
  const int64_t i0 = (int64_t)tm * 256;
  uint8_t* const smemP = smem;
  uint8_t* const smemB = smem + 3 * PSLOT;
  const uint32_t ldsP = (uint32_t)(uintptr_t)(lds_u8*)smemP, ldsB = (uint32_t)(uintptr_t)(lds_u8*)smemB;

  const int rows_b = (int)((a.T - t0) < BN ? (a.T - t0) : BN);
  const i32x4 bb = rsrc_words(a.dY + t0 * a.lddy_bytes, (uint32_t)((rows_b - 1) * a.lddy_bytes + a.O * EB));
  const i32x4 bp = rsrc_words(a.vals, (uint32_t)(rbn * a.isteps * 1024)), bm = rsrc_words(a.meta, (uint32_t)(rbn * a.isteps * MBLK));
  const int row_bytes = (int)a.O * EB;
  constexpr uint32_t DEAD = 0x80000000u;            // offset past every descriptor: zeros arrive
  uint32_t offb[LB], offp[LP], offm[LM];
#pragma unroll
  for (int i = 0; i < LB; i++) {
    const int r = 8 * (LB * wave + i) + (lane >> 3);
    offb[i] = (uint32_t)(r * a.lddy_bytes + dy_piece(lane, LB * wave + i));
  }
#pragma unroll
  for (int i = 0; i < LP; i++) {
    const int bl = LP * wave + i, cs = FST * tm + bl % FST;
    offp[i] = cs < a.isteps ? (uint32_t)((bl / FST) * a.isteps + cs) * 1024u + lane * 16u : DEAD;
  }
#pragma unroll
  for (int i = 0; i < LM; i++) {
    const int d = 64 * (LM * wave + i) + lane, bl = d / (MBLK / 4), cs = FST * tm + bl % FST;
    offm[i] = cs < a.isteps ? (uint32_t)((bl / FST) * a.isteps + cs) * (uint32_t)MBLK + 4u * (d % (MBLK / 4)) : DEAD;
  }
  const int rb_w = LP * wave / FST;                 // packed row block of this wave's loads inside the k-step (the same for all)
  auto load_p = [&](int step, int slot) {
    const bool live = RBK * step + rb_w < (int)rbn;
    const uint32_t sv = (uint32_t)step * (uint32_t)(RBK * a.isteps);
#pragma unroll
    for (int i = 0; i < LP; i++) dma_b128(bp, ldsP + (uint32_t)(slot * PSLOT + (LP * wave + i) * 1024), offp[i], live ? sv * 1024u : DEAD);
#pragma unroll
    for (int i = 0; i < LM; i++)
      dma_b32(bm, ldsP + (uint32_t)(slot * PSLOT + P_BYTES + (LM * wave + i) * 256), offm[i], live ? sv * (uint32_t)MBLK : DEAD);
  };
  auto load_b = [&](int step, int slot) {
#pragma unroll
    for (int i = 0; i < LB; i++)
      dma_b128(bb, ldsB + (uint32_t)(slot * BSLOT + (LB * wave + i) * 1024), dy_offset(offb[i], dy_piece(lane, LB * wave + i), row_bytes - 128 * step),
               (uint32_t)step * 128u);
  };

  // expansion: the lane's slot of the packed blocks and the identity operand
  const int rho = 16 * ((n >> 2) & 1) + 4 * (n >> 3) + (n & 3);
  const uint32_t sl_blk = (uint32_t)((rho >> 4) * FST + wm), sl_slot = (uint32_t)(16 * hh + (rho & 15));
  const uint32_t pv_off = sl_blk * 1024u + sl_slot * 16u, pm_off = (uint32_t)P_BYTES + sl_blk * (uint32_t)MBLK + sl_slot * (uint32_t)(MBLK / 64);
  i32x8 ident;                                      // elements 0..7 of lane (n, hh) are k = 8 hh + e, 8..15 k = 16 + 8 hh + e
#pragma unroll
  for (int d = 0; d < 8; d++) {
    const int rel = n - (d < 4 ? 8 * hh : 16 + 8 * hh) - 2 * (d & 3);
    ident[d] = rel == 0 ? 0x3F80 : (rel == 1 ? 0x3F800000 : 0);
  }
  // unit v (0, 1) of a half k-step: feature block v of channel block `half`
  i32x4 pk;
  int pm;
  f32x16 ex;
  int fa[2][MT][8];                                 // A fragments of the current / next half k-step
  auto unit_read = [&](int v, int half, const uint8_t* slot) {
    pk = *(const i32x4*)(slot + pv_off + half * 2 * FST * 1024 + v * 512);
    pm = *(const uint16_t*)(slot + pm_off + half * 2 * FST * MBLK + v * 64);
  };
  auto unit_mma = [&]() {
    zero16(ex);
    bf16x8 av;
    bf16x16 bv;
    __builtin_memcpy(&av, &pk, 16);
    __builtin_memcpy(&bv, &ident, 32);
    ex = __builtin_amdgcn_smfmac_f32_32x32x32_bf16(av, bv, ex, pm, 0, 0);
  };
  auto unit_cvt = [&](int v, int half) {
#pragma unroll
    for (int d = 0; d < 8; d++) fa[half][v][d] = (int)bf16_rne_pack(ex[2 * d], ex[2 * d + 1]);
  };

  f32x16 acc[MT][NT];
#pragma unroll
  for (int m = 0; m < MT; m++)
#pragma unroll
    for (int t = 0; t < NT; t++)
#pragma unroll
      for (int r = 0; r < 16; r++) acc[m][t][r] = 0.f;

  // grad_Z fragments of quarter qt (channels 16 hh + 8 (qt % 2) .. of channel block qt / 2): piece 4 (qt / 2) + 2 hh + qt % 2
  uint4 fb[2][NT];
  const uint32_t fr = (uint32_t)((wn * NT * 32 + n) * 128 + (((2 * hh) ^ ((n >> 1) & 7)) * 16));
  auto read_b = [&](int qt, int t, const uint8_t* sb) {
    fb[qt & 1][t] = *(const uint4*)(sb + (fr ^ (uint32_t)(16 * (4 * (qt >> 1) + (qt & 1)))) + t * 4096);
  };
  auto mma = [&](int qt, int k) {
    const int m = k % MT, t = k / MT;
    bf16x8 av, bv;
    __builtin_memcpy(&av, &fa[qt >> 1][m][4 * (qt & 1)], 16);
    __builtin_memcpy(&bv, &fb[qt & 1][t], 16);
    acc[m][t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av, bv, acc[m][t], 0, 0, 0);
  };

  // prologue
  if (nsteps > 0) {
    load_p(0, 0);
    load_b(0, 0);
    load_p(1, 1);
    load_b(1, 1);
    load_p(2, 2);
    load_b(2, 2);
    wait_vmcnt<2 * LB + LP + LM>();      // P0, B0, P1
    __syncthreads();
#pragma unroll
    for (int v = 0; v < 2; v++) {
      unit_read(v, 0, smemP);
      unit_mma();
      unit_cvt(v, 0);
    }
#pragma unroll
    for (int t = 0; t < NT; t++) read_b(0, t, smemB);
    unit_read(0, 1, smemP);
  }

  int s0 = 0, s1 = 1, s2 = 2;
  for (int s = 0; s < nsteps; s++) {
    const uint8_t* const p0 = smemP + s0 * PSLOT;
    const uint8_t* const p1 = smemP + s1 * PSLOT;
    const uint8_t* const b0 = smemB + s0 * BSLOT;
    const uint8_t* const b1 = smemB + s1 * BSLOT;
#pragma unroll
    for (int qt = 0; qt < 4; qt++) {
      const int half = qt >> 1;
      if (qt == 3) {
        wait_vmcnt<LB>();                // grad_Z tile s + 1 and the packed blocks of s + 2 have landed (grad_Z s + 2 may be in flight)
        __syncthreads();
      }
#pragma unroll
      for (int k = 0; k < NM; k++) {
        const int i = (qt & 1) * NM + k;             // MFMA number inside the half k-step
        // fragments of the next quarter
#pragma unroll
        for (int t = 0; t < NT; t++)
          if (t == k) read_b((qt + 1) & 3, t, qt == 3 ? b1 : b0);
        // decoding of the next half k-step: (s, 1) during half 0, (s + 1, 0) during half 1
        if (i % NM == 0) unit_mma();
        __builtin_amdgcn_sched_barrier(0);
        mma(qt, k);
        __builtin_amdgcn_sched_barrier(0);
        if (qt == 3 && k == 0) {
          load_p(s + 3, s0);
          load_b(s + 3, s0);
        }
        if (i == 0) unit_read(1, 1 - half, half == 0 ? p0 : p1);        // packed slots of the unit after this one
        if (i == NM) unit_read(0, half, p1);
        if (i % NM == NM - 1) unit_cvt(qt & 1, 1 - half);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    const int t_ = s0;
    s0 = s1;
    s1 = s2;
    s2 = t_;
  }
  wait_vmcnt<0>();
  __syncthreads();
  dgrad_store<4, WN, MT, NT>(smem, a, acc, wave, lane, i0, t0);
}

// ---------------------------------------------------------------------------------------------------------
// 8-bit operands, large problems: features [256 tm, 256 tm + 256) x tokens [t0, t0 + 64 NI_) by 8 waves (2 x 4).
// v_mfma_f32_16x16x128_f8f6f4, one per 16 x 16 tile and k-step of 128 channels.  Each wave loads two 1 KiB blocks of packed values
// plus their position bits into registers, expands every group with one byte permute and writes dense rows [channel][feature]
// into a three-slot LDS ring: 256-byte rows, 16-byte chunk c of row r at position c ^ x_swizzle(r) (common.h); the contraction
// index is strided there, so the fragments are read with ds_read_b64_tr_b8.
// Pipeline per k-step s: wait for everything issued during s - 1 (grad_Z tile s + 1 in LDS, packed blocks s + 2 in registers),
// barrier, expansion of blocks s + 2 into LDS (256 x 256: at once, no registers to spare; 256 x 128: spread over the MFMA groups),
// then eight groups of MFMAs during which the grad_Z fragments of s + 1 are read (register double buffer), the S(W) fragments
// roll ahead, the grad_Z tile s + 2 is requested and the packed blocks s + 3 are loaded.
template <int NI_>
constexpr int dgrad8_smem() {
  return 3 * 128 * 256 + 2 * 64 * NI_ * 128;
}

template <int NI_, bool BF8>
__device__ __forceinline__ void dgrad8_tile(uint8_t* smem, const DgradArgs& a, int tm, int64_t t0) {
  constexpr int WN = 4, NW = 8, MI_ = 8;
  constexpr int KC = 128;                           // channels per k-step (128 bytes of a grad_Z row)
  constexpr int RBK = KC / 16;                      // packed row blocks per k-step
  constexpr int CST = 2;                            // packed column steps per 256 features
  constexpr int MBLK = 256;                         // metadata bytes per packed block
  constexpr int BM = 256, BN = 64 * NI_;            // features x tokens per workgroup (256 x 256 or 256 x 128)
  constexpr int AROW = BM;                          // bytes of one channel row of the decoded tile
  constexpr int ASLOT = KC * AROW;                  // decoded S(W): KC channels x 256 features
  constexpr int BSLOT = BN * 128;                   // grad_Z: BN tokens x KC channels
  constexpr int NRA = 3, NRB = 2;
  constexpr int LB = BSLOT / 1024 / NW;             // direct-to-LDS loads per wave and k-step: 4 / 2
  constexpr int EROW = 32 * MI_ + 16;
  constexpr int NPIECE = 2 * NI_;
  static_assert(NRA * ASLOT + NRB * BSLOT == dgrad8_smem<NI_>(), "LDS size");
  static_assert(NRA * ASLOT + NRB * BSLOT <= 160 * 1024 && NW * 16 * NI_ * EROW <= NRA * ASLOT + NRB * BSLOT, "LDS budget");
  uint8_t* const smemA = smem;
  uint8_t* const smemB = smem + NRA * ASLOT;

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / WN, wn = wave % WN;
  const int j = lane & 15, q = lane >> 4;
  const int64_t i0 = (int64_t)tm * BM;
  const int nsteps = (int)((a.O + KC - 1) / KC);
  const int64_t rbn = (a.O + 15) / 16;
  const int isteps = a.isteps;
  const float scale = a.scale;

  // grad_Z tile: exactly the valid rows and channels; what lies outside reads as zeros
  const int rows_b = (int)((a.T - t0) < BN ? (a.T - t0) : BN);
  const i32x4 bb = rsrc_words(a.dY + t0 * a.lddy_bytes, (uint32_t)((rows_b - 1) * a.lddy_bytes + a.O));
  const int row_bytes = (int)a.O;
  uint32_t offb[LB];
#pragma unroll
  for (int i = 0; i < LB; i++) {
    int wl = LB * wave + i;
    int r = 8 * wl + (lane >> 3);
    offb[i] = (uint32_t)(r * a.lddy_bytes + dy_piece(lane, wl));
  }
  const uint32_t ldsB = (uint32_t)(uintptr_t)(lds_u8*)smemB;

  // packed S(W): this wave's two blocks of a k-step are (row block RBK s + rbl, column step CST tm + csl)
  const BufferRsrc rv = make_rsrc(a.vals, (uint32_t)(rbn * isteps * 1024));
  const BufferRsrc rm = make_rsrc(a.meta, (uint32_t)(rbn * isteps * MBLK));
  uint32_t pv_off[2], pm_off[2], dec_off[2];
#pragma unroll
  for (int e = 0; e < 2; e++) {
    const int blkid = 2 * wave + e, rbl = blkid / CST, csl = blkid % CST;
    const int cs = CST * tm + csl;
    const bool live = cs < isteps;                  // column steps past the last feature: nothing to fetch
    pv_off[e] = live ? (uint32_t)((rbl * isteps + cs) * 1024 + lane * 16) : 0x80000000u;
    pm_off[e] = live ? (uint32_t)((rbl * isteps + cs) * MBLK + lane * (MBLK / 64)) : 0x80000000u;
    // the lane's 32 dense bytes: two 16-byte chunks (second at ^ 16)
    const int row = 16 * rbl + j, p = 8 * csl + 2 * q;
    dec_off[e] = (uint32_t)(row * AROW + ((p ^ x_swizzle<true>(row)) * 16));
  }
  uint4 pk[2], pk2[2];                // packed blocks in flight / being expanded (second set: 256 x 128 tile only)
  uint32_t pmeta[2], pmeta2[2];
  uint32_t dec[8];                    // one block row being expanded: 16 dense bf16
#define DG_LOAD_PACKED(step, PK, PM)                                                                            \
  do {                                                                                                    \
    const uint32_t sv_ = (uint32_t)(step) * (uint32_t)RBK * (uint32_t)isteps * 1024u;                     \
    const uint32_t sm_ = (uint32_t)(step) * (uint32_t)RBK * (uint32_t)isteps * (uint32_t)MBLK;            \
    _Pragma("unroll") for (int e = 0; e < 2; e++) {                                                       \
      /* row blocks past the last one (tail of the channel axis, k-steps past the end) fetch nothing */    \
      const bool live_ = RBK * (int64_t)(step) + ((2 * wave + e) / CST) < rbn;                            \
      PK[e] = buffer_load_b128(rv, live_ ? pv_off[e] : 0x80000000u, live_ ? sv_ : 0u);                    \
      PM[e] = (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(rm, (int)(live_ ? pm_off[e] : 0x80000000u),  \
                                                             (int)(live_ ? sm_ : 0u), 0);                 \
    }                                                                                                     \
  } while (0)
// expansion of quarter g of block e (two groups: eight dense bytes) into the staging registers; after the fourth quarter the 32 bytes are written
#define DG_DECODE_PIECE(slot_, e, g, PK, PM)                                                                    \
  do {                                                                                                    \
    const uint32_t w_ = (g) == 0 ? PK[e].x : (g) == 1 ? PK[e].y : (g) == 2 ? PK[e].z : PK[e].w;           \
    dec[2 * (g)] = expand_group8(w_, 0u, (PM[e] >> (8 * (g))) & 15u);                                     \
    dec[2 * (g) + 1] = expand_group8(w_, 2u, (PM[e] >> (8 * (g) + 4)) & 15u);                             \
    if ((g) == 3) {                                                                                       \
      uint8_t* dst_ = smemA + (slot_) * ASLOT + dec_off[e];                                               \
      uint8_t* dst2_ = smemA + (slot_) * ASLOT + (dec_off[e] ^ 16u);                                      \
      *(uint4*)dst_ = make_uint4(dec[0], dec[1], dec[2], dec[3]);                                         \
      *(uint4*)dst2_ = make_uint4(dec[4], dec[5], dec[6], dec[7]);                                        \
    }                                                                                                     \
  } while (0)
#define DG_DECODE(slot_, PK, PM)                                                                             \
  do {                                                                                                    \
    _Pragma("unroll") for (int d_ = 0; d_ < 8; d_++) DG_DECODE_PIECE(slot_, d_ >> 2, d_ & 3, PK, PM);     \
  } while (0)
#define DG_DMA_B(i, step, slot_)                                                                          \
  dma_b128(bb, ldsB + (uint32_t)(slot_) * BSLOT + (LB * wave + (i)) * 1024,                               \
           dy_offset(offb[i], dy_piece(lane, LB * wave + (i)), row_bytes - 128 * (int)(step)), (uint32_t)(step) * 128u)

  f32x4 acc[MI_][NI_];
#pragma unroll
  for (int a = 0; a < MI_; a++)
#pragma unroll
    for (int b = 0; b < NI_; b++) acc[a][b] = (f32x4){0.f, 0.f, 0.f, 0.f};

  // fragment addresses.  S(W): transposing reads, piece r covers channels 16q + 8 (r & 1) + 64 (r >> 1) .. + 7 of the 16
  // features of chunk 8 wm + mi; mi enters through the XOR below (it only touches the low three bits of the position).
  uint32_t fa_off[4];
#pragma unroll
  for (int r = 0; r < 4; r++) {
    const int row = 16 * q + 8 * (r & 1) + 64 * (r >> 1) + (j >> 1);
    fa_off[r] = (uint32_t)(row * AROW + (((8 * wm) ^ x_swizzle<true>(row)) * 16) + 8 * (j & 1));
  }
  const int rb0 = 16 * NI_ * wn + j;
  const int cb0 = q ^ ((j >> 1) & 7);
  const uint32_t fb_off0 = (uint32_t)(rb0 * 128 + cb0 * 16);
  const uint32_t fb_off1 = (uint32_t)(rb0 * 128 + (cb0 ^ 4) * 16);

#define DG_READ_A(dst, base, mi_)                                                                         \
  do {                                                                                                    \
    _Pragma("unroll") for (int r = 0; r < 4; r++) {                                                       \
      /* 256 x 256 tile: the offset is made opaque so that the 32 swizzled addresses of a k-step are      */ \
      /* formed where they are used (one XOR each); kept in registers across the loop they spill          */ \
      uint32_t o_ = fa_off[r];                                                                            \
      if (NI_ == 4) asm volatile("" : "+v"(o_));                                                          \
      i32x2 t_ = __builtin_amdgcn_ds_read_tr8_b64_v2i32((lds_i32x2*)((base) + (o_ ^ (uint32_t)((mi_) * 16)))); \
      dst[r] = make_uint2((uint32_t)t_[0], (uint32_t)t_[1]);                                              \
    }                                                                                                     \
  } while (0)

  // prologue: grad_Z tiles 0 and 1 requested, S(W) tiles 0 and 1 decoded, packed blocks of k-step 2 in registers
#pragma unroll
  for (int i = 0; i < LB; i++) DG_DMA_B(i, 0, 0);
#pragma unroll
  for (int i = 0; i < LB; i++) DG_DMA_B(i, 1, 1);
  DG_LOAD_PACKED(0, pk, pmeta);
  DG_DECODE(0, pk, pmeta);
  DG_LOAD_PACKED(1, pk, pmeta);
  DG_DECODE(1, pk, pmeta);
  DG_LOAD_PACKED(2, pk, pmeta);

  uint4 fb0[NI_][2], fb1[NI_][2];     // grad_Z fragments: current / next k-step
  // S(W) fragments roll AD row blocks ahead of their use (two where registers allow: the 256 x 128 tile
  // issues only four MFMAs per group, too few to cover an LDS round trip); block mi lives in fa[mi % AB]
  constexpr int AD = NI_ == 2 ? 2 : 1, AB = 2 * AD;
  uint2 fa[AB][4];
  wait_vmcnt<0>();
  __syncthreads();
#pragma unroll
  for (int ni = 0; ni < NI_; ni++) {
    fb0[ni][0] = *(const uint4*)(smemB + fb_off0 + ni * 2048);
    fb0[ni][1] = *(const uint4*)(smemB + fb_off1 + ni * 2048);
  }
#pragma unroll
  for (int b = 0; b < AD; b++) DG_READ_A(fa[b], smemA, b);

  int a0 = 0, a1 = 1, a2 = 2;         // S(W) ring slots of k-steps step, step + 1, step + 2
  int b1 = 1;                         // grad_Z ring slot of k-step step + 1 (step + 2 goes to the other one)

#define DG_STEP(BC, BX, PKC, PMC, PKN, PMN)                                                                                 \
  do {                                                                                                    \
    wait_vmcnt<0>();                  /* everything issued during the previous k-step has arrived */      \
    __syncthreads();                  /* ... for every wave; S(W) slot a2 and grad_Z slot 1 - b1 are free */ \
    /* the 256 x 256 tile has no registers to spare for an expansion in flight across the MFMA groups */ \
    if (NI_ == 4) DG_DECODE(a2, PKC, PMC);                                                                \
    const uint8_t* pa = smemA + a0 * ASLOT;                                                               \
    const uint8_t* pa1 = smemA + a1 * ASLOT;                                                              \
    const uint8_t* pb1 = smemB + b1 * BSLOT;                                                              \
    _Pragma("unroll") for (int mi = 0; mi < MI_; mi++) {                                                  \
      if (NI_ != 4) DG_DECODE_PIECE(a2, mi >> 2, mi & 3, PKC, PMC);   /* blocks of k-step step + 2 -> dense, a group per MFMA group */ \
      /* next packed blocks: into the second register set at once (256 x 128), or into the same one    */ \
      /* at the end of the k-step (256 x 256: a load in flight across the groups would spill)           */ \
      if (NI_ != 4 && mi == 0) DG_LOAD_PACKED(step + 3, PKN, PMN);                                        \
      if (NI_ == 4 && mi == MI_ - 1) DG_LOAD_PACKED(step + 3, PKC, PMC);                                  \
      if (mi + AD < MI_) DG_READ_A(fa[(mi + AD) & (AB - 1)], pa, mi + AD);                                \
      else DG_READ_A(fa[(mi + AD) & (AB - 1)], pa1, mi + AD - MI_);                                       \
      _Pragma("unroll") for (int pc = 0; pc < NPIECE; pc++)                                               \
        if (spread(pc, NPIECE, MI_) == mi)                                                                \
          BX[pc >> 1][pc & 1] = *(const uint4*)(pb1 + ((pc & 1) ? fb_off1 : fb_off0) + (pc >> 1) * 2048); \
      _Pragma("unroll") for (int n = 0; n < LB; n++)                                                      \
        if (n == mi) DG_DMA_B(n, step + 2, 1 - b1);                                                       \
      _Pragma("unroll") for (int ni = 0; ni < NI_; ni++) {                                                \
        /* one 128-channel instruction; byte e of both operands is the same channel (16q + e, then        */ \
        /* 64 + 16q + e - 16), zero scale arguments select the unscaled form                              */ \
        i32x8 av, bv;                                                                                     \
        __builtin_memcpy(&av, &fa[mi & (AB - 1)][0], 32);                                                 \
        __builtin_memcpy(&bv, &BC[ni][0], 32);                                                            \
        /* format arguments: A (expanded weight) e4m3; B (grad_Z) e4m3, or e5m2 when BF8                  */ \
        acc[mi][ni] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(av, bv, acc[mi][ni], 0, BF8 ? 1 : 0, 0, 0, 0, 0); \
      }                                                                                                   \
      __builtin_amdgcn_sched_barrier(0);                                                                  \
    }                                                                                                     \
    const int t_ = a0;                                                                                    \
    a0 = a1;                                                                                              \
    a1 = a2;                                                                                              \
    a2 = t_;                                                                                              \
    b1 = 1 - b1;                                                                                          \
  } while (0)

  int step = 0;
  for (; step + 1 < nsteps; step += 2) {
    if (NI_ == 4) {
      DG_STEP(fb0, fb1, pk, pmeta, pk, pmeta);
      step++;
      DG_STEP(fb1, fb0, pk, pmeta, pk, pmeta);
      step--;
    } else {
      DG_STEP(fb0, fb1, pk, pmeta, pk2, pmeta2);
      step++;
      DG_STEP(fb1, fb0, pk2, pmeta2, pk, pmeta);
      step--;
    }
  }
  if (step < nsteps) {
    if (NI_ == 4) DG_STEP(fb0, fb1, pk, pmeta, pk, pmeta);
    else DG_STEP(fb0, fb1, pk, pmeta, pk2, pmeta2);
  }
#undef DG_STEP
#undef DG_READ_A
#undef DG_DMA_B
#undef DG_DECODE
#undef DG_DECODE_PIECE
#undef DG_LOAD_PACKED

  // epilogue: accumulators -> LDS (row = token, the wave's 128 features contiguous) -> 16-byte stores
  wait_vmcnt<0>();
  __syncthreads();
  uint8_t* eb = smem + wave * (16 * NI_ * EROW);
#pragma unroll
  for (int mi = 0; mi < MI_; mi++)
#pragma unroll
    for (int ni = 0; ni < NI_; ni++) {
      uint2 v;
      v.x = bf16_rne_pack(acc[mi][ni][0] * scale, acc[mi][ni][1] * scale);
      v.y = bf16_rne_pack(acc[mi][ni][2] * scale, acc[mi][ni][3] * scale);
      *(uint2*)(eb + (16 * ni + j) * EROW + (16 * mi + 4 * q) * 2) = v;
    }
  constexpr int CHUNKS = 2 * MI_, NCH = 16 * NI_ * CHUNKS;
  static_assert(NCH % 64 == 0, "whole rounds of lanes");
  if (a.H) {
    dgrad_store_act<NCH / 64>(a, t0 + 16 * NI_ * wn, i0 + 16 * MI_ * wm, 16 * NI_, CHUNKS, lane,
                              [&](int row, int chunk) { return *(const uint4*)(eb + row * EROW + chunk * 16); });
    return;
  }
#pragma unroll
  for (int it = 0; it < NCH / 64; it++) {
    const int c = 64 * it + lane, row = c / CHUNKS, chunk = c % CHUNKS;
    const uint4 v = *(const uint4*)(eb + row * EROW + chunk * 16);
    const int64_t t = t0 + 16 * NI_ * wn + row, i = i0 + 16 * MI_ * wm + 8 * chunk;
    if (t < a.T && i < a.I) store_stream_b128(a.dX + t * a.lddx + i, v);
  }
}

// ---------------------------------------------------------------------------------------------------------
// kernels: one tile shape for the whole grid, or whole rounds of 256 x 256 tiles (workgroups 0 .. n_big - 1) followed by the tiles of
// the last, partial round as twice as many 256 x 128 tiles, so that the round takes half a tile time on twice the CUs
template <bool FP8, bool BF8, int WM, int WN, int MT, int NT, int KG, int NSB>
__global__ void __launch_bounds__(64 * WM * WN * KG, 1)
k_linear_dgrad(DgradArgs a, int m_tiles) {
  __shared__ __align__(1024) uint8_t smem[dgrad_smem<WM, WN, MT, NT, KG, NSB>()];
  const int logical = xcd_contiguous(blockIdx.x, gridDim.x);
  dgrad_tile<FP8, BF8, WM, WN, MT, NT, KG, NSB>(smem, a, (int64_t)(logical % m_tiles) * (32 * WM * MT), (int64_t)(logical / m_tiles) * (32 * WN * NT));
}

// NI: tokens / 64 of the tile
template <bool FP8, bool BF8, int NI>
constexpr int dgrad_large_smem() {
  return FP8 ? dgrad8_smem<NI>() : dgrad_direct_smem<NI>();
}
template <bool FP8, bool BF8, int NI>
__device__ __forceinline__ void dgrad_large_tile(uint8_t* smem, const DgradArgs& a, int tm, int64_t t0) {
  if constexpr (FP8) dgrad8_tile<NI, BF8>(smem, a, tm, t0);
  else dgrad_direct_tile<NI>(smem, a, tm, t0);
}

template <bool FP8, bool BF8, int NI>
__global__ void __launch_bounds__(512, 1)
k_linear_dgrad_large(DgradArgs a, int m_tiles) {
  __shared__ __align__(1024) uint8_t smem[dgrad_large_smem<FP8, BF8, NI>()];
  const int logical = xcd_contiguous(blockIdx.x, gridDim.x);
  dgrad_large_tile<FP8, BF8, NI>(smem, a, logical % m_tiles, (int64_t)(logical / m_tiles) * (64 * NI));
}

template <bool FP8, bool BF8>
__global__ void __launch_bounds__(512, 1)
k_linear_dgrad_dual(DgradArgs a, int m_tiles, int n_big) {
  __shared__ __align__(1024) uint8_t smem[dgrad_large_smem<FP8, BF8, 4>()];
  const int bid = blockIdx.x;
  if (bid < n_big) {
    const int logical = xcd_contiguous(bid, n_big);
    dgrad_large_tile<FP8, BF8, 4>(smem, a, logical % m_tiles, (int64_t)(logical / m_tiles) * 256);
  } else {
    const int h = xcd_contiguous(bid - n_big, (int)gridDim.x - n_big);      // half-tile number
    const int tile = n_big + (h >> 1);
    const int64_t t0 = (int64_t)(tile / m_tiles) * 256 + 128 * (h & 1);
    if (t0 >= a.T) return;                     // second half of a ragged last token tile: nothing to do
    dgrad_large_tile<FP8, BF8, 2>(smem, a, tile % m_tiles, t0);
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
// Choice of the tile.  Time model in microseconds: a workgroup costs F + nk * step, nk = its k-steps (each k-group of a workgroup takes
// a KG-th of them) and step = max(lat, r * thr) with r workgroups sharing a CU: lat is the time one k-step's loads, barrier and
// MFMAs take end to end, thr what a CU needs per workgroup and k-step when its pipes are shared; R workgroups fit a CU (LDS), and what
// does not fit runs in further rounds.  Fitted to event times of 160 random problems (64 ... 32768 tokens, 64 ... 5120 channels and
// features) for every shape: 5...10 % off per problem, and the shape it picks is 1 % (bf16) / 2 % (8-bit) slower than the best one on
// the geometric mean, 10 / 16 % at worst.
struct DgradShape {
  int bm, bn, kg, r, threads;
  double f, lat, thr, base;
};
enum { DG_256, DG_256x128, DG_128_KG1, DG_128_KG2, DG_64_KG1, DG_64_KG2, DG_64_KG4, DG_SHAPES, DG_DUAL = DG_SHAPES };
static const DgradShape kDgrad16[DG_SHAPES] = {
  {256, 256, 1, 1, 512, 6.24, 1.34, 0.00, 0.0},
  {256, 128, 1, 1, 512, 4.71, 0.825, 0.00, 0.0},
  {128, 128, 1, 2, 256, 2.61, 0.818, 0.627, 1.7},
  {128, 128, 2, 1, 512, 3.26, 1.17, 0.00, 0.8},
  {64, 64, 1, 3, 256, 0.77, 0.427, 0.248, 2.9},
  {64, 64, 2, 2, 512, 1.52, 0.548, 0.446, 2.1},
  {64, 64, 4, 1, 1024, 2.30, 0.927, 0.00, 1.5},
};
static const DgradShape kDgrad8[DG_SHAPES] = {
  {256, 256, 1, 1, 512, 6.19, 1.536, 0.00, 0.0},
  {256, 128, 1, 1, 512, 4.33, 1.036, 0.00, 0.4},
  {128, 128, 1, 2, 256, 2.28, 1.044, 0.774, 1.9},
  {128, 128, 2, 1, 512, 3.13, 1.437, 0.00, 1.2},
  {64, 64, 1, 3, 256, 0.73, 0.524, 0.292, 3.0},
  {64, 64, 2, 2, 512, 1.42, 0.610, 0.543, 2.4},
  {64, 64, 4, 1, 1024, 2.32, 1.098, 0.00, 1.6},
};

static int dgrad_choice(bool fp8, int64_t T, int64_t O, int64_t I) {
  const DgradShape* tab = fp8 ? kDgrad8 : kDgrad16;
  const int64_t steps = (O + (fp8 ? 127 : 63)) / (fp8 ? 128 : 64);
  int best = DG_256;
  double best_t = 1e30;
  for (int c = 0; c < DG_SHAPES; c++) {
    const DgradShape& s = tab[c];
    const int64_t wgs = ((I + s.bm - 1) / s.bm) * ((T + s.bn - 1) / s.bn);
    if (c != DG_256 && wgs > 0x7FFFFFFFll) continue;                                  // grid size
    const double nk = (double)((steps + s.kg - 1) / s.kg);
    const int64_t n = (wgs + 255) / 256, full = n / s.r, rem = n % s.r;      // workgroups on the busiest CU: full rounds of r, and a rest
    double t = s.base + (double)full * (s.f + nk * (s.lat > s.r * s.thr ? s.lat : s.r * s.thr));
    if (rem) t += s.f + nk * (s.lat > rem * s.thr ? s.lat : rem * s.thr);
    if (t < best_t) {
      best_t = t;
      best = c;
    }
    // 256 x 256 tiles whose last round is at most half full: that round as 256 x 128 tiles
    if (c == DG_256 && wgs > 256 && wgs % 256 != 0 && wgs % 256 <= 128) {
      const double td = (double)(wgs / 256) * (s.f + nk * s.lat) + tab[DG_256x128].f + nk * tab[DG_256x128].lat;
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
  const DgradShape& s = kDgrad16[cfg];
  snprintf(text, n, "%dx%d kg %d r %d grid %lld block %d", s.bm, s.bn, s.kg, s.r, (long long)(((I + s.bm - 1) / s.bm) * ((T + s.bn - 1) / s.bn)), s.threads);
}

template <bool FP8, bool BF8>
static void launch_dgrad_type(const DgradArgs& a, hipStream_t s) {
  const int m256 = (int)((a.I + 255) / 256);
  const int cfg = dgrad_choice(FP8, a.T, a.O, a.I);
#define DG_SMALL(WM, WN, MT, NT, KG, NSB)                                                                                      \
  do {                                                                                                                         \
    const int mt_ = (int)((a.I + 32 * WM * MT - 1) / (32 * WM * MT));                                                          \
    const int64_t nt_ = (a.T + 32 * WN * NT - 1) / (32 * WN * NT);                                                             \
    SSTE_LAUNCH(SSTE_K_DGRAD, (k_linear_dgrad<FP8, BF8, WM, WN, MT, NT, KG, NSB>), dim3((unsigned)(mt_ * nt_)), dim3(64 * WM * WN * KG), s, a, mt_); \
  } while (0)
#define DG_LARGE(NI)                                                                                                           \
  SSTE_LAUNCH(SSTE_K_DGRAD, (k_linear_dgrad_large<FP8, BF8, NI>), dim3((unsigned)(m256 * ((a.T + 64 * NI - 1) / (64 * NI)))), dim3(512), s, a, m256)
  switch (cfg) {
    case DG_DUAL: {
      const int64_t big = (int64_t)m256 * ((a.T + 255) / 256), rem = big % 256;
      SSTE_LAUNCH(SSTE_K_DGRAD, (k_linear_dgrad_dual<FP8, BF8>), dim3((unsigned)(big + rem)), dim3(512), s, a, m256, (int)(big - rem));
      break;
    }
    case DG_256: DG_LARGE(4); break;
    case DG_256x128: DG_LARGE(2); break;
    case DG_128_KG1: DG_SMALL(2, 2, 2, 2, 1, 3); break;
    case DG_128_KG2: DG_SMALL(2, 2, 2, 2, 2, 2); break;
    case DG_64_KG1: DG_SMALL(2, 2, 1, 1, 1, 3); break;
    case DG_64_KG2: DG_SMALL(2, 2, 1, 1, 2, 2); break;
    default: DG_SMALL(2, 2, 1, 1, 4, 2); break;
  }
#undef DG_SMALL
#undef DG_LARGE
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
