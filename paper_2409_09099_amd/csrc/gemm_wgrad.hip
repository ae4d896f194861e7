// Weight-gradient path of the S-STE linear layer (paper Sec. 5.1): grad_W = MVUE(grad_Z^T) X.
//
// Most problems run in two or three kernels on the caller's stream:
//   1. k_mvue_pack: the estimator is applied once per group of four tokens and the result is written
//      to the workspace as a packed 2:4 operand in sparse-MFMA fragment order (the format of
//      include/sste.h with rows = output channels, columns = tokens).  It streams dY once: at about
//      84 vector instructions per group (bf16; 61 for 8-bit types) the bf16 kernel runs at the rate of a
//      plain copy, the 8-bit kernel (twice the groups per byte) is bound by the vector pipe.
//   2. k_wgrad_gemm (large tiles) or k_wgrad_tile (small ones): sparse MFMA GEMM, rows = channels o, columns =
//      input features i, contraction = tokens.  The packed operand is loaded like the packed weight of the
//      forward GEMM; X arrives with the contraction index strided (X is [t][i]) and its fragments are
//      read with the transposing LDS load (ds_read_b64_tr_b16 / _b8).
//   3. where the token axis is split to fill the chip, k_wgrad_reduce: sums the splits in a fixed order
//      (bitwise reproducible) and applies the scale.
// Tile shape and split count are chosen per problem (make_wgrad_plan).  Small tiles fill the chip without a split where large ones
// would need several: 2112 tokens, 1544 x 832, bf16: 14.1 + 4.4 us (256 x 192 tiles, three splits and their sum) -> 12.9 us (128 x 64).
// Why not fuse the estimator into the GEMM's operand load everywhere: a GEMM tile that is N columns
// wide re-derives every group I / N times, and the vector pipe, not the matrix pipe or HBM, sets the time (on the 5120 x 1280 layer
// a 256-wide tile would issue five times the pre-pass's vector work, about 260 us against the 110 us of the whole GEMM).  The fused
// kernel (gemm_wgrad_fused.hip) is kept for small problems, where one launch and no workspace matter more.
#include "common.h"
#include "mvue_device.h"
#include "wgrad_deal.h"

#include <atomic>
#include <mutex>
#include <numeric>
#include <type_traits>

#include <stdio.h>

namespace sste {

hipError_t launch_wgrad_fused(const void* dY, int64_t T, int64_t O, int64_t lddy, int dtype, const void* X, int64_t I, int64_t ldx,
                              RngKey key, float scale, int accumulate, float* dW, int64_t lddw, hipStream_t s);

namespace {
constexpr int NUM_CU = 256;
typedef __attribute__((address_space(3))) bf16x4 lds_bf16x4;
typedef __attribute__((address_space(3))) i32x2 lds_i32x2;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;

}  // namespace

// ---------------------------------------------------------------------------------------------------------
// 1. estimator -> packed operand.  One workgroup: one k-step (64 / 128 tokens) x BC channels.  A lane works on the two groups of eight
// consecutive tokens for VB bytes of channels, so that each of its results is a whole metadata byte and a 4-byte (bf16: 8-byte) piece
// of the packed values.  Measured against one group per lane in four rows of 16 bytes: e5m2 32768 x 5120 83 -> 76 us, e4m3 3200 x 1552
// 8.4 -> 6.6, bf16 16384 x 4096 41.2 -> 40.2.  The 8-bit kernel is bound by its vector instructions: 73 a group -> 61 (counts of the recorded
// positions from sign bits by byte permutes, one comparison and for e4m3 a minimum less, the shared first step of the hash, fixed distances
// in the staging LDS): 32768 x 5120 78 -> 65 us (e4m3), 78 -> 71 (e5m2), 32768 x 3840 59 -> 51, 32768 x 1280 23.4 -> 20.8.
template <bool FP8, int BC, int VB>
constexpr int mvue_threads() { return (FP8 ? 128 : 64) / 8 * BC * (FP8 ? 1 : 2) / VB; }

// LOW: every group id is below 2^32.  Ids that differ in their last bits then share the first step of the hash but for those bits.
template <bool FP8, bool BF8, int BC, int VB, bool LOW>
__global__ void __launch_bounds__((mvue_threads<FP8, BC, VB>()))
k_mvue_pack(const uint8_t* __restrict__ dY, int64_t T, int64_t O, int64_t lddy_bytes, RngKey key,
            uint8_t* __restrict__ vals, uint8_t* __restrict__ meta) {
  constexpr int EB = FP8 ? 1 : 2;
  constexpr int KS = FP8 ? 128 : 64;              // tokens per k-step
  constexpr int NT = mvue_threads<FP8, BC, VB>();
  constexpr int CH = VB / EB, DW = VB / 4;        // channels, dwords per row of a lane
  constexpr int OC = BC / CH;                     // lanes across the channels
  constexpr int PPQ = KS / 32;                    // group pairs per lane quarter of the operand: 2 / 4
  constexpr int MBLK = FP8 ? 256 : 128;           // metadata bytes per block
  // LDS staging in the operand's own order, the blocks of 16 channels padded so that the lanes of a wave, which write the same place of
  // different blocks, are spread over the banks
  constexpr int VPITCH = 1024 + 16, MPITCH = MBLK + (FP8 ? 16 : 32);
  __shared__ __align__(16) uint8_t sV[BC / 16 * VPITCH];
  __shared__ __align__(16) uint8_t sM[BC / 16 * MPITCH];

  const int tid = threadIdx.x;
  const int kp = tid / OC, oc = tid % OC;         // group pair of the k-step, lane across the channels
  const int64_t s = blockIdx.y, steps = T / KS;
  const int64_t o0 = (int64_t)blockIdx.x * BC;
  const int64_t och = o0 + (int64_t)oc * CH;

  uint32_t rdy[8][DW];
#pragma unroll
  for (int r = 0; r < 8; r++)
#pragma unroll
    for (int w = 0; w < DW; w++) rdy[r][w] = 0;
  if (och < O) {
    typedef __attribute__((__vector_size__(VB))) uint32_t row_t;
    const uint8_t* p = dY + (s * KS + 8 * kp) * lddy_bytes + och * EB;
#pragma unroll
    for (int r = 0; r < 8; r++) {
      const row_t t = __builtin_nontemporal_load((const row_t*)(p + r * lddy_bytes));
#pragma unroll
      for (int w = 0; w < DW; w++) rdy[r][w] = t[w];
    }
  }
  // Group ids of this lane: gid_a + e and gid_b + e.  O and och are multiples of CH, so both are too and the
  // CH consecutive ids share their high word (no carry out of the low word inside the piece) and adding e is an exclusive or, which the
  // draw begins with.
  const uint64_t gid_a = (key.first_group + (uint64_t)(s * (KS / 4) + 2 * kp)) * (uint64_t)O + (uint64_t)och, gid_b = gid_a + (uint64_t)O;
  const uint32_t hi_a = (uint32_t)(gid_a >> 32) * 0x9E3779B9u, hi_b = (uint32_t)(gid_b >> 32) * 0x9E3779B9u;
  const uint32_t lo_a = (uint32_t)gid_a ^ key.k0, lo_b = (uint32_t)gid_b ^ key.k0;
  const uint32_t fold_a = lo_a ^ (lo_a >> 17), fold_b = lo_b ^ (lo_b >> 17);
  const int q = kp / PPQ, gp = kp % PPQ;
  // the lane's channels are consecutive rows of one block: its first value and metadata byte, and the rows follow at fixed distances
  static_assert(16 % CH == 0, "channels of a lane inside a block");
  const int blk = oc * CH / 16, row0 = 16 * q + oc * CH % 16;
  uint8_t* const slot0 = sV + blk * VPITCH + row0 * 16 + (FP8 ? 4 : 8) * gp;
  uint8_t* const meta0 = sM + blk * MPITCH + row0 * PPQ + gp;
  // 8-bit: the four token rows' dwords of four channels, transposed 4 x 4 bytes at a time (eight byte permutes
  // for four groups): grp[h][k] holds channel 4 (e / 4) + k with the group's first token in byte 0
  uint32_t grp[2][4] = {};
#pragma unroll
  for (int e = 0; e < CH; e++) {
    const uint32_t xa = LOW ? draw_u32_folded(fold_a ^ (uint32_t)e, key.k1) : draw_u32_mixed((lo_a ^ (uint32_t)e) + hi_a, key.k1);
    const uint32_t xb = LOW ? draw_u32_folded(fold_b ^ (uint32_t)e, key.k1) : draw_u32_mixed((lo_b ^ (uint32_t)e) + hi_b, key.k1);
    uint32_t m;
    if (FP8) {
      if ((e & 3) == 0) {
#pragma unroll
        for (int h = 0; h < 2; h++) {
          const uint32_t w0 = rdy[4 * h][e >> 2], w1 = rdy[4 * h + 1][e >> 2], w2 = rdy[4 * h + 2][e >> 2], w3 = rdy[4 * h + 3][e >> 2];
          const uint32_t a01 = __builtin_amdgcn_perm(w1, w0, 0x05010400u), b01 = __builtin_amdgcn_perm(w1, w0, 0x07030602u);
          const uint32_t a23 = __builtin_amdgcn_perm(w3, w2, 0x05010400u), b23 = __builtin_amdgcn_perm(w3, w2, 0x07030602u);
          grp[h][0] = __builtin_amdgcn_perm(a23, a01, 0x05040100u);
          grp[h][1] = __builtin_amdgcn_perm(a23, a01, 0x07060302u);
          grp[h][2] = __builtin_amdgcn_perm(b23, b01, 0x05040100u);
          grp[h][3] = __builtin_amdgcn_perm(b23, b01, 0x07060302u);
        }
      }
      *(uint32_t*)(slot0 + 16 * e) = mvue_pair_f8<BF8>(grp[0][e & 3], grp[1][e & 3], xa, xb, m);
    } else {
      const uint32_t sel = (e & 1) ? 0x07060302u : 0x05040100u;
      uint2 v;
      uint32_t ma, mb;
      v.x = mvue_group_bf16(__builtin_amdgcn_perm(rdy[1][e >> 1], rdy[0][e >> 1], sel), __builtin_amdgcn_perm(rdy[3][e >> 1], rdy[2][e >> 1], sel), xa, ma);
      v.y = mvue_group_bf16(__builtin_amdgcn_perm(rdy[5][e >> 1], rdy[4][e >> 1], sel), __builtin_amdgcn_perm(rdy[7][e >> 1], rdy[6][e >> 1], sel), xb, mb);
      *(uint2*)(slot0 + 16 * e) = v;
      m = 0xEEu - (ma + (mb << 4));
    }
    meta0[PPQ * e] = (uint8_t)m;
  }
  __syncthreads();

  const int64_t rb0 = o0 / 16, rbn = (O + 15) / 16;
#pragma unroll
  for (int ci = tid; ci < BC * 4; ci += NT) {
    const int rb = ci >> 6, sl = ci & 63;         // block and slot inside the tile
    if (rb0 + rb < rbn) *(uint4*)(vals + ((rb0 + rb) * steps + s) * 1024 + sl * 16) = *(const uint4*)(sV + rb * VPITCH + sl * 16);
  }
#pragma unroll
  for (int ci = tid; ci < BC * MBLK / 256; ci += NT) {
    const int rb = ci / (MBLK / 16), sl = ci % (MBLK / 16);
    if (rb0 + rb < rbn) *(uint4*)(meta + ((rb0 + rb) * steps + s) * MBLK + sl * 16) = *(const uint4*)(sM + rb * MPITCH + sl * 16);
  }
}

static void launch_mvue_pack(const void* dY, int64_t T, int64_t O, int64_t lddy, int dtype, RngKey key, void* vals,
                             void* meta, hipStream_t s, int timed_kind) {
  const bool fp8 = dtype != SSTE_BF16;
  const int ks = fp8 ? 128 : 64;
  // Many short-lived lanes fill the chip on small problems and keep each lane's chain of estimators short; large ones stream better with
  // wider rows per lane.  Crossover at 2^25 elements (narrow against wide, bf16 16384 x 1280: 15.0 / 15.3 us, 16384 x 2048: 21.6 / 20.8, 16384 x 4096:
  // 39.8 / 37.5; e4m3 3200 x 1552: 7.2 / 7.0, 16384 x 1280: 11.9 / 11.4, 16384 x 2048: 17.9 / 16.5, 32768 x 5120: 84.9 / 59.7).  With the 8-bit
  // estimator as short as it is now, 8-bit problems between 2^24 and 2^25 elements are 4 ... 8 % slower for it.
  const bool small = !product_reaches(T, O, 1ll << 25);
  const bool low = (unsigned __int128)(key.first_group + (uint64_t)(T / 4)) * (uint64_t)O <= 0x100000000ull;
#define MP_LAUNCH(F8, B8, BC, VB, LOW)                                                                                   \
  do {                                                                                                                   \
    const dim3 grid((unsigned)((O + BC - 1) / BC), (unsigned)(T / ks)), block(mvue_threads<F8, BC, VB>());               \
    if (timed_kind >= 0)                                                                                                 \
      SSTE_LAUNCH(timed_kind, (k_mvue_pack<F8, B8, BC, VB, LOW>), grid, block, s, (const uint8_t*)dY, T, O, lddy*(F8 ? 1 : 2), key, \
                  (uint8_t*)vals, (uint8_t*)meta);                                                                       \
    else                                                                                                                 \
      hipLaunchKernelGGL((k_mvue_pack<F8, B8, BC, VB, LOW>), grid, block, 0, s, (const uint8_t*)dY, T, O, lddy*(F8 ? 1 : 2), key, \
                         (uint8_t*)vals, (uint8_t*)meta);                                                                \
  } while (0)
#define MP_CASE(F8, B8, BC, VB)                   \
  do {                                            \
    if (low) MP_LAUNCH(F8, B8, BC, VB, true);     \
    else MP_LAUNCH(F8, B8, BC, VB, false);        \
  } while (0)
#define MP_TYPE(BC, VB)                                          \
  do {                                                           \
    if (dtype == SSTE_F8E5M2) MP_CASE(true, true, BC, VB);       \
    else if (fp8) MP_CASE(true, false, BC, VB);                  \
    else MP_CASE(false, false, BC, VB);                          \
  } while (0)
  if (small) MP_TYPE(64, 4);
  else MP_TYPE(128, 8);
#undef MP_TYPE
#undef MP_CASE
#undef MP_LAUNCH
}

hipError_t launch_mvue_materialize(const void* dY, int64_t T, int64_t O, int64_t lddy, int dtype, RngKey key,
                                   void* vals, void* meta, hipStream_t s) {
  if (T == 0 || O == 0) return hipSuccess;
  launch_mvue_pack(dY, T, O, lddy, dtype, key, vals, meta, s, -1);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------------------------------------
// 2. sparse GEMM on the packed operand.  8 waves (2 x 4), each owning MI_ x NI_ MFMA tiles: a workgroup
// covers 32 MI_ channels x 64 NI_ features (256 x 256, 192 x 192, ...) over one split of the token axis.
// Same software pipeline as the forward GEMM: X fragments double-buffered in registers and read one
// k-step ahead, packed fragments rolling one row block ahead, direct-to-LDS loads spread over the MFMA
// groups, separate three-slot rings for the two operands, one barrier per k-step.
// X tile in LDS: one row per token, 512 B (bf16: 256 features) or 256 B (fp8) whatever the tile width;
// narrower tiles leave the tail of each row unused.  32-byte feature pair p (bf16) / 16-byte chunk c
// (fp8) of token row r is stored at position p ^ x_swizzle(r) (common.h), which keeps the transposing
// reads below -- 4 (8) consecutive token rows x 16 features per 16 lanes, the four lane quarters 8 (16)
// rows apart -- off each other's banks.

// The tile order: channel tiles or feature tiles run fastest.
struct WgradTiles {
  int m_tiles, n_tiles, features_fastest;
};

// Splits of the token axis: `groups` tiles, `steps` k-steps to a workgroup.  A type of its own: with the deal's bounds, which a workgroup has to look up
// before its first load, splits of few k-steps cost 3 % more (640 x 1216 x 4864 bf16 18.1 -> 18.7 us).
struct WgradSplits {
  int groups, steps;
};

template <bool FP8, int MI_, int NI_, bool BF8, bool DEALT>
__global__ void __launch_bounds__(512, 1)
k_wgrad_gemm(const uint8_t* __restrict__ vals, const uint8_t* __restrict__ meta, int64_t O, int64_t total_steps,
             const uint8_t* __restrict__ X, int64_t I, int64_t ldx_bytes, std::conditional_t<DEALT, WgradDeal, WgradSplits> deal, float scale,
             int accumulate, float* __restrict__ out, int64_t ld_out, int64_t split_stride, WgradTiles order) {
  constexpr int WN = 4, NW = 8, NR = 3;
  constexpr int BM = 32 * MI_, BN = 64 * NI_;
  constexpr int EB = FP8 ? 1 : 2;
  constexpr int KS = FP8 ? 128 : 64;              // tokens per k-step
  constexpr int MB = FP8 ? 16 : 8, MBLK = 16 * MB;
  constexpr int ROWB = 256 * EB;                  // LDS bytes per token row: 512 / 256
  constexpr int LA = (BM / 16 + NW - 1) / NW;     // packed blocks (1 KiB) per wave and k-step
  constexpr int LM = (BM * MB / 256 + NW - 1) / NW;
  constexpr int BSTAGE = KS * ROWB;               // 32 KiB
  constexpr int LB = BSTAGE / 1024 / NW;          // 4
  constexpr int A_BYTES = NW * LA * 1024, M_BYTES = NW * LM * 256, ASTAGE = A_BYTES + M_BYTES;
  constexpr int NLOAD = LA + LM + LB;             // issue order inside a k-step: A.., M.., B..
  constexpr int NPIECE = 4 * NI_;                 // 8-byte pieces of the next X fragments
  constexpr int RPL = 1024 / ROWB;                // token rows per 1 KiB load: 2 / 4
  constexpr int CPR = ROWB / 16;                  // 16-byte chunks per row: 32 / 16
  __shared__ __align__(1024) uint8_t smem[NR * (ASTAGE + BSTAGE)];
  uint8_t* const smemA = smem;
  uint8_t* const smemB = smem + NR * ASTAGE;

  // XCD x owns a contiguous range of (part, group) pairs, groups fastest
  const int logical = xcd_contiguous(blockIdx.x, gridDim.x);
  const int part = logical / deal.groups, group = logical % deal.groups;

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / WN, wn = wave % WN;
  const int j = lane & 15, q = lane >> 4;
  int at, part_end;
  if constexpr (DEALT) {
    at = deal.bound[part];
    part_end = deal.bound[part + 1];
  } else {
    at = part * deal.steps;
    part_end = total_steps - at < deal.steps ? (int)total_steps : at + deal.steps;
  }
  do {
  // the next segment: k-steps [step_begin, step_begin + nsteps) of one tile
  const int member = DEALT ? at / (int)total_steps : 0, tile = member * deal.groups + group;
  const int64_t step_begin = at - member * (int)total_steps;
  const int nsteps = DEALT && part_end - at > (int)(total_steps - step_begin) ? (int)(total_steps - step_begin) : part_end - at;
  at += nsteps;
  if (DEALT && tile >= order.m_tiles * order.n_tiles) break;      // the last group may have fewer members
  const int tm = order.features_fastest ? tile / order.n_tiles : tile % order.m_tiles;
  const int tn = order.features_fastest ? tile % order.n_tiles : tile / order.m_tiles;
  const int64_t o0 = (int64_t)tm * BM, i0 = (int64_t)tn * BN;

  const int64_t rblk0 = o0 / 16, rbn = (O + 15) / 16;
  const int blks_a = (int)((rbn - rblk0) < BM / 16 ? (rbn - rblk0) : BM / 16);
  const i32x4 ba = rsrc_words(vals + (rblk0 * total_steps + step_begin) * 1024, (uint32_t)((blks_a * total_steps - step_begin) * 1024));
  const i32x4 bm = rsrc_words(meta + (rblk0 * total_steps + step_begin) * MBLK, (uint32_t)((blks_a * total_steps - step_begin) * MBLK));
  const int cols_b = (int)((I - i0) < BN ? (I - i0) : BN);
  const i32x4 bb = rsrc_words(X + step_begin * KS * ldx_bytes + i0 * EB, (uint32_t)(((int64_t)nsteps * KS - 1) * ldx_bytes + cols_b * EB));

  // Packed blocks past the tile's last one must fetch nothing although the descriptor (which runs to
  // the end of the tile's last block row) may still cover their offsets: push them out of range.
  uint32_t offa[LA], offb[LB], offm[LM];
#pragma unroll
  for (int i = 0; i < LA; i++)
    offa[i] = (LA * wave + i) < blks_a ? (uint32_t)((LA * wave + i) * total_steps * 1024 + lane * 16) : 0x80000000u;
#pragma unroll
  for (int i = 0; i < LB; i++) {
    int wl = LB * wave + i;
    int r = RPL * wl + lane / CPR, cs = lane % CPR;          // token row inside the k-step, stored chunk
    int c = FP8 ? (cs ^ x_swizzle<true>(r)) : ((((cs >> 1) ^ x_swizzle<false>(r)) << 1) | (cs & 1));   // source chunk
    // chunks past the last feature column of the tile must read as zeros
    offb[i] = (c * 16 < cols_b * EB) ? (uint32_t)(r * ldx_bytes + c * 16) : 0x80000000u;
  }
#pragma unroll
  for (int i = 0; i < LM; i++) {
    int d = 64 * (LM * wave + i) + lane;
    int blk = d / (MBLK / 4);
    offm[i] = blk < blks_a ? (uint32_t)(blk * total_steps * MBLK + 4 * (d % (MBLK / 4))) : 0x80000000u;
  }
  const uint32_t ldsA = (uint32_t)(uintptr_t)(lds_u8*)smemA;
  const uint32_t ldsB = (uint32_t)(uintptr_t)(lds_u8*)smemB;
  constexpr uint32_t DEAD = 0x40000000u;

#define WG_LOAD(n, sa, slot_a, sb, slot_b)                                                                \
  do {                                                                                                    \
    if ((n) < LA)                                                                                         \
      dma_b128(ba, ldsA + (uint32_t)(slot_a) * ASTAGE + (LA * wave + (n)) * 1024, offa[(n) < LA ? (n) : 0], \
               (sa) < nsteps ? (uint32_t)(sa) * 1024u : DEAD);                                            \
    else if ((n) < LA + LM)                                                                               \
      dma_b32(bm, ldsA + (uint32_t)(slot_a) * ASTAGE + A_BYTES + (LM * wave + ((n) - LA)) * 256,          \
              offm[((n) >= LA && (n) < LA + LM) ? (n) - LA : 0],                                          \
              (sa) < nsteps ? (uint32_t)(sa) * (uint32_t)MBLK : DEAD);                                    \
    else                                                                                                  \
      dma_b128(bb, ldsB + (uint32_t)(slot_b) * BSTAGE + (LB * wave + ((n) - LA - LM)) * 1024,             \
               offb[(n) >= LA + LM ? (n) - LA - LM : 0],                                                  \
               (sb) < nsteps ? (uint32_t)((sb) * KS * ldx_bytes) : DEAD);                                 \
  } while (0)

  f32x4 acc[MI_][NI_];
#pragma unroll
  for (int a = 0; a < MI_; a++)
#pragma unroll
    for (int b = 0; b < NI_; b++) acc[a][b] = (f32x4){0.f, 0.f, 0.f, 0.f};

  const uint32_t fa_off = (uint32_t)(MI_ * wm * 1024 + lane * 16);
  const uint32_t fm_off = (uint32_t)(A_BYTES + MI_ * wm * MBLK + lane * (MB / 4));
  // transposing reads of X: piece r of tile ni covers tokens k0 .. k0 + 3 (bf16) / k0 .. k0 + 7 (fp8)
  uint32_t fb_off[NI_][4];
#pragma unroll
  for (int ni = 0; ni < NI_; ni++)
#pragma unroll
    for (int r = 0; r < 4; r++) {
      int p = NI_ * wn + ni;                                      // feature pair (bf16) / chunk (fp8) of the tile
      if (FP8) {
        int row = 16 * q + 8 * (r & 1) + 64 * (r >> 1) + (j >> 1);
        fb_off[ni][r] = (uint32_t)(row * ROWB + ((p ^ x_swizzle<true>(row)) * 16) + 8 * (j & 1));
      } else {
        int row = 8 * q + 4 * (r & 1) + 32 * (r >> 1) + (j >> 2);
        fb_off[ni][r] = (uint32_t)(row * ROWB + ((p ^ x_swizzle<false>(row)) * 32) + ((j & 3) >> 1) * 16 + 8 * (j & 1));
      }
    }

#define WG_READ_B(dst, base, pc)                                                                          \
  do {                                                                                                    \
    const uint8_t* p_ = (base) + fb_off[(pc) >> 2][(pc) & 3];                                             \
    if (FP8) {                                                                                            \
      i32x2 t_ = __builtin_amdgcn_ds_read_tr8_b64_v2i32((lds_i32x2*)p_);                                  \
      dst[(pc) >> 2][(pc) & 3] = make_uint2((uint32_t)t_[0], (uint32_t)t_[1]);                            \
    } else {                                                                                              \
      bf16x4 t_ = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4*)p_);                              \
      __builtin_memcpy(&dst[(pc) >> 2][(pc) & 3], &t_, 8);                                                \
    }                                                                                                     \
  } while (0)

  // prologue: packed tiles 0, 1 and X tiles 0, 1, 2 in flight, in the order the barriers expect
#pragma unroll
  for (int n = 0; n < NLOAD; n++) WG_LOAD(n, 0, 0, 0, 0);
#pragma unroll
  for (int n = 0; n < NLOAD; n++) WG_LOAD(n, 1, 1, 1, 1);
#pragma unroll
  for (int n = LA + LM; n < NLOAD; n++) WG_LOAD(n, 0, 0, 2, 2);

  uint2 fb0[NI_][4], fb1[NI_][4];     // X fragments: current / next k-step, roles swap every k-step
  uint4 fa[2];                        // packed fragment of row block mi in fa[mi % 2]
  int fidx[2];
  wait_vmcnt<LA + LM + 2 * LB>();     // tiles of k-step 0 have landed
  __syncthreads();
#pragma unroll
  for (int pc = 0; pc < NPIECE; pc++) WG_READ_B(fb0, smemB, pc);
  fa[0] = *(const uint4*)(smemA + fa_off);
  if (FP8) fidx[0] = *(const int*)(smemA + fm_off);
  else fidx[0] = *(const uint16_t*)(smemA + fm_off);

  int s0 = 0, s1 = 1, s2 = 2;         // ring slots of k-steps step, step + 1, step + 2 (both rings)

#define WG_STEP(BC, BX)                                                                                   \
  do {                                                                                                    \
    wait_vmcnt<LB>();                 /* all but the newest X tile: k-step step + 1 has landed */          \
    __syncthreads();                  /* ... for every wave; slots of step - 1 (packed) and step (X) are free */ \
    const uint8_t* pa = smemA + s0 * ASTAGE;                                                              \
    const uint8_t* pa1 = smemA + s1 * ASTAGE;                                                             \
    const uint8_t* pb1 = smemB + s1 * BSTAGE;                                                             \
    _Pragma("unroll") for (int mi = 0; mi < MI_; mi++) {                                                  \
      const uint8_t* an = mi < MI_ - 1 ? pa + (mi + 1) * 1024 : pa1;                                      \
      const uint8_t* mn = mi < MI_ - 1 ? pa + (mi + 1) * MBLK : pa1;                                      \
      fa[(mi + 1) & 1] = *(const uint4*)(an + fa_off);                                                    \
      if (FP8) fidx[(mi + 1) & 1] = *(const int*)(mn + fm_off);                                           \
      else fidx[(mi + 1) & 1] = *(const uint16_t*)(mn + fm_off);                                          \
      _Pragma("unroll") for (int pc = 0; pc < NPIECE; pc++)                                               \
        if (spread(pc, NPIECE, MI_) == mi) WG_READ_B(BX, pb1, pc);                                        \
      _Pragma("unroll") for (int n = 0; n < NLOAD; n++)                                                   \
        if (spread(n, NLOAD, MI_) == mi) WG_LOAD(n, step + 2, s2, step + 3, s0);                          \
      _Pragma("unroll") for (int ni = 0; ni < NI_; ni++) {                                                \
        if (FP8) {                                                                                        \
          i32x4 av;                                                                                       \
          i32x8 bv;                                                                                       \
          __builtin_memcpy(&av, &fa[mi & 1], 16);                                                         \
          __builtin_memcpy(&bv, &BC[ni][0], 32);                                                          \
          /* e5m2 sparsified gradient (packed operand) against e4m3 activations, or both e4m3 */          \
          if (BF8) acc[mi][ni] = __builtin_amdgcn_smfmac_f32_16x16x128_bf8_fp8(av, bv, acc[mi][ni], fidx[mi & 1], 0, 0); \
          else acc[mi][ni] = __builtin_amdgcn_smfmac_f32_16x16x128_fp8_fp8(av, bv, acc[mi][ni], fidx[mi & 1], 0, 0); \
        } else {                                                                                          \
          bf16x8 av;                                                                                      \
          bf16x16 bv;                                                                                     \
          __builtin_memcpy(&av, &fa[mi & 1], 16);                                                         \
          __builtin_memcpy(&bv, &BC[ni][0], 32);                                                          \
          acc[mi][ni] = __builtin_amdgcn_smfmac_f32_16x16x64_bf16(av, bv, acc[mi][ni], fidx[mi & 1], 0, 0); \
        }                                                                                                 \
      }                                                                                                   \
      __builtin_amdgcn_sched_barrier(0);                                                                  \
    }                                                                                                     \
    const int t_ = s0;                                                                                    \
    s0 = s1;                                                                                              \
    s1 = s2;                                                                                              \
    s2 = t_;                                                                                              \
  } while (0)

  int step = 0;
  for (; step + 1 < nsteps; step += 2) {
    WG_STEP(fb0, fb1);
    step++;
    WG_STEP(fb1, fb0);
    step--;
  }
  if (step < nsteps) WG_STEP(fb0, fb1);
#undef WG_STEP
#undef WG_READ_B
#undef WG_LOAD
  wait_vmcnt<0>();
  if (DEALT && at < part_end) __syncthreads();   // every wave has read its last fragments: the next segment may fill the slots

  // epilogue: lane (j, q) register r of tile (mi, ni) is element (o + r, i)
  int plane = part;
  if constexpr (DEALT) plane -= deal.first[member];
  float* dst = out + (int64_t)plane * split_stride;
#pragma unroll
  for (int mi = 0; mi < MI_; mi++)
#pragma unroll
    for (int ni = 0; ni < NI_; ni++) {
      int64_t o = o0 + 16 * MI_ * wm + 16 * mi + 4 * q;
      int64_t i = i0 + 16 * NI_ * wn + 16 * ni + j;
      if (i < I) {
#pragma unroll
        for (int r = 0; r < 4; r++) {
          if (o + r < O) {
            float v = acc[mi][ni][r] * scale;
            float* p = dst + (o + r) * ld_out + i;
            *p = accumulate ? (*p + v) : v;
          }
        }
      }
    }
  } while (DEALT && at < part_end);
}

// ---------------------------------------------------------------------------------------------------------
// 2b. the same GEMM for small and middle problems: 32 WM MT channels x 32 WN NT features by KG groups of WM x WN waves on the 32 x 32
// sparse instructions, group kg taking the k-steps kg, kg + KG, ... of its split through LDS slots of its own; the groups' sums are
// added inside the workgroup, so a problem with few tiles needs neither split partials in memory nor the kernel that sums them.
// Structure as k_linear_fwd_tile.  X tile in LDS: one row per token, 32 NT WN features; the block of 32 features (64 B bf16, 32 B 8-bit)
// number u of token row r lies at position u ^ key(r), so that the rows and columns one transposing read gathers per 32 lanes (4 rows
// x 64 B, 8 rows x 32 B) cover all 64 banks once.
template <bool FP8, int WM, int WN, int MT, int NT, int KG, int NS>
constexpr int wgrad_tile_smem() {
  constexpr int NWG = WM * WN, MB = FP8 ? 16 : 8;
  constexpr int LM = (32 * WM * MT * MB / 256 + NWG - 1) / NWG;
  constexpr int RING = KG * NS * (32 * WM * MT * 64 + NWG * LM * 256 + 128 * 32 * WN * NT);
  constexpr int RED = (KG - 1) * NWG * MT * NT * 4096;
  return RING > RED ? RING : RED;
}

template <bool FP8, bool BF8, int WM, int WN, int MT, int NT, int KG, int NS>
__global__ void __launch_bounds__(64 * WM * WN * KG, 1)
k_wgrad_tile(const uint8_t* __restrict__ vals, const uint8_t* __restrict__ meta, int64_t O, int64_t total_steps,
             const uint8_t* __restrict__ X, int64_t I, int64_t ldx_bytes, int steps_per_split, float scale,
             int accumulate, float* __restrict__ out, int64_t ld_out, int64_t split_stride, int m_tiles, int n_tiles,
             int features_fastest) {
  constexpr int NWG = WM * WN;
  constexpr int BM = 32 * WM * MT, BN = 32 * WN * NT;
  constexpr int EB = FP8 ? 1 : 2, KS = FP8 ? 128 : 64;
  constexpr int MB = FP8 ? 16 : 8, MBLK = 16 * MB;
  constexpr int ROWB = BN * EB;                     // LDS bytes per token row
  constexpr int BSLOT = KS * ROWB;                  // 128 BN for both types
  constexpr int LA = BM / 16 / NWG, LB = BSLOT / 1024 / NWG, LM = (BM * MB / 256 + NWG - 1) / NWG;   // loads per wave and k-step
  constexpr int LPW = LA + LB + LM;
  constexpr int A_BYTES = BM * 64, M_BYTES = NWG * LM * 256, SLOT = A_BYTES + M_BYTES + BSLOT;
  constexpr int UB = 32 * EB, UNITS = ROWB / UB;    // a block of 32 features; blocks per row
  constexpr int CPR = ROWB / 16;                    // 16-byte chunks per row
  static_assert(LA >= 1 && LB >= 1 && ROWB <= 256, "tile shape");
  __shared__ __align__(1024) uint8_t smem[wgrad_tile_smem<FP8, WM, WN, MT, NT, KG, NS>()];
  auto key = [](int r) { return (r / (256 / ROWB)) % UNITS; };

  const int logical = xcd_contiguous(blockIdx.x, gridDim.x);
  const int tiles = m_tiles * n_tiles;
  const int z = logical / tiles, tile = logical % tiles;
  const int tm = features_fastest ? tile / n_tiles : tile % m_tiles;
  const int tn = features_fastest ? tile % n_tiles : tile / m_tiles;

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave_all = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int kg = KG > 1 ? wave_all / NWG : 0, wave = KG > 1 ? wave_all % NWG : wave_all;
  const int wm = wave / WN, wn = wave % WN;
  const int n = lane & 31, hh = lane >> 5, j = lane & 15, jq = (lane >> 4) & 1;
  const int64_t o0 = (int64_t)tm * BM, i0 = (int64_t)tn * BN;
  const int64_t step_begin = (int64_t)z * steps_per_split;
  const int nsteps = (int)((step_begin + steps_per_split < total_steps ? step_begin + steps_per_split : total_steps) - step_begin);
  const int nloc = (nsteps + KG - 1) / KG;
  uint8_t* const ring = smem + kg * NS * SLOT;
  const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_u8*)ring;

  const int64_t rblk0 = o0 / 16, rbn = (O + 15) / 16;
  const int blks_a = (int)((rbn - rblk0) < BM / 16 ? (rbn - rblk0) : BM / 16);
  const i32x4 ba = rsrc_words(vals + (rblk0 * total_steps + step_begin) * 1024, (uint32_t)((blks_a * total_steps - step_begin) * 1024));
  const i32x4 bm = rsrc_words(meta + (rblk0 * total_steps + step_begin) * MBLK, (uint32_t)((blks_a * total_steps - step_begin) * MBLK));
  const int cols_b = (int)((I - i0) < BN ? (I - i0) : BN);
  const i32x4 bb = rsrc_words(X + step_begin * KS * ldx_bytes + i0 * EB, (uint32_t)(((int64_t)nsteps * KS - 1) * ldx_bytes + cols_b * EB));
  // packed blocks past the tile's last one and chunks past its last feature fetch nothing: zeros arrive
  constexpr uint32_t DEAD = 0x80000000u;
  uint32_t offa[LA], offb[LB], offm[LM];
#pragma unroll
  for (int i = 0; i < LA; i++)
    offa[i] = (LA * wave + i) < blks_a ? (uint32_t)((LA * wave + i) * total_steps * 1024 + lane * 16) : DEAD;
#pragma unroll
  for (int i = 0; i < LB; i++) {
    const int d = 64 * (LB * wave + i) + lane;      // 16-byte chunk of the slot
    const int r = d / CPR, cs = d % CPR;            // token row inside the k-step, stored chunk
    const int c = ((cs / (UB / 16)) ^ key(r)) * (UB / 16) + cs % (UB / 16);   // source chunk
    offb[i] = (c * 16 < cols_b * EB) ? (uint32_t)(r * ldx_bytes + c * 16) : DEAD;
  }
#pragma unroll
  for (int i = 0; i < LM; i++) {
    const int d = 64 * (LM * wave + i) + lane, blk = d / (MBLK / 4);
    offm[i] = blk < blks_a ? (uint32_t)(blk * total_steps * MBLK + 4 * (d % (MBLK / 4))) : DEAD;
  }
  auto issue = [&](int ls, int slot) {
    // a step past the last one reads zeros on both sides (its own operand's last values would do for finite inputs only: zero times an
    // infinity is a NaN)
    const int st = ls * KG + kg;
    const uint32_t dead = st < nsteps ? 0u : DEAD, sc = st < nsteps ? (uint32_t)st : 0u;
    const uint32_t base = lds0 + (uint32_t)slot * SLOT;
#pragma unroll
    for (int i = 0; i < LA; i++) dma_b128(ba, base + (LA * wave + i) * 1024, offa[i] | dead, sc * 1024u);
#pragma unroll
    for (int i = 0; i < LM; i++) dma_b32(bm, base + A_BYTES + (LM * wave + i) * 256, offm[i] | dead, sc * (uint32_t)MBLK);
#pragma unroll
    for (int i = 0; i < LB; i++) dma_b128(bb, base + A_BYTES + M_BYTES + (LB * wave + i) * 1024, offb[i] | dead, sc * (uint32_t)(KS * ldx_bytes));
  };

  f32x16 acc[MT][NT];
#pragma unroll
  for (int m = 0; m < MT; m++)
#pragma unroll
    for (int t = 0; t < NT; t++)
#pragma unroll
      for (int r = 0; r < 16; r++) acc[m][t][r] = 0.f;

  // fragments of half kk of a k-step.  A as in the forward kernel.  B lane (column n, hh): tokens 8 hh .. and 16 + 8 hh .. of the half's 32
  // (bf16; 8-bit: 16 hh .. and 32 + 16 hh .. of 64), by transposing reads of 4 (8) token rows x 16 features each.
  const uint32_t fa_off = (uint32_t)((2 * wm * MT + (n >> 4)) * 1024 + (16 * hh + j) * 16);
  const uint32_t fm_off = (uint32_t)(A_BYTES + (2 * wm * MT + (n >> 4)) * MBLK + (16 * hh + j) * (MB / 4));
  uint32_t fb_off[NT][4];                           // + kk * KS / 2 * ROWB (the key does not change: KS / 2 rows are whole periods)
#pragma unroll
  for (int t = 0; t < NT; t++)
#pragma unroll
    for (int r = 0; r < 4; r++) {
      const int row = FP8 ? 16 * hh + 8 * (r & 1) + 32 * (r >> 1) + (j >> 1) : 8 * hh + 4 * (r & 1) + 16 * (r >> 1) + (j >> 2);
      const int in_unit = FP8 ? 16 * jq + 8 * (j & 1) : 32 * jq + 8 * (j & 3);
      fb_off[t][r] = (uint32_t)(A_BYTES + M_BYTES + row * ROWB + (((wn * NT + t) ^ key(row)) * UB) + in_unit);
    }
  uint4 fa[2][MT];
  uint2 fb[2][NT][4];
  int fi[2][MT];
  auto read_frag = [&](int kk, const uint8_t* sl) {
#pragma unroll
    for (int m = 0; m < MT; m++) {
      fa[kk][m] = *(const uint4*)(sl + fa_off + m * 2048 + kk * 512);
      if (FP8) fi[kk][m] = *(const int*)(sl + fm_off + m * 2 * MBLK + kk * 32 * (MB / 4));
      else fi[kk][m] = *(const uint16_t*)(sl + fm_off + m * 2 * MBLK + kk * 32 * (MB / 4));
    }
#pragma unroll
    for (int t = 0; t < NT; t++)
#pragma unroll
      for (int r = 0; r < 4; r++) {
        const uint8_t* p = sl + fb_off[t][r] + kk * (KS / 2) * ROWB;
        if (FP8) {
          const i32x2 v = __builtin_amdgcn_ds_read_tr8_b64_v2i32((lds_i32x2*)p);
          fb[kk][t][r] = make_uint2((uint32_t)v[0], (uint32_t)v[1]);
        } else {
          const bf16x4 v = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4*)p);
          __builtin_memcpy(&fb[kk][t][r], &v, 8);
        }
      }
  };
  auto mma = [&](int kk) {
#pragma unroll
    for (int m = 0; m < MT; m++)
#pragma unroll
      for (int t = 0; t < NT; t++) {
        if (FP8) {
          i32x4 av;
          i32x8 bv;
          __builtin_memcpy(&av, &fa[kk][m], 16);
          __builtin_memcpy(&bv, &fb[kk][t][0], 32);
          if (BF8) acc[m][t] = __builtin_amdgcn_smfmac_f32_32x32x64_bf8_fp8(av, bv, acc[m][t], fi[kk][m], 0, 0);
          else acc[m][t] = __builtin_amdgcn_smfmac_f32_32x32x64_fp8_fp8(av, bv, acc[m][t], fi[kk][m], 0, 0);
        } else {
          bf16x8 av;
          bf16x16 bv;
          __builtin_memcpy(&av, &fa[kk][m], 16);
          __builtin_memcpy(&bv, &fb[kk][t][0], 32);
          acc[m][t] = __builtin_amdgcn_smfmac_f32_32x32x32_bf16(av, bv, acc[m][t], fi[kk][m], 0, 0);
        }
      }
  };

#pragma unroll
  for (int k = 0; k < NS; k++) issue(k, k);
  wait_vmcnt<(NS - 1) * LPW>();
  __syncthreads();
  read_frag(0, ring);
  int slot = 0, slot1 = 1 % NS;
  for (int s = 0; s < nloc; s++) {
    read_frag(1, ring + slot * SLOT);
    mma(0);
    __builtin_amdgcn_sched_barrier(0);
    wait_vmcnt<(NS - 2) * LPW>();          // this wave's share of tile s + 1 has landed
    __syncthreads();                       // ... everybody's; the slot of s has been read
    read_frag(0, ring + slot1 * SLOT);
    issue(s + NS, slot);
    mma(1);
    __builtin_amdgcn_sched_barrier(0);
    slot = slot1;
    slot1 = slot1 == NS - 1 ? 0 : slot1 + 1;
  }
  wait_vmcnt<0>();

  if (KG > 1) {
    // sums of the k-groups: groups 1 .. KG - 1 leave theirs in LDS, lane for lane
    __syncthreads();
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
    if (kg > 0) return;
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
  // lane (n, hh) register 4 g + r of tile (m, t) is element (o + 8 g + 4 hh + r, i + n): 128 contiguous bytes per row
  float* dst = out + (int64_t)z * split_stride;
#pragma unroll
  for (int m = 0; m < MT; m++)
#pragma unroll
    for (int t = 0; t < NT; t++) {
      const int64_t o = o0 + 32 * (wm * MT + m) + 4 * hh, i = i0 + 32 * (wn * NT + t) + n;
      if (i < I) {
#pragma unroll
        for (int r = 0; r < 16; r++) {
          const int64_t row = o + 8 * (r >> 2) + (r & 3);
          if (row < O) {
            const float v = acc[m][t][r] * scale;
            float* p = dst + row * ld_out + i;
            *p = accumulate ? (*p + v) : v;
          }
        }
      }
    }
}

// ---------------------------------------------------------------------------------------------------------
// 3. out[o][i] = scale * sum_z ws[z][o][i]  (+ out[o][i]); z ascending: a fixed order.  DEALT: a tile has as many z as its member of the
// group has segments.
template <bool DEALT>
__global__ void __launch_bounds__(256)
k_wgrad_reduce(const float* __restrict__ ws, int splits, int64_t O, int64_t I, float scale, int accumulate,
               float* __restrict__ dW, int64_t lddw, uint32_t segments, int groups, int bm, int bn, WgradTiles order) {
  int64_t n4 = O * (I / 4);
  for (int64_t c = (int64_t)blockIdx.x * 256 + threadIdx.x; c < n4; c += (int64_t)gridDim.x * 256) {
    int64_t row = c / (I / 4), col = (c - row * (I / 4)) * 4;
    if (DEALT) {
      const uint32_t tm = (uint32_t)row / (uint32_t)bm, tn = (uint32_t)col / (uint32_t)bn;
      const uint32_t tile = order.features_fastest ? tm * (uint32_t)order.n_tiles + tn : tn * (uint32_t)order.m_tiles + tm;
      splits = (int)((segments >> (4 * (tile / (uint32_t)groups))) & 15u);
    }
    f32x4 s0 = __builtin_nontemporal_load((const f32x4*)(ws + row * I + col));
    float4 s = make_float4(s0[0], s0[1], s0[2], s0[3]);
    for (int z = 1; z < splits; z++) {
      f32x4 v0 = __builtin_nontemporal_load((const f32x4*)(ws + (int64_t)z * O * I + row * I + col));
      float4 v = make_float4(v0[0], v0[1], v0[2], v0[3]);
      s.x += v.x; s.y += v.y; s.z += v.z; s.w += v.w;
    }
    float4* p = (float4*)(dW + row * lddw + col);
    float4 r = make_float4(s.x * scale, s.y * scale, s.z * scale, s.w * scale);
    if (accumulate) { float4 d = *p; r.x += d.x; r.y += d.y; r.z += d.z; r.w += d.w; }
    store_stream_b128(p, r);
  }
}

__global__ void __launch_bounds__(256)
k_zero_rows(float* __restrict__ dW, int64_t O, int64_t I, int64_t lddw) {
  int64_t n = O * I;
  for (int64_t c = (int64_t)blockIdx.x * 256 + threadIdx.x; c < n; c += (int64_t)gridDim.x * 256) {
    int64_t row = c / I, col = c - row * I;
    dW[row * lddw + col] = 0.0f;
  }
}

// ---------------------------------------------------------------------------------------------------------
// host: path choice, tile and split choice, workspace layout
struct WgradPlan {
  bool packed;          // true: estimator pre-pass + GEMM on the packed operand; false: fused kernel
  int shape;            // tile of the packed GEMM
  int splits;           // token-axis splits; with several members to a group: the most segments of a tile
  int steps_per_split;
  WgradDeal deal;       // 256- and 192-wide tiles: how the k-steps go to workgroups (members > 1 only where the whole token axis is one chunk)
  int64_t chunk_steps;  // k-steps the packed path takes at a time (all of them, unless the operand would not fit the built-in scratch)
  size_t vals_bytes, meta_bytes, partial_bytes;   // workspace sections (each a multiple of 256)
  size_t bytes() const { return vals_bytes + meta_bytes + partial_bytes; }
};

static size_t round256(size_t x) { return (x + 255) / 256 * 256; }

// Tile shapes of the packed GEMM and their time model in microseconds: a workgroup costs F + nk * step with nk its k-steps (each k-group
// of a workgroup takes a KG-th of its split's) and step = max(lat, r * thr) for r workgroups sharing a CU; R fit a CU, what does not fit
// runs in further rounds; base + store * (bytes written at 5 TB/s) on top.  Fitted to 760 problems of random size (64 to 32768 tokens,
// 64 to 5120 channels and features) in all shapes and up to 24 splits: 2 % rms for the large tiles, 5 % for the small ones; the choice
// costs 1 % against the fastest candidate on average.
struct WgradShape {
  int bm, bn, kg, r;
  double f, lat, thr, base, store;
};
enum { WG_256x256, WG_192x192, WG_256x192, WG_128, WG_128_KG2, WG_128x64, WG_64, WG_64_KG2, WG_SHAPES, WG_SHAPES8 = WG_64_KG2 };   // two groups on 64 x 64: bf16 only (in 8 bits the best of 3 in 150 000 random problems)
static const WgradShape kWgrad16[WG_SHAPES] = {
  {256, 256, 1, 1, 6.40, 0.644, 0.144, 3.52, 0.68},
  {192, 192, 1, 1, 1.58, 0.499, 0.410, 5.51, 0.89},
  {256, 192, 1, 1, 2.20, 0.568, 0.165, 6.19, 0.80},
  {128, 128, 1, 2, 0.00, 0.310, 0.280, 6.21, 1.07},
  {128, 128, 2, 1, 2.84, 0.569, 0.255, 4.07, 1.55},
  {128, 64, 1, 2, 0.00, 0.211, 0.221, 4.36, 1.35},
  {64, 64, 1, 3, 0.00, 0.187, 0.153, 3.53, 1.73},
  {64, 64, 2, 1, 1.88, 0.006, 0.319, 1.93, 2.38},
};
static const WgradShape kWgrad8[WG_SHAPES8] = {
  {256, 256, 1, 1, 7.49, 0.689, 0.587, 1.95, 0.69},
  {192, 192, 1, 1, 1.73, 0.243, 0.544, 5.34, 0.85},
  {256, 192, 1, 1, 3.50, 0.056, 0.609, 4.79, 0.72},
  {128, 128, 1, 2, 0.07, 0.349, 0.313, 5.90, 1.14},
  {128, 128, 2, 1, 2.90, 0.664, 0.171, 3.76, 1.49},
  {128, 64, 1, 2, 0.40, 0.247, 0.265, 3.76, 1.27},
  {64, 64, 1, 3, 0.00, 0.178, 0.201, 3.45, 1.45},
};

static double wgrad_model_us(const WgradShape& w, int64_t O, int64_t I, int64_t sps, int64_t splits) {
  const int64_t wgs = ((O + w.bm - 1) / w.bm) * ((I + w.bn - 1) / w.bn) * splits;
  const double nk = (double)((sps + w.kg - 1) / w.kg), out_us = (double)O * (double)I * 4.0 / 5e6;
  const int64_t n = (wgs + NUM_CU - 1) / NUM_CU, full = n / w.r, rem = n % w.r;      // workgroups on the busiest CU: full rounds of r, and a rest
  double t = w.base + w.store * out_us * (double)splits + (double)full * (w.f + nk * (w.lat > w.r * w.thr ? w.lat : w.r * w.thr));
  if (rem) t += w.f + nk * (w.lat > rem * w.thr ? w.lat : rem * w.thr);
  if (splits > 1) {
    const double red = 2.0 + 0.61 * (double)(splits + 1) * out_us;
    t += (red > 4.0 ? red : 4.0) + 0.1 * (double)splits;
  }
  return t;
}

static double dealt_model_us(const WgradShape& w, const WgradDeal& d, int64_t O, int64_t I, int64_t steps) {
  const double step = w.lat > w.thr ? w.lat : w.thr, out_us = (double)O * (double)I * 4.0 / 5e6;
  double longest = 0.0, planes = 0.0;
  for (int c = 0; c < d.parts; c++) {
    const int64_t segments = d.bound[c + 1] > d.bound[c] ? (d.bound[c + 1] - 1) / steps - d.bound[c] / steps + 1 : 0;
    const double t = (double)segments * w.f + (double)(d.bound[c + 1] - d.bound[c]) * step;
    planes += (double)segments / (double)d.members;
    longest = t > longest ? t : longest;
  }
  const double red = 2.0 + 0.61 * (planes + 1.0) * out_us;
  return w.base + w.store * out_us * planes + longest + (red > 4.0 ? red : 4.0) + 0.1 * planes;
}

// The two ways to run a problem, same units: estimator pre-pass (streaming) and a second launch before the packed GEMM; or the fused
// kernel, whose workgroups fill a CU each and whose time per k-step is the vector pipe's.  The pre-pass's 8-bit row is that of an estimator that took
// one and a half times as long as today's (0.36e-6 us per element).  Refitted, it would take the packed path in 9 of 1000 random problems that run the fused kernel now, narrow ones of a few us,
// and would let 7 of 10000 grow out of the built-in scratch, whose calls without a workspace of their own run today.
static double mvue_model_us(int64_t T, int64_t O, bool fp8) {
  const double t = 3.7 + (fp8 ? 0.56e-6 : 0.68e-6) * (double)T * (double)O;
  return (t > 4.5 ? t : 4.5) + 1.0;
}
static double fused_model_us(int64_t steps, int64_t O, int64_t I, bool fp8) {
  const int64_t wgs = ((O + 15) / 16) * ((I + 63) / 64), rounds = (wgs + NUM_CU - 1) / NUM_CU;
  const double t = 1.2 + (double)rounds * ((fp8 ? 1.8 : 2.1) + (double)((steps + 3) / 4) * (fp8 ? 1.37 : 0.77));
  return t > 4.0 ? t : 4.0;
}

// Tile shape / split count forced by sste_wgrad_plan_override (-1 / 0 = automatic choice).
static std::atomic<int> g_force_shape{-1}, g_force_splits{0};

bool wgrad_plan_override(int mi, int ni, int splits) {
  int shape;
  if (mi == 0 && ni == 0) shape = -1;
  else if (mi == 8 && ni == 4) shape = WG_256x256;
  else if (mi == 6 && ni == 3) shape = WG_192x192;
  else if (mi == 8 && ni == 3) shape = WG_256x192;
  else return false;
  if (splits < 0 || splits > 32) return false;
  g_force_shape = shape;
  g_force_splits = splits;
  return true;
}

// deals: tiles may be dealt in groups.
static WgradPlan make_wgrad_plan(int64_t T, int64_t O, int64_t I, int dtype, bool deals) {
  WgradPlan p{};
  const bool fp8 = dtype != SSTE_BF16;
  const int ks = fp8 ? 128 : 64;
  int64_t steps = T / ks;
  if (steps <= 0 || O == 0 || I == 0 || product_reaches(T, O / 16 * 16 + 16, 1ll << 40)) return p;
  const int64_t rows = (O + 15) / 16 * 16, all_steps = steps;
  const int64_t step_vals = rows * 64, step_meta = rows * (ks / 8);        // operand bytes per k-step
  const bool long_wide = T >= 2048 && O >= 256 && I >= 256;
  if (!long_wide) {
    // Callers without a workspace are served from SSTE_NOALLOC_SCRATCH_BYTES, and short or narrow problems never ask for more: theirs
    // run in chunks of the token axis, each added to the one before, where the operand alone would take three quarters of that.
    const int64_t most = (int64_t)(SSTE_NOALLOC_SCRATCH_BYTES / 4 * 3) / (step_vals + step_meta);
    if (most == 0) return p;
    const int64_t chunks = (steps + most - 1) / most;
    steps = (steps + chunks - 1) / chunks;
  }
  const size_t vals_bytes = round256((size_t)(steps * step_vals)), meta_bytes = round256((size_t)(steps * step_meta));
  const WgradShape* tab = fp8 ? kWgrad8 : kWgrad16;
  const int fshape = g_force_shape, fs = g_force_splits;
  const int64_t smax = steps / 8 < 1 ? 1 : steps / 8 < 32 ? steps / 8 : 32;
  struct Choice {
    double t;
    int shape;
    int64_t sps, splits;
    size_t partial_bytes;
  } any{1e30, 0, 1, 1, 0}, small = any;                       // the fastest; the fastest that fits the built-in scratch
  for (int k = 0; k < (fp8 ? WG_SHAPES8 : WG_SHAPES); k++) {
    if (fshape >= 0 && k != fshape) continue;
    const int64_t tiles = ((O + tab[k].bm - 1) / tab[k].bm) * ((I + tab[k].bn - 1) / tab[k].bn);
    for (int64_t s = fs ? (fs < smax ? fs : smax) : 1; s <= smax; s++) {
      if (s > 1 && !fs && (s - 1) * tiles >= 4 * NUM_CU) break;                          // splits are there to fill the chip
      const int64_t sps = (steps + s - 1) / s, splits = (steps + sps - 1) / sps;       // no empty split
      const size_t partial_bytes = splits > 1 ? round256((size_t)splits * (size_t)O * (size_t)I * sizeof(float)) : 0;
      const double t = wgrad_model_us(tab[k], O, I, sps, splits);
      if (t < any.t) any = {t, k, sps, splits, partial_bytes};
      if (t < small.t && vals_bytes + meta_bytes + partial_bytes <= SSTE_NOALLOC_SCRATCH_BYTES) small = {t, k, sps, splits, partial_bytes};
      if (fs) break;
    }
  }
  const double pre = mvue_model_us(steps * ks, O, fp8);
  // what fits the built-in scratch is taken where it costs little (more, where few splits have anything to give: the unsplit 192 x 192
  // tiles nearly fill the chip), so that calls without a workspace run as well
  const int64_t t192 = ((O + 191) / 192) * ((I + 191) / 192);
  const double worth = t192 >= NUM_CU * 5 / 8 && t192 <= NUM_CU ? 1.2 : 1.1;
  const Choice& c = !long_wide || pre + small.t < worth * (pre + any.t) ? small : any;
  // The same tiles dealt in groups, where that is faster by more than the model errs (5 %; with 3 % a fifth of the problems lose).  It takes the place of a choice only on the same side of
  // the built-in scratch, so that the same calls run without a workspace.
  struct {
    double t;
    int shape;
    WgradDeal deal;
    size_t partial_bytes;
  } dealt{0.95 * c.t, 0, {}, 0};
  const size_t operand_bytes = vals_bytes + meta_bytes;
  const bool fits = operand_bytes + c.partial_bytes <= SSTE_NOALLOC_SCRATCH_BYTES;
  for (int k = WG_256x256; k <= WG_256x192; k++) {
    if (!deals || !long_wide || fs || (fshape >= 0 && k != fshape)) continue;
    const int64_t tiles = ((O + tab[k].bm - 1) / tab[k].bm) * ((I + tab[k].bn - 1) / tab[k].bn);
    if (tiles >= NUM_CU) continue;
    for (int members = 2; members <= DEAL_MEMBERS; members++) {
      const int64_t groups = (tiles + members - 1) / members, parts = NUM_CU / groups;
      if (parts <= members || parts > DEAL_PARTS || std::gcd((int)parts, members) != 1) continue;
      WgradDeal d;
      if (!deal_group(d, tab[k].f, tab[k].lat > tab[k].thr ? tab[k].lat : tab[k].thr, steps, members, (int)parts, (int)groups)) continue;
      const size_t partial_bytes = round256((size_t)most_segments(d) * (size_t)O * (size_t)I * sizeof(float));
      if ((operand_bytes + partial_bytes <= SSTE_NOALLOC_SCRATCH_BYTES) != fits) continue;
      const double t = dealt_model_us(tab[k], d, O, I, steps);
      if (t < dealt.t) dealt = {t, k, d, partial_bytes};
    }
  }
  // The fused kernel serves problems that are short or narrow, where the second launch would cost more than the repeated estimator.
  p.packed = long_wide || (double)((all_steps + steps - 1) / steps) * (pre + c.t) < fused_model_us(all_steps, O, I, fp8);
  if (p.packed && c.t < 1e30) {
    const bool group = dealt.deal.members > 1;
    p.shape = group ? dealt.shape : c.shape;
    p.splits = group ? most_segments(dealt.deal) : (int)c.splits;
    p.steps_per_split = (int)c.sps;
    p.deal = dealt.deal;
    p.chunk_steps = steps;
    p.vals_bytes = vals_bytes;
    p.meta_bytes = meta_bytes;
    p.partial_bytes = group ? dealt.partial_bytes : c.partial_bytes;
  } else {
    p.packed = false;
  }
  return p;
}

// The plan of a problem, kept per thread for the last few problems asked for (a call asks several times, and a layer calls again).
static WgradPlan wgrad_plan(int64_t T, int64_t O, int64_t I, int dtype, bool deals = true) {
  struct Entry {
    int64_t T, O, I;
    int dtype, shape, splits;
    bool deals;
    WgradPlan plan;
    bool used;
  };
  static thread_local Entry cache[16];
  static thread_local unsigned oldest = 0;
  const int shape = g_force_shape, splits = g_force_splits;
  for (const Entry& e : cache)
    if (e.used && e.T == T && e.O == O && e.I == I && e.dtype == dtype && e.shape == shape && e.splits == splits && e.deals == deals) return e.plan;
  Entry& e = cache[oldest];
  oldest = (oldest + 1) % 16;
  e = Entry{T, O, I, dtype, shape, splits, deals, make_wgrad_plan(T, O, I, dtype, deals), true};
  return e.plan;
}

void describe_wgrad(int64_t T, int64_t O, int64_t I, int dtype, char* text, size_t n) {
  const WgradPlan p = wgrad_plan(T, O, I, dtype);
  if (!p.packed) {
    snprintf(text, n, "fused kg 8 r 1 splits 1 chunks 1 grid %lld block 512", (long long)(((O + 15) / 16) * ((I + 63) / 64)));
    return;
  }
  const WgradShape& w = kWgrad16[p.shape];
  const int64_t steps = T / (dtype != SSTE_BF16 ? 128 : 64), chunks = (steps + p.chunk_steps - 1) / p.chunk_steps;
  if (p.deal.members > 1) {
    snprintf(text, n, "%dx%d kg %d r %d splits %d/%d chunks %lld grid %lld block 512", w.bm, w.bn, w.kg, w.r, p.deal.parts, p.deal.members, (long long)chunks,
             (long long)p.deal.parts * p.deal.groups);
    return;
  }
  snprintf(text, n, "%dx%d kg %d r %d splits %d chunks %lld grid %lld block %d", w.bm, w.bn, w.kg, w.r, p.splits, (long long)chunks,
           (long long)(((O + w.bm - 1) / w.bm) * ((I + w.bn - 1) / w.bn) * p.splits), p.shape <= WG_256x192 ? 512 : 256 * w.kg);
}

// Arguments of the packed GEMM's kernels.
struct WgradGemm {
  const uint8_t* vals;
  const uint8_t* meta;
  int64_t O, steps;
  const uint8_t* X;
  int64_t I, ldx_bytes;
  int splits, steps_per_split;
  float scale;
  int accumulate;
  float* out;
  int64_t ld_out, split_stride;
  WgradDeal deal;         // members 0: splits of steps_per_split
};

static WgradTiles wgrad_tiles(int shape, int64_t O, int64_t I, int splits, const WgradDeal& deal) {
  const WgradShape& w = kWgrad16[shape];
  const int m_tiles = (int)((O + w.bm - 1) / w.bm), n_tiles = (int)((I + w.bn - 1) / w.bn);
  // Tile order inside a split.  The workgroups of one XCD (an eighth of the grid, consecutive logical numbers)
  // share an L2: with channel tiles fastest they cover many channel tiles of few feature tiles, with feature
  // tiles fastest the other way round.  Each channel tile costs the XCD a slice of the packed operand
  // (0.5625 bytes per element), each feature tile a slice of X (1 byte per element): take the cheaper order
  // (measured 1...4 % on the layers where the choice differs from channel tiles fastest).
  const int per_xcd = ((deal.members > 1 ? deal.groups * deal.parts : m_tiles * n_tiles * splits) + 7) / 8;
  auto xcd_cost = [&](int fast, int slow, double fast_bytes, double slow_bytes) {
    const int nfast = per_xcd < fast ? per_xcd : fast;
    int nslow = (per_xcd + fast - 1) / fast;
    if (nslow > slow) nslow = slow;
    return nfast * fast_bytes + nslow * slow_bytes;
  };
  const double a_bytes = w.bm * 0.5625, x_bytes = w.bn;
  const int features_fastest = xcd_cost(n_tiles, m_tiles, x_bytes, a_bytes) < xcd_cost(m_tiles, n_tiles, a_bytes, x_bytes) ? 1 : 0;
  return {m_tiles, n_tiles, features_fastest};
}

template <bool FP8, bool BF8>
static void launch_wgrad_gemm(int shape, const WgradGemm& g, const WgradTiles& order, hipStream_t s) {
  const int tiles = order.m_tiles * order.n_tiles;
  const WgradSplits plain{tiles, g.steps_per_split};
#define WG_DEAL(MI, NI, DEALT, DEAL, PARTS)                                                                                           \
  SSTE_LAUNCH(SSTE_K_WGRAD, (k_wgrad_gemm<FP8, MI, NI, BF8, DEALT>), dim3((unsigned)((DEAL).groups * (PARTS))), dim3(512), s, g.vals, g.meta,   \
              g.O, g.steps, g.X, g.I, g.ldx_bytes, DEAL, g.scale, g.accumulate, g.out, g.ld_out, g.split_stride, order)
#define WG_LARGE(MI, NI)                                                  \
  do {                                                                    \
    if (g.deal.members > 1) WG_DEAL(MI, NI, true, g.deal, g.deal.parts);  \
    else WG_DEAL(MI, NI, false, plain, g.splits);                         \
  } while (0)
#define WG_TILE(WM, WN, MT, NT, KG, NS)                                                                                               \
  SSTE_LAUNCH(SSTE_K_WGRAD, (k_wgrad_tile<FP8, BF8, WM, WN, MT, NT, KG, NS>), dim3((unsigned)(tiles * g.splits)), dim3(64 * WM * WN * KG), s,   \
              g.vals, g.meta, g.O, g.steps, g.X, g.I, g.ldx_bytes, g.steps_per_split, g.scale, g.accumulate, g.out, g.ld_out, g.split_stride,   \
              order.m_tiles, order.n_tiles, order.features_fastest)
  switch (shape) {
    case WG_256x256: WG_LARGE(8, 4); break;
    case WG_192x192: WG_LARGE(6, 3); break;
    case WG_256x192: WG_LARGE(8, 3); break;
    case WG_128: WG_TILE(2, 2, 2, 2, 1, 3); break;
    case WG_128_KG2: WG_TILE(2, 2, 2, 2, 2, 3); break;
    case WG_128x64: WG_TILE(2, 2, 2, 1, 1, 4); break;
    case WG_64: WG_TILE(2, 2, 1, 1, 1, 4); break;
    default:
      if constexpr (!FP8) WG_TILE(2, 2, 1, 1, 2, 4);
      break;
  }
#undef WG_TILE
#undef WG_LARGE
#undef WG_DEAL
}

size_t wgrad_workspace_bytes(int64_t T, int64_t O, int64_t I, int dtype) {
  return wgrad_plan(T, O, I, dtype).bytes();
}

// What a call needs at least: where the plan deals tiles in groups and a workspace for that is missing, the splits it would take otherwise, whose
// partial sums may be fewer.
size_t wgrad_least_workspace_bytes(int64_t T, int64_t O, int64_t I, int dtype) {
  const WgradPlan p = wgrad_plan(T, O, I, dtype);
  if (p.deal.members <= 1) return p.bytes();
  const size_t splits = wgrad_plan(T, O, I, dtype, false).bytes();
  return splits < p.bytes() ? splits : p.bytes();
}

bool linear_wgrad_supported(int64_t T, int64_t O, int64_t I, int64_t ldx, int dtype) {
  int64_t eb = dtype != SSTE_BF16 ? 1 : 2;
  if (product_reaches(O / 128 + 1, I / 128 + 1, 0x80000000ll / 32)) return false;
  if (product_reaches(T, O / 16 * 16 + 16, 1ll << 40)) return false;                            // the packed operand's size
  // 32-bit offsets of the packed GEMM: short or narrow problems beyond them run the fused kernel
  return !product_reaches(T, ldx, (1ll << 31) / eb) || T < 2048 || O < 256 || I < 256;
}

hipError_t launch_linear_wgrad(const void* dY, int64_t T, int64_t O, int64_t lddy, int dtype, const void* X,
                               int64_t I, int64_t ldx, float scale, RngKey key, float* dW, int64_t lddw,
                               int accumulate, void* ws, size_t ws_bytes, hipStream_t s) {
  if (O == 0 || I == 0) return hipSuccess;
  bool fp8 = dtype != SSTE_BF16;
  int ks = fp8 ? 128 : 64, eb = fp8 ? 1 : 2;
  int64_t steps = T / ks;
  if (steps == 0) {
    if (!accumulate) {
      int64_t blocks = (O * I + 255) / 256;
      if (blocks > 4096) blocks = 4096;
      hipLaunchKernelGGL(k_zero_rows, dim3((unsigned)blocks), dim3(256), 0, s, dW, O, I, lddw);
    }
    return hipGetLastError();
  }
  WgradPlan p = wgrad_plan(T, O, I, dtype);
  if (p.deal.members > 1 && ws_bytes < p.bytes()) p = wgrad_plan(T, O, I, dtype, false);
  if (!p.packed || !ws || product_reaches(T, ldx, (1ll << 31) / eb)) return launch_wgrad_fused(dY, T, O, lddy, dtype, X, I, ldx, key, scale, accumulate, dW, lddw, s);
  uint8_t* const vals = (uint8_t*)ws;
  uint8_t* const meta = vals + p.vals_bytes;
  float* const partial = (float*)(meta + p.meta_bytes);
  for (int64_t step0 = 0; step0 < steps; step0 += p.chunk_steps) {
    const int64_t n = steps - step0 < p.chunk_steps ? steps - step0 : p.chunk_steps;
    const bool group = p.deal.members > 1;
    const int splits = group ? p.splits : (int)((n + p.steps_per_split - 1) / p.steps_per_split), acc = step0 > 0 ? 1 : accumulate;
    const uint8_t* const dYc = (const uint8_t*)dY + step0 * ks * lddy * eb;
    const uint8_t* const Xc = (const uint8_t*)X + step0 * ks * ldx * eb;
    RngKey kc = key;
    kc.first_group += (uint64_t)(step0 * (ks / 4));
    launch_mvue_pack(dYc, n * ks, O, lddy, dtype, kc, vals, meta, s, SSTE_K_MVUE_PACK);
    const WgradGemm g = splits > 1 ? WgradGemm{vals, meta, O, n, Xc, I, ldx * eb, splits, p.steps_per_split, 1.0f, 0, partial, I, O * I, p.deal}
                                   : WgradGemm{vals, meta, O, n, Xc, I, ldx * eb, 1, p.steps_per_split, scale, acc, dW, lddw, 0, p.deal};
    const WgradTiles order = wgrad_tiles(p.shape, O, I, splits, p.deal);
    if (dtype == SSTE_F8E5M2) launch_wgrad_gemm<true, true>(p.shape, g, order, s);
    else if (fp8) launch_wgrad_gemm<true, false>(p.shape, g, order, s);
    else launch_wgrad_gemm<false, false>(p.shape, g, order, s);
    if (splits > 1) {
      int64_t blocks = (O * (I / 4) + 255) / 256;
      if (blocks > 2048) blocks = 2048;
      const WgradShape& w = kWgrad16[p.shape];
      if (group)
        SSTE_LAUNCH(SSTE_K_WGRAD_REDUCE, k_wgrad_reduce<true>, dim3((unsigned)blocks), dim3(256), s, (const float*)partial, splits, O, I, scale, acc,
                    dW, lddw, p.deal.segments, p.deal.groups, w.bm, w.bn, order);
      else
        SSTE_LAUNCH(SSTE_K_WGRAD_REDUCE, k_wgrad_reduce<false>, dim3((unsigned)blocks), dim3(256), s, (const float*)partial, splits, O, I, scale, acc,
                    dW, lddw, 0u, 1, 1, 1, order);
    }
  }
  return hipGetLastError();
}

// ---------------------------------------------------------------------------------------------------------
// Scratch for callers that cannot allocate: the workspace of launch_linear_wgrad inside the library's own
// device image.  Every GPU the library runs on holds its own copy of the array until the process ends.  In
// host code the array's name is only a handle for the runtime; the device address is asked for once per
// device (with that device current) and used from then on.
static __device__ __align__(256) unsigned char scratch[SSTE_NOALLOC_SCRATCH_BYTES];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxDevices] = {};
}  // namespace

// Device address of this GPU's scratch array (nullptr + *err on failure).  No allocation takes place.
void* noalloc_scratch(hipError_t* err) {
  int dev = -1;
  *err = hipGetDevice(&dev);
  if (*err != hipSuccess) return nullptr;
  if (dev < 0 || dev >= kMaxDevices) {
    *err = hipErrorInvalidDevice;
    return nullptr;
  }
  std::lock_guard<std::mutex> lk(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    *err = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (*err != hipSuccess) return nullptr;
    g_scratch_ptr[dev] = p;
  }
  return g_scratch_ptr[dev];
}

}  // namespace sste
