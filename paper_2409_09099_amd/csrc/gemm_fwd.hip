// Forward GEMM of the S-STE linear layer (paper Sec. 5.1): Z = X S(W)^T with S(W) 2:4 sparse.
//
// MFMA mapping: Z^T = S(W) X^T, so the sparse matrix is MFMA operand A (rows = output channels o,
// contraction k = input features, 2:4 along k) and X supplies operand B with k contiguous in memory.
// One sparse MFMA (v_smfmac_f32_16x16x64_bf16 / v_smfmac_f32_16x16x128_fp8_fp8) consumes, per lane,
// 16 bytes of packed values, their position bits, and two 16-byte pieces of an X row:
//   A: lane (row i = lane % 16, qa = lane / 16) holds compressed values [8 qa, 8 qa + 8) of the 32
//      (64 for fp8) that make up the k-step, and their 2-bit positions, 2 bits per value;
//   B: lane (col j = lane % 16, qb = lane / 16) holds dense k in [8 qb, 8 qb + 8) and [32 + 8 qb, 32 + 8 qb + 8)
//      (bf16; for fp8 16-element pieces at 16 qb and 64 + 16 qb): byte offsets 16 qb and 64 + 16 qb.
//   D: lane (j, q) register r holds element (row 4 q + r, col j).
// In bytes a k-step is the same for both types: 64 B of values + 128 B of X per row.
//
// Tiling: every wave owns a grid of 16 x 16 MFMA tiles (8 x 4 = 128 channels x 64 tokens in the main
// shape): per sparse MFMA it reads about 540 B of fragments from LDS, inside the LDS read rate of the CU.
// Six kernels share the operand layouts; a time model fitted to a sweep picks one (fwd_choice):
//   k_linear_fwd_pipe   software-pipelined 128 x 256 tiles, 8 waves, one workgroup per CU;
//   k_linear_fwd_dual   the same tile code for 256 x 256 tiles and, in the same grid, 256 x 128 tiles for layers
//                       whose last round of 256 x 256 tiles would fill at most half of the CUs;
//   k_linear_fwd_pair   256 x 128 tiles by 4 waves with the same share each, two workgroups per CU;
//   k_linear_fwd_tile   128 x 128 down to 32 x 32 tiles on the 32 x 32 instruction, with the contraction split over
//                       groups of waves where there are few tiles;
//   k_linear_fwd_dual128 128 x 128 tiles and 128 x 64 halves in one grid, for little more than one tile per CU;
//   k_linear_fwd_skinny 16 x 16 tiles straight from memory to registers, for decode batches.
// Operand tiles travel L2 -> LDS directly (buffer_load ... lds, no staging registers) into rings of
// LDS slots.  What limits all of them is the L1 of the CU: it keeps 64 line requests in flight, and a
// request takes 400 - 500 clocks under load, so a CU receives about 20 B/clk (measured; a 256 x 256
// k-step needs 50 KiB per 1024 MFMA clocks).
// The packed weight is stored in memory in the order the sparse MFMA consumes it (1 KiB blocks of
// 16 rows x one k-step, one 16-byte slot per lane), so its loads are contiguous and its fragment
// reads are lane-contiguous.  For X, whose 64 lanes of a load land on consecutive LDS addresses, bank
// conflicts are avoided by choosing WHICH 16-byte piece each lane fetches: piece c of row r is stored
// at position c ^ ((r / 2) % 8), which makes every fragment read (16 rows x one piece) hit 16
// different 16-byte bank groups.
// The loads are written in inline assembly: the compiler otherwise orders every later LDS read
// behind ALL outstanding LDS-writing loads, which would drain the ring each k-step.  Their
// completion is tracked by hand with s_waitcnt vmcnt(n) + a workgroup barrier.
// The epilogue transposes the accumulators through LDS so that each lane stores 16 contiguous bytes
// and each wave writes whole 256-byte rows of Z.
// Workgroups are numbered so that each XCD (the chip routes consecutive workgroup ids to its 8 XCDs
// in turn) works on a contiguous range of tiles, o-tiles fastest: the packed weight stays in that
// XCD's L2 and an X tile is fetched from HBM once per XCD.
#include "common.h"
#include "tile_order.h"

#include <stdio.h>

namespace sste {

namespace {
constexpr int NUM_CU = 256;

}  // namespace

// Output side of the forward GEMMs.  z8 == nullptr: Z is bf16, value = acc * scale.  Otherwise Z is e4m3
// with its own per-tensor scale folded into `scale` by the host (Sec. 5.2: the output of an FP8 layer is
// rescaled per tensor and cast; the consumer multiplies by z_scale again).  amax_bits, if given,
// receives max |acc| * amax_scale over the whole tensor (float32 bits; non-negative floats order like
// their patterns): one atomic per workgroup, skipped when it cannot raise the value.
struct FwdOut {
  uint16_t* z16;          // bf16 output (ZF8 = false); with `act`: the pre-activation H, may then be null
  uint8_t* z8;            // e4m3 output (ZF8 = true)
  int64_t ldz;            // leading dimension in elements
  float scale;            // acc -> stored value (before rounding)
  float amax_scale;       // acc -> the tensor's real units
  uint32_t* amax_bits;    // nullable
  // activation fused into the bf16 epilogue (kernels instantiated with ZF8 = false, AMAX = false):
  // H = RNE_bf16(acc * scale) goes to z16 (if given), A = GELU(H) to a16 (bf16) or a8 (e4m3 of A * a_inv_scale);
  // with a8 the largest |A| goes to amax_bits.
  int act;                // 0: none
  uint16_t* a16;
  uint8_t* a8;
  int64_t lda;
  float a_inv_scale;
  // A is the next product's operand: written with the streaming hint only where it is larger than half of the 256 MB cache, from which that
  // product otherwise reads it, and in bf16 only.  Against the hint everywhere (us): two layers 1280 -> 5120 -> 1280 forward, bf16 2048 tokens 64.7 -> 53.7,
  // 333 tokens of width 768 17.1 -> 15.5, e4m3 1021 tokens 30.3 -> 26.9; with the backward pass, which reads A once more, bf16 width 1024, 4096 tokens
  // 239.5 -> 228, 8192 tokens 403 -> 391.5, 16384 tokens (128 MiB of A) 675 -> 666; e4m3 width 1280, 32768 tokens (160 MiB, the largest) 1368 -> 1360.
  // The product that writes A takes up to 20 % longer by itself without the hint, and the one that reads it less.  Both together, 78 random pairs:
  // up to 100 MB of A between 0.7 % slower and 32 % faster (7 % on the mean), 100 ... 134 MB between 4 % slower and 13 % faster (1 %).
  int a_stream;
};

// Activation stage of the epilogue on one 16-byte piece (8 consecutive channels of one token): stores A in
// the requested format and returns max |A| of the piece (float32 bits; NaN where a value is NaN, whose bits lie above every number's).
__device__ __forceinline__ uint32_t fwd_act_piece(const uint4& h, const FwdOut& out, int64_t t, int64_t o) {
  const uint32_t w[4] = {h.x, h.y, h.z, h.w};
  float a[8], m = 0.0f;
#pragma unroll
  for (int e = 0; e < 4; e++) {
    a[2 * e] = gelu_tanh(bf16lo_f32(w[e]));
    a[2 * e + 1] = gelu_tanh(bf16hi_f32(w[e]));
  }
  if (out.a8) {
    // two values per three-operand maximum, their absolute values as source modifiers; of the two float maxima the one that keeps NaN
#pragma unroll
    for (int e = 0; e < 8; e += 2)
      m = __builtin_elementwise_maximum(__builtin_elementwise_maximum(m, __builtin_fabsf(a[e])), __builtin_fabsf(a[e + 1]));
    const float r = out.a_inv_scale;
    int lo = __builtin_amdgcn_cvt_pk_fp8_f32(clamp448(a[0] * r), clamp448(a[1] * r), 0, false);
    lo = __builtin_amdgcn_cvt_pk_fp8_f32(clamp448(a[2] * r), clamp448(a[3] * r), lo, true);
    int hi = __builtin_amdgcn_cvt_pk_fp8_f32(clamp448(a[4] * r), clamp448(a[5] * r), 0, false);
    hi = __builtin_amdgcn_cvt_pk_fp8_f32(clamp448(a[6] * r), clamp448(a[7] * r), hi, true);
    i32x2 v = {lo, hi};
    *(i32x2*)(out.a8 + t * out.lda + o) = v;
  } else {
    uint4 v = make_uint4(bf16_rne_pack(a[0], a[1]), bf16_rne_pack(a[2], a[3]), bf16_rne_pack(a[4], a[5]), bf16_rne_pack(a[6], a[7]));
    if (out.a_stream) store_stream_b128(out.a16 + t * out.lda + o, v);
    else *(uint4*)(out.a16 + t * out.lda + o) = v;
  }
  return f2u(m);
}

// max |acc| of the calling workgroup (NW waves) -> *amax_bits.  `red` is NW dwords of LDS nobody else uses
// between the two barriers.
template <int NW>
__device__ __forceinline__ void publish_tile_amax(uint32_t m, float amax_scale, uint32_t* __restrict__ amax_bits, uint32_t* red) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) m = max(m, (uint32_t)__shfl_xor((int)m, off, 64));
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = m;
  __syncthreads();
  if (threadIdx.x == 0) {
#pragma unroll
    for (int w = 1; w < NW; w++) m = max(m, red[w]);
    const uint32_t v = f2u(u2f(m) * amax_scale);
    if (v > __hip_atomic_load(amax_bits, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicMax(amax_bits, v);
  }
  __syncthreads();
}

__global__ void k_fill_u32_fwd(uint32_t* p, uint32_t v) { *p = v; }

// ---------------------------------------------------------------------------------------------------------
// Software-pipelined variant: 8 waves (2 x 4), each owning MI_ x NI_ MFMA tiles, so a workgroup covers
// 32 MI_ channels x 64 NI_ tokens (256 x 256, 192 x 256, ...).  Instead of
// alternating, workgroup-wide, between a phase that reads fragments from LDS and a phase that issues MFMAs, the
// three pipes (vector memory, LDS, matrix) run side by side within a k-step:
//   * X fragments are double-buffered in registers: while the MFMAs of k-step s run on one set, the
//     set for k-step s + 1 is read from LDS, spread over the groups of NI_ MFMAs;
//   * packed-weight fragments roll through a two-deep register buffer, one row block ahead of its use;
//   * the direct-to-LDS loads of a k-step are spread over the groups instead of issued in one burst.
// Weight and X tiles live in separate three-slot rings because their LDS lifetimes differ: X of
// k-step s is consumed during k-step s - 1, the weight tile of k-step s during s - 1 (row block 0)
// and s.  At the single barrier of k-step s the tiles of s + 1 must have landed; the loads issued
// during s are the weight tile of s + 2 and the X tile of s + 3.
// Every wave issues the same number of loads per k-step (the counts in s_waitcnt are compile-time
// constants); where the tile has fewer 1 KiB blocks than 8 waves x loads, the surplus loads address
// blocks past the end of the tile's buffer descriptor and fetch nothing.

// LDS bytes of the output stage of NW waves: 16 NI_ token rows of the wave's 16 MI_ channels each.  The padded row, that of the e4m3 output
// and of the narrow tiles, is the longest.
constexpr int fwd_store_smem(int NW, int MI_, int NI_) { return NW * 16 * NI_ * (32 * MI_ + 16); }

// LDS bytes one tile of the pipelined kernel needs (rings, reused by the epilogue)
template <bool FP8, int MI_, int NI_>
constexpr int fwd_pipe_smem() {
  constexpr int NW = 8, NR = 3, MB = FP8 ? 16 : 8;
  constexpr int LA = (32 * MI_ / 16 + NW - 1) / NW, LM = (32 * MI_ * MB / 256 + NW - 1) / NW;
  constexpr int RING = NR * (NW * LA * 1024 + NW * LM * 256 + 64 * NI_ * 128);
  constexpr int EPI = fwd_store_smem(NW, MI_, NI_);
  return RING > EPI ? RING : EPI;
}

// Output stage of the pipelined tiles: accumulators -> LDS (row = token, the wave's 16 MI_ channels contiguous) -> 16-byte stores.  Waves
// 2 x WN; called behind a barrier, with all LDS bytes of the workgroup free.
template <int LDS, int WN, int MI_, int NI_, bool ZF8, bool AMAX>
__device__ __forceinline__ void fwd_pipe_store(uint8_t* smem, const f32x4 (&acc)[MI_][NI_], int64_t T, int64_t O, const FwdOut& out, int64_t o0,
                                               int64_t t0) {
  constexpr int NW = 2 * WN;
  // row of a token: the wave's channels + pad; bf16 rows of the 256-channel tile are XOR-swizzled instead of padded
  constexpr int EROW = (MI_ == 8 && !ZF8) ? 256 : 32 * MI_ + 16;
  static_assert(NW * 16 * NI_ * EROW <= LDS, "the output stage's rows fit the workgroup's LDS");
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave / WN, wn = wave % WN;
  const int j = lane & 15, q = lane >> 4;
  const float scale = out.scale;
  uint16_t* __restrict__ Z = out.z16;
  const int64_t ldz = out.ldz;
  if (AMAX) {
    // float maxima of magnitudes: the absolute value is a free source modifier and two values go into one
    // three-operand maximum (the accumulators are finite)
    float mf = 0.0f;
#pragma unroll
    for (int mi = 0; mi < MI_; mi++)
#pragma unroll
      for (int ni = 0; ni < NI_; ni++)
#pragma unroll
        for (int r = 0; r < 4; r++) mf = __builtin_fmaxf(mf, __builtin_fabsf(acc[mi][ni][r]));
    publish_tile_amax<NW>(f2u(mf), out.amax_scale, out.amax_bits, (uint32_t*)smem);
  }
  uint8_t* eb = smem + wave * (16 * NI_ * EROW);
  if (ZF8) {
    // e4m3 output: a lane's four values of a tile are four consecutive channels = one dword; a token row of
    // the wave is 16 MI_ bytes
#pragma unroll
    for (int mi = 0; mi < MI_; mi++)
#pragma unroll
      for (int ni = 0; ni < NI_; ni++) {
        int w = __builtin_amdgcn_cvt_pk_fp8_f32(clamp448(acc[mi][ni][0] * scale), clamp448(acc[mi][ni][1] * scale), 0, false);
        w = __builtin_amdgcn_cvt_pk_fp8_f32(clamp448(acc[mi][ni][2] * scale), clamp448(acc[mi][ni][3] * scale), w, true);
        *(int*)(eb + (16 * ni + j) * EROW + 16 * mi + 4 * q) = w;
      }
    constexpr int CHUNKS8 = MI_;                                 // 16-byte chunks (16 channels) per token row
    constexpr int NCH8 = 16 * NI_ * CHUNKS8;
#pragma unroll
    for (int it = 0; it < (NCH8 + 63) / 64; it++) {
      int c = 64 * it + lane;
      if (c < NCH8) {
        int row = c / CHUNKS8, chunk = c % CHUNKS8;
        uint4 v = *(const uint4*)(eb + row * EROW + chunk * 16);
        int64_t t = t0 + 16 * NI_ * wn + row, o = o0 + 16 * MI_ * wm + 16 * chunk;
        if (t < T && o < O) store_stream_b128(out.z8 + t * ldz + o, v);
      }
    }
    return;
  }
#pragma unroll
  for (int mi = 0; mi < MI_; mi++)
#pragma unroll
    for (int ni = 0; ni < NI_; ni++) {
      uint2 v;
      v.x = bf16_rne_pack(acc[mi][ni][0] * scale, acc[mi][ni][1] * scale);
      v.y = bf16_rne_pack(acc[mi][ni][2] * scale, acc[mi][ni][3] * scale);
      // 16-byte chunk c of token row t sits at position c ^ (t % 16) (MI_ == 8: a row is 256 B = every bank once,
      // and the padding is not needed): the four-row reads below then run at the full LDS rate, where rows
      // shifted by the 16-byte pad cost half as much again (measured 567 vs 860 clocks per 128 KiB)
      if (MI_ == 8) *(uint2*)(eb + (16 * ni + j) * EROW + (((2 * mi + (q >> 1)) ^ j) * 16) + 8 * (q & 1)) = v;
      else *(uint2*)(eb + (16 * ni + j) * EROW + (16 * mi + 4 * q) * 2) = v;
    }
  // same-wave LDS accesses are ordered; no barrier needed for a wave-private region
  constexpr int CHUNKS = 2 * MI_;                                // 16-byte chunks per token row
  constexpr int NCH = 16 * NI_ * CHUNKS;
  uint32_t act_max = 0;
#pragma unroll
  for (int it = 0; it < (NCH + 63) / 64; it++) {
    int c = 64 * it + lane;
    if (c < NCH) {
      int row = c / CHUNKS, chunk = c % CHUNKS;
      uint4 v = *(const uint4*)(eb + row * EROW + (MI_ == 8 ? (chunk ^ (row & 15)) : chunk) * 16);
      int64_t t = t0 + 16 * NI_ * wn + row, o = o0 + 16 * MI_ * wm + 8 * chunk;
      if (t < T && o < O) {
        if (Z) store_stream_b128(Z + t * ldz + o, v);
        if (out.act) act_max = max(act_max, fwd_act_piece(v, out, t, o));
      }
    }
  }
  if (out.act && out.amax_bits) {           // uniform over the workgroup
    __syncthreads();                        // every wave is done with its part of the LDS
    publish_tile_amax<NW>(act_max, 1.0f, out.amax_bits, (uint32_t*)smem);
  }
}

// One output tile: channels [o0, o0 + 32 MI_) x tokens [t0, t0 + 64 NI_).  `smem` is the workgroup's LDS.
template <bool FP8, int MI_, int NI_, bool ZF8, bool AMAX>
__device__ __forceinline__ void fwd_pipe_tile(uint8_t* smem, const uint8_t* __restrict__ X, int64_t T, int64_t k_bytes,
                                              int64_t ldx_bytes, const uint8_t* __restrict__ vals,
                                              const uint8_t* __restrict__ meta, int64_t O, const FwdOut& out,
                                              int64_t o0, int64_t t0) {
  constexpr int WN = 4, NW = 8, BM = 32 * MI_, BN = 64 * NI_, NR = 3;
  constexpr int MB = FP8 ? 16 : 8, MBLK = 16 * MB;
  constexpr int LA = (BM / 16 + NW - 1) / NW;                    // weight blocks (1 KiB) per wave and k-step
  constexpr int LM = (BM * MB / 256 + NW - 1) / NW;              // 256-byte pieces of position bits
  constexpr int LB = NI_;                                        // 8-token slabs (1 KiB) of X
  constexpr int A_BYTES = NW * LA * 1024, M_BYTES = NW * LM * 256;
  constexpr int ASTAGE = A_BYTES + M_BYTES, BSTAGE = BN * 128;
  constexpr int NLOAD = LA + LM + LB;                            // issue order inside a k-step: A.., M.., B..
  constexpr int NPIECE = 2 * NI_;                                // 16-byte pieces of the next X fragments
  static_assert(NR * (ASTAGE + BSTAGE) <= fwd_pipe_smem<FP8, MI_, NI_>(), "LDS size helper out of step with the tile layout");
  uint8_t* const smemA = smem;
  uint8_t* const smemB = smem + NR * ASTAGE;

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / WN, wn = wave % WN;
  const int j = lane & 15, q = lane >> 4;
  const int nsteps = (int)(k_bytes / 128);

  const int64_t rblk0 = o0 / 16, rbn = (O + 15) / 16;
  const int blks_a = (int)((rbn - rblk0) < BM / 16 ? (rbn - rblk0) : BM / 16);
  const int rows_b = (int)((T - t0) < BN ? (T - t0) : BN);
  const i32x4 ba = rsrc_words(vals + rblk0 * nsteps * 1024, (uint32_t)(blks_a * nsteps * 1024));
  const i32x4 bm = rsrc_words(meta + rblk0 * nsteps * MBLK, (uint32_t)(blks_a * nsteps * MBLK));
  const i32x4 bb = rsrc_words(X + t0 * ldx_bytes, (uint32_t)((rows_b - 1) * ldx_bytes + k_bytes));

  uint32_t offa[LA], offb[LB], offm[LM];
#pragma unroll
  for (int i = 0; i < LA; i++) offa[i] = (uint32_t)((LA * wave + i) * nsteps * 1024 + lane * 16);
#pragma unroll
  for (int i = 0; i < LB; i++) {
    int wl = LB * wave + i;
    int r = 8 * wl + (lane >> 3), c = (lane & 7) ^ ((r >> 1) & 7);
    offb[i] = (uint32_t)(r * ldx_bytes + c * 16);
  }
#pragma unroll
  for (int i = 0; i < LM; i++) {
    int d = 64 * (LM * wave + i) + lane;
    offm[i] = (uint32_t)((d / (MBLK / 4)) * nsteps * MBLK + 4 * (d % (MBLK / 4)));
  }
  const uint32_t ldsA = (uint32_t)(uintptr_t)(lds_u8*)smemA;
  const uint32_t ldsB = (uint32_t)(uintptr_t)(lds_u8*)smemB;
  constexpr uint32_t DEAD = 0x40000000u;            // scalar offset past every descriptor: the load fetches nothing

  // load number n (0 .. NLOAD-1) of this wave for weight k-step sa -> slot slot_a, X k-step sb -> slot slot_b
#define PIPE_LOAD(n, sa, slot_a, sb, slot_b)                                                              \
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
               offb[(n) >= LA + LM ? (n) - LA - LM : 0], (sb) < nsteps ? (uint32_t)(sb) * 128u : DEAD);   \
  } while (0)

  f32x4 acc[MI_][NI_];
#pragma unroll
  for (int a = 0; a < MI_; a++)
#pragma unroll
    for (int b = 0; b < NI_; b++) acc[a][b] = (f32x4){0.f, 0.f, 0.f, 0.f};

  const uint32_t fa_off = (uint32_t)(MI_ * wm * 1024 + lane * 16);                  // + 1024 mi
  const uint32_t fm_off = (uint32_t)(A_BYTES + MI_ * wm * MBLK + lane * (MB / 4));  // + MBLK mi
  const int rb0 = 16 * NI_ * wn + j;                                                // + 16 ni
  const int cb0 = q ^ ((j >> 1) & 7);
  const uint32_t fb_off0 = (uint32_t)(rb0 * 128 + cb0 * 16);
  const uint32_t fb_off1 = (uint32_t)(rb0 * 128 + (cb0 ^ 4) * 16);

  // prologue: weight tiles 0, 1 and X tiles 0, 1, 2 in flight, in the order the barriers expect
#pragma unroll
  for (int n = 0; n < NLOAD; n++) PIPE_LOAD(n, 0, 0, 0, 0);
#pragma unroll
  for (int n = 0; n < NLOAD; n++) PIPE_LOAD(n, 1, 1, 1, 1);
#pragma unroll
  for (int n = LA + LM; n < NLOAD; n++) PIPE_LOAD(n, 0, 0, 2, 2);

  uint4 fb0[NI_][2], fb1[NI_][2];     // X fragments: current / next k-step, roles swap every k-step
  uint4 fa[2];                        // packed-weight fragment of row block mi in fa[mi % 2]
  int fidx[2];
  wait_vmcnt<LA + LM + 2 * LB>();     // tiles of k-step 0 have landed
  __syncthreads();
#pragma unroll
  for (int ni = 0; ni < NI_; ni++) {
    fb0[ni][0] = *(const uint4*)(smemB + fb_off0 + ni * 2048);
    fb0[ni][1] = *(const uint4*)(smemB + fb_off1 + ni * 2048);
  }
  fa[0] = *(const uint4*)(smemA + fa_off);
  if (FP8) fidx[0] = *(const int*)(smemA + fm_off);
  else fidx[0] = *(const uint16_t*)(smemA + fm_off);

  int s0 = 0, s1 = 1, s2 = 2;         // ring slots of k-steps step, step + 1, step + 2 (both rings)

  // one k-step: MFMAs on BC, next X fragments into BX
#define PIPE_STEP(BC, BX)                                                                                 \
  do {                                                                                                    \
    wait_vmcnt<LB>();                 /* all but the newest X tile: k-step step + 1 has landed */          \
    __syncthreads();                  /* ... for every wave; slots of step - 1 (weights) and step (X) are free */ \
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
        if (spread(pc, NPIECE, MI_) == mi)                                                                \
          BX[pc >> 1][pc & 1] = *(const uint4*)(pb1 + ((pc & 1) ? fb_off1 : fb_off0) + (pc >> 1) * 2048); \
      _Pragma("unroll") for (int n = 0; n < NLOAD; n++)                                                   \
        if (spread(n, NLOAD, MI_) == mi) PIPE_LOAD(n, step + 2, s2, step + 3, s0);                        \
      _Pragma("unroll") for (int ni = 0; ni < NI_; ni++) {                                                \
        if (FP8) {                                                                                        \
          i32x4 av;                                                                                       \
          i32x8 bv;                                                                                       \
          __builtin_memcpy(&av, &fa[mi & 1], 16);                                                         \
          __builtin_memcpy(&bv, &BC[ni][0], 32);                                                          \
          acc[mi][ni] = __builtin_amdgcn_smfmac_f32_16x16x128_fp8_fp8(av, bv, acc[mi][ni], fidx[mi & 1], 0, 0); \
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
    PIPE_STEP(fb0, fb1);
    step++;
    PIPE_STEP(fb1, fb0);
    step--;
  }
  if (step < nsteps) PIPE_STEP(fb0, fb1);
#undef PIPE_STEP
#undef PIPE_LOAD

  wait_vmcnt<0>();
  __syncthreads();
  fwd_pipe_store<fwd_pipe_smem<FP8, MI_, NI_>(), WN, MI_, NI_, ZF8, AMAX>(smem, acc, T, O, out, o0, t0);
}

// ---------------------------------------------------------------------------------------------------------
// The same wave tile in workgroups of 2 x WN = 4 waves, 256 channels x 128 tokens, two workgroups per CU: one workgroup's prologue and
// output stage run beside the other's k-steps.  Two slots per operand.  The one barrier of a k-step stands before its last group of
// MFMAs, whose fragments are in registers by then: behind it the weight tile of this k-step and the X tile of the next one (read into
// registers during this one) are free, and what was requested behind the last barrier -- the weight tile of the next k-step, the X tile of the one
// after -- is complete.  Fetches a third more bytes per result than 256 x 256 tiles and is slower than those on long contractions.
// On the 16 x 16 instruction, which takes less power per result than the 32 x 32 one of k_linear_fwd_tile's 256 x 128 tile, whose place it took
// (us, old -> this / 256 x 256 tiles or the two-shape grid; T x O x I): e4m3 32768 x 5120 x 1280 168.7 -> 159.9 / 158.3, 32768 x 3840 x 1280 119.2 ->
// 117.9 / 118.0; bf16 16384 x 3840 x 1280 103.5 -> 95.4 / 93.5, 16384 x 5120 x 1280 136.1 -> 128.1 / 124.6, 8192 x 3072 x 768 30.3 -> 30.6 / 28.7.
template <bool FP8, int WN, int MI_, int NI_>
constexpr int fwd_pair_smem() {
  constexpr int NW = 2 * WN, MB = FP8 ? 16 : 8;
  constexpr int RING = 2 * (32 * MI_ * (64 + MB) + 16 * NI_ * WN * 128);
  constexpr int EPI = fwd_store_smem(NW, MI_, NI_);
  return RING > EPI ? RING : EPI;
}

template <bool FP8, int WN, int MI_, int NI_, bool ZF8, bool AMAX>
__device__ __forceinline__ void fwd_pair_tile(uint8_t* smem, const uint8_t* __restrict__ X, int64_t T, int64_t k_bytes, int64_t ldx_bytes,
                                              const uint8_t* __restrict__ vals, const uint8_t* __restrict__ meta, int64_t O, const FwdOut& out,
                                              int64_t o0, int64_t t0) {
  constexpr int NW = 2 * WN, BM = 32 * MI_, BN = 16 * NI_ * WN;
  constexpr int MB = FP8 ? 16 : 8, MBLK = 16 * MB;
  constexpr int LA = BM / 16 / NW, LM = BM * MB / 256 / NW, LB = BN / 8 / NW;
  constexpr int A_BYTES = BM * 64, ASTAGE = A_BYTES + BM * MB, BSTAGE = BN * 128;
  constexpr int NLOAD = LA + LM + LB, NPIECE = 2 * NI_;
  static_assert(LA * NW * 16 == BM && LM * NW * 256 == BM * MB && LB * NW * 8 == BN, "loads per wave");
  constexpr int LG = 4;                             // groups behind the barrier that the loads are spread over
  static_assert(2 * (ASTAGE + BSTAGE) <= fwd_pair_smem<FP8, WN, MI_, NI_>(), "LDS size helper out of step with the tile layout");
  uint8_t* const smemA = smem;
  uint8_t* const smemB = smem + 2 * ASTAGE;

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / WN, wn = wave % WN;
  const int j = lane & 15, q = lane >> 4;
  const int nsteps = (int)(k_bytes / 128);

  const int64_t rblk0 = o0 / 16, rbn = (O + 15) / 16;
  const int blks_a = (int)((rbn - rblk0) < BM / 16 ? (rbn - rblk0) : BM / 16);
  const int rows_b = (int)((T - t0) < BN ? (T - t0) : BN);
  const i32x4 ba = rsrc_words(vals + rblk0 * nsteps * 1024, (uint32_t)(blks_a * nsteps * 1024));
  const i32x4 bm = rsrc_words(meta + rblk0 * nsteps * MBLK, (uint32_t)(blks_a * nsteps * MBLK));
  const i32x4 bb = rsrc_words(X + t0 * ldx_bytes, (uint32_t)((rows_b - 1) * ldx_bytes + k_bytes));
  uint32_t offa[LA], offb[LB], offm[LM];
#pragma unroll
  for (int i = 0; i < LA; i++) offa[i] = (uint32_t)((LA * wave + i) * nsteps * 1024 + lane * 16);
#pragma unroll
  for (int i = 0; i < LB; i++) {
    const int r = 8 * (LB * wave + i) + (lane >> 3), c = (lane & 7) ^ ((r >> 1) & 7);
    offb[i] = (uint32_t)(r * ldx_bytes + c * 16);
  }
#pragma unroll
  for (int i = 0; i < LM; i++) {
    const int d = 64 * (LM * wave + i) + lane;
    offm[i] = (uint32_t)((d / (MBLK / 4)) * nsteps * MBLK + 4 * (d % (MBLK / 4)));
  }
  const uint32_t ldsA = (uint32_t)(uintptr_t)(lds_u8*)smemA;
  const uint32_t ldsB = (uint32_t)(uintptr_t)(lds_u8*)smemB;
  constexpr uint32_t DEAD = 0x40000000u;            // scalar offset past every descriptor: the load fetches nothing
  // load n (0 .. LA + LM - 1: weight of k-step sa into slot pa, then X of k-step sb into slot pb)
#define PAIR_LOAD(n, sa, pa_, sb, pb_)                                                                       \
  do {                                                                                                    \
    if ((n) < LA)                                                                                         \
      dma_b128(ba, ldsA + (uint32_t)(pa_) * ASTAGE + (LA * wave + (n)) * 1024, offa[(n) < LA ? (n) : 0],    \
               (sa) < nsteps ? (uint32_t)(sa) * 1024u : DEAD);                                            \
    else if ((n) < LA + LM)                                                                               \
      dma_b32(bm, ldsA + (uint32_t)(pa_) * ASTAGE + A_BYTES + (LM * wave + ((n) - LA)) * 256,               \
              offm[((n) >= LA && (n) < LA + LM) ? (n) - LA : 0],                                          \
              (sa) < nsteps ? (uint32_t)(sa) * (uint32_t)MBLK : DEAD);                                    \
    else                                                                                                  \
      dma_b128(bb, ldsB + (uint32_t)(pb_) * BSTAGE + (LB * wave + ((n) - LA - LM)) * 1024,                  \
               offb[(n) >= LA + LM ? (n) - LA - LM : 0], (sb) < nsteps ? (uint32_t)(sb) * 128u : DEAD);   \
  } while (0)

  f32x4 acc[MI_][NI_];
#pragma unroll
  for (int a = 0; a < MI_; a++)
#pragma unroll
    for (int b = 0; b < NI_; b++) acc[a][b] = (f32x4){0.f, 0.f, 0.f, 0.f};

  const uint32_t fa_off = (uint32_t)(MI_ * wm * 1024 + lane * 16);                  // + 1024 mi
  const uint32_t fm_off = (uint32_t)(A_BYTES + MI_ * wm * MBLK + lane * (MB / 4));  // + MBLK mi
  const int rb0 = 16 * NI_ * wn + j;                                                // + 16 ni
  const int cb0 = q ^ ((j >> 1) & 7);
  const uint32_t fb_off0 = (uint32_t)(rb0 * 128 + cb0 * 16);
  const uint32_t fb_off1 = (uint32_t)(rb0 * 128 + (cb0 ^ 4) * 16);

#pragma unroll
  for (int n = 0; n < NLOAD; n++) PAIR_LOAD(n, 0, 0, 0, 0);
#pragma unroll
  for (int n = LA + LM; n < NLOAD; n++) PAIR_LOAD(n, 0, 0, 1, 1);
  uint4 fb0[NI_][2], fb1[NI_][2];     // X fragments: current / next k-step, roles swap every k-step
  uint4 fa[2];                        // packed-weight fragment of row block mi in fa[mi % 2]
  int fidx[2];
  wait_vmcnt<0>();
  __syncthreads();
#pragma unroll
  for (int ni = 0; ni < NI_; ni++) {
    fb0[ni][0] = *(const uint4*)(smemB + fb_off0 + ni * 2048);
    fb0[ni][1] = *(const uint4*)(smemB + fb_off1 + ni * 2048);
  }
  fa[0] = *(const uint4*)(smemA + fa_off);
  if (FP8) fidx[0] = *(const int*)(smemA + fm_off);
  else fidx[0] = *(const uint16_t*)(smemA + fm_off);
  __syncthreads();                    // X tile 0 has been read
#pragma unroll
  for (int n = 0; n < NLOAD; n++)
    if (spread(n, NLOAD, LG) == 0) PAIR_LOAD(n, 1, 1, 2, 0);

  // one k-step of parity P: MFMAs on BC, next X fragments into BX
#define PAIR_STEP(BC, BX, P)                                                                              \
  do {                                                                                                    \
    const uint8_t* pa = smemA + (P) * ASTAGE;                                                             \
    const uint8_t* pa1 = smemA + (1 - (P)) * ASTAGE;                                                      \
    const uint8_t* pb1 = smemB + (1 - (P)) * BSTAGE;                                                      \
    _Pragma("unroll") for (int mi = 0; mi < MI_; mi++) {                                                  \
      if (mi == MI_ - 1) {                                                                                \
        wait_vmcnt<0>();              /* weight tile step + 1 and X tile step + 2 have landed ... */       \
        __syncthreads();              /* ... for every wave; weight tile step and X tile step + 1 have been read */ \
      }                                                                                                   \
      const uint8_t* an = mi < MI_ - 1 ? pa + (mi + 1) * 1024 : pa1;                                      \
      const uint8_t* mn = mi < MI_ - 1 ? pa + (mi + 1) * MBLK : pa1;                                      \
      fa[(mi + 1) & 1] = *(const uint4*)(an + fa_off);                                                    \
      if (FP8) fidx[(mi + 1) & 1] = *(const int*)(mn + fm_off);                                           \
      else fidx[(mi + 1) & 1] = *(const uint16_t*)(mn + fm_off);                                          \
      _Pragma("unroll") for (int pc = 0; pc < NPIECE; pc++)                                               \
        if (spread(pc, NPIECE, MI_ - 1) == mi)                                                            \
          BX[pc >> 1][pc & 1] = *(const uint4*)(pb1 + ((pc & 1) ? fb_off1 : fb_off0) + (pc >> 1) * 2048); \
      _Pragma("unroll") for (int n = 0; n < NLOAD; n++) {                                                 \
        if (mi == MI_ - 1 && spread(n, NLOAD, LG) == 0) PAIR_LOAD(n, step + 2, P, step + 3, 1 - (P));       \
        if (mi < MI_ - 1 && spread(n, NLOAD, LG) == mi + 1) PAIR_LOAD(n, step + 1, 1 - (P), step + 2, P);   \
      }                                                                                                   \
      _Pragma("unroll") for (int ni = 0; ni < NI_; ni++) {                                                \
        if (FP8) {                                                                                        \
          i32x4 av;                                                                                       \
          i32x8 bv;                                                                                       \
          __builtin_memcpy(&av, &fa[mi & 1], 16);                                                         \
          __builtin_memcpy(&bv, &BC[ni][0], 32);                                                          \
          acc[mi][ni] = __builtin_amdgcn_smfmac_f32_16x16x128_fp8_fp8(av, bv, acc[mi][ni], fidx[mi & 1], 0, 0); \
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
  } while (0)

  int step = 0;
  for (; step + 1 < nsteps; step += 2) {
    PAIR_STEP(fb0, fb1, 0);
    step++;
    PAIR_STEP(fb1, fb0, 1);
    step--;
  }
  if (step < nsteps) PAIR_STEP(fb0, fb1, 0);
#undef PAIR_STEP
#undef PAIR_LOAD
  wait_vmcnt<0>();
  __syncthreads();
  fwd_pipe_store<fwd_pair_smem<FP8, WN, MI_, NI_>(), WN, MI_, NI_, ZF8, AMAX>(smem, acc, T, O, out, o0, t0);
}

template <bool FP8, int WN, int MI_, int NI_, bool ZF8, bool AMAX>
__global__ void __launch_bounds__(128 * WN, 2)
k_linear_fwd_pair(const uint8_t* __restrict__ X, int64_t T, int64_t k_bytes, int64_t ldx_bytes,
                  const uint8_t* __restrict__ vals, const uint8_t* __restrict__ meta, int64_t O, FwdOut out, int m_tiles) {
  __shared__ __align__(1024) uint8_t smem[fwd_pair_smem<FP8, WN, MI_, NI_>()];
  const int logical = xcd_contiguous(blockIdx.x, gridDim.x);
  const int tm = logical % m_tiles, tn = logical / m_tiles;
  fwd_pair_tile<FP8, WN, MI_, NI_, ZF8, AMAX>(smem, X, T, k_bytes, ldx_bytes, vals, meta, O, out, (int64_t)tm * (32 * MI_),
                                              (int64_t)tn * (16 * NI_ * WN));
}

// ---------------------------------------------------------------------------------------------------------
// Small and middle problems: 32 WM MT channels x 32 WN NT tokens by KG groups of WM x WN waves on the 32 x 32 sparse instructions
// (v_smfmac_f32_32x32x32_bf16 / 32x32x64_fp8_fp8, two per k-step).  Group kg takes the k-steps kg, kg + KG, ... through LDS slots
// of its own and the groups' sums are added at the end: such problems have too few tiles to fill the chip and are bound by the time
// a k-step's loads take to arrive, so it is loads in flight that count (NS slots per group, KG groups, several workgroups per CU).
// The only barrier of a k-step stands before its second half, whose fragments are in registers by then: behind it the slot
// of this k-step is free, the next tile is complete, and its first fragments are read under the second half's MFMAs.
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;

template <bool FP8, int WM, int WN, int MT, int NT, int KG, int NS>
constexpr int fwd_tile_smem() {
  constexpr int NWG = WM * WN, MB = FP8 ? 16 : 8;
  constexpr int LM = (32 * WM * MT * MB / 256 + NWG - 1) / NWG;
  constexpr int RING = KG * NS * (32 * WM * MT * 64 + NWG * LM * 256 + 32 * WN * NT * 128);
  constexpr int EPI = NWG * 32 * NT * (64 * MT + 16);
  constexpr int RED = (KG - 1) * NWG * MT * NT * 4096;
  constexpr int M1 = RING > EPI ? RING : EPI;
  return M1 > RED ? M1 : RED;
}

// One output tile: channels [32 WM MT tm, ...) x tokens [t0, t0 + 32 WN NT).
template <bool FP8, int WM, int WN, int MT, int NT, int KG, int NS, bool ZF8, bool AMAX>
__device__ __forceinline__ void fwd_tile(uint8_t* smem, const uint8_t* __restrict__ X, int64_t T, int64_t k_bytes, int64_t ldx_bytes,
                                         const uint8_t* __restrict__ vals, const uint8_t* __restrict__ meta, int64_t O, const FwdOut& out, int tm,
                                         int64_t t0) {
  constexpr int NWG = WM * WN, NW = NWG * KG;
  constexpr int BM = 32 * WM * MT, BN = 32 * WN * NT;
  constexpr int MB = FP8 ? 16 : 8, MBLK = 16 * MB;
  constexpr int LA = BM / 16 / NWG, LB = BN / 8 / NWG, LM = (BM * MB / 256 + NWG - 1) / NWG;   // loads per wave and k-step
  constexpr int LPW = LA + LB + LM;
  constexpr int A_BYTES = BM * 64, M_BYTES = NWG * LM * 256, SLOT = A_BYTES + M_BYTES + BN * 128;
  static_assert(LA >= 1 && LB >= 1, "tile too small for this many waves");

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave_all = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int kg = KG > 1 ? wave_all / NWG : 0, wave = KG > 1 ? wave_all % NWG : wave_all;
  const int wm = wave / WN, wn = wave % WN;
  const int n = lane & 31, hh = lane >> 5;
  const int64_t o0 = (int64_t)tm * BM;
  const int nsteps = (int)(k_bytes / 128);
  const int nloc = (nsteps + KG - 1) / KG;
  uint8_t* const ring = smem + kg * NS * SLOT;
  const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_u8*)ring;

  const int64_t rblk0 = o0 / 16, rbn = (O + 15) / 16;
  const int blks_a = (int)((rbn - rblk0) < BM / 16 ? (rbn - rblk0) : BM / 16);
  const int rows_b = (int)((T - t0) < BN ? (T - t0) : BN);
  const i32x4 ba = rsrc_words(vals + rblk0 * nsteps * 1024, (uint32_t)(blks_a * nsteps * 1024));
  const i32x4 bm = rsrc_words(meta + rblk0 * nsteps * MBLK, (uint32_t)(blks_a * nsteps * MBLK));
  const i32x4 bb = rsrc_words(X + t0 * ldx_bytes, (uint32_t)((rows_b - 1) * ldx_bytes + k_bytes));
  uint32_t offa[LA], offb[LB], offm[LM];
#pragma unroll
  for (int i = 0; i < LA; i++) offa[i] = (uint32_t)((LA * wave + i) * nsteps * 1024 + lane * 16);
#pragma unroll
  for (int i = 0; i < LB; i++) {
    const int r = 8 * (LB * wave + i) + (lane >> 3), c = (lane & 7) ^ ((r >> 1) & 7);
    offb[i] = (uint32_t)(r * ldx_bytes + c * 16);
  }
#pragma unroll
  for (int i = 0; i < LM; i++) {
    const int d = 64 * (LM * wave + i) + lane;
    offm[i] = (uint32_t)((d / (MBLK / 4)) * nsteps * MBLK + 4 * (d % (MBLK / 4)));
  }
  // k-step number ls of this group into slot `slot`; past the last one the loads are pushed out of range (zeros arrive: such a step
  // adds nothing), so that the same number is always in flight
  auto issue = [&](int ls, int slot) {
    const int st = ls * KG + kg;
    const bool live = st < nsteps;
    const uint32_t sa = live ? (uint32_t)st * 1024u : 0x40000000u, sx = live ? (uint32_t)st * 128u : 0x40000000u;
    const uint32_t sm = live ? (uint32_t)st * (uint32_t)MBLK : 0x40000000u;
    const uint32_t base = lds0 + (uint32_t)slot * SLOT;
#pragma unroll
    for (int i = 0; i < LA; i++) dma_b128(ba, base + (LA * wave + i) * 1024, offa[i], sa);
#pragma unroll
    for (int i = 0; i < LM; i++) dma_b32(bm, base + A_BYTES + (LM * wave + i) * 256, offm[i], sm);
#pragma unroll
    for (int i = 0; i < LB; i++) dma_b128(bb, base + A_BYTES + M_BYTES + (LB * wave + i) * 1024, offb[i], sx);
  };

  f32x16 acc[MT][NT];
#pragma unroll
  for (int m = 0; m < MT; m++)
#pragma unroll
    for (int t = 0; t < NT; t++)
#pragma unroll
      for (int r = 0; r < 16; r++) acc[m][t][r] = 0.f;

  // fragments of half kk of a k-step.  A lane (row n, hh): slot 16 (2 kk + hh) + n % 16 of row block n / 16; B lane (column n, hh):
  // pieces 4 kk + hh and 4 kk + 2 + hh of the token row.
  const uint32_t fa_off = (uint32_t)((2 * wm * MT + (n >> 4)) * 1024 + (16 * hh + (n & 15)) * 16);
  const uint32_t fm_off = (uint32_t)(A_BYTES + (2 * wm * MT + (n >> 4)) * MBLK + (16 * hh + (n & 15)) * (MB / 4));
  const uint32_t fb_row = (uint32_t)(A_BYTES + M_BYTES + (32 * wn * NT + n) * 128), key = (uint32_t)((n >> 1) & 7);
  const uint32_t fb_off[2] = {fb_row + ((hh ^ key) * 16), fb_row + (((4 + hh) ^ key) * 16)};
  uint4 fa[2][MT], fb[2][NT][2];
  int fi[2][MT];
  auto read_frag = [&](int kk, const uint8_t* sl) {
#pragma unroll
    for (int m = 0; m < MT; m++) {
      fa[kk][m] = *(const uint4*)(sl + fa_off + m * 2048 + kk * 512);
      if (FP8) fi[kk][m] = *(const int*)(sl + fm_off + m * 2 * MBLK + kk * 32 * (MB / 4));
      else fi[kk][m] = *(const uint16_t*)(sl + fm_off + m * 2 * MBLK + kk * 32 * (MB / 4));
    }
#pragma unroll
    for (int t = 0; t < NT; t++) {
      fb[kk][t][0] = *(const uint4*)(sl + fb_off[kk] + t * 4096);
      fb[kk][t][1] = *(const uint4*)(sl + (fb_off[kk] ^ 32u) + t * 4096);
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
          acc[m][t] = __builtin_amdgcn_smfmac_f32_32x32x64_fp8_fp8(av, bv, acc[m][t], fi[kk][m], 0, 0);
        } else {
          bf16x8 av;
          bf16x16 bv;
          __builtin_memcpy(&av, &fa[kk][m], 16);
          __builtin_memcpy(&bv, &fb[kk][t][0], 32);
          acc[m][t] = __builtin_amdgcn_smfmac_f32_32x32x32_bf16(av, bv, acc[m][t], fi[kk][m], 0, 0);
        }
      }
  };

  if (nloc > 0) {
#pragma unroll
    for (int k = 0; k < NS; k++) issue(k, k);
    wait_vmcnt<(NS - 1) * LPW>();
    __syncthreads();
    read_frag(0, ring);
  }
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
  }

  // output stage (group 0 holds the sums; the others only take part in the barriers)
  const float scale = out.scale;
  const bool own = KG == 1 || kg == 0;
  if (AMAX) {
    float mf = 0.0f;
    if (own) {
#pragma unroll
      for (int m = 0; m < MT; m++)
#pragma unroll
        for (int t = 0; t < NT; t++)
#pragma unroll
          for (int r = 0; r < 16; r++) mf = __builtin_fmaxf(mf, __builtin_fabsf(acc[m][t][r]));
    }
    publish_tile_amax<NW>(f2u(mf), out.amax_scale, out.amax_bits, (uint32_t*)smem);
  }
  uint32_t act_max = 0;
  if (own) {
    const int64_t tw = t0 + 32 * NT * wn, ow = o0 + 32 * MT * wm;
    if (ZF8) {
      // a lane's registers 4g .. 4g + 3 are four consecutive channels = one dword; padded token rows of 32 MT bytes
      constexpr int EROW = 32 * MT + 16, CH = 2 * MT, NIT = 32 * NT * CH / 64;
      uint8_t* const eb = smem + wave * (32 * NT * EROW);
#pragma unroll
      for (int t = 0; t < NT; t++)
#pragma unroll
        for (int m = 0; m < MT; m++)
#pragma unroll
          for (int g = 0; g < 4; g++) {
            int w = __builtin_amdgcn_cvt_pk_fp8_f32(clamp448(acc[m][t][4 * g] * scale), clamp448(acc[m][t][4 * g + 1] * scale), 0, false);
            w = __builtin_amdgcn_cvt_pk_fp8_f32(clamp448(acc[m][t][4 * g + 2] * scale), clamp448(acc[m][t][4 * g + 3] * scale), w, true);
            *(int*)(eb + (32 * t + n) * EROW + 32 * m + 8 * g + 4 * hh) = w;
          }
#pragma unroll
      for (int it = 0; it < NIT; it++) {
        const int c = 64 * it + lane, row = c / CH, chunk = c % CH;
        const uint4 v = *(const uint4*)(eb + row * EROW + chunk * 16);
        if (tw + row < T && ow + 16 * chunk < O) store_stream_b128(out.z8 + (tw + row) * out.ldz + ow + 16 * chunk, v);
      }
    } else {
      // chunk c of token row t at c ^ key(t), 8-byte halves swapped in rows with bit 4 set: all banks covered both ways
      constexpr int CH = 4 * MT, NIT = 32 * NT * CH / 64;
      uint8_t* const eb = smem + wave * (32 * NT * 64 * MT);
      auto ekey = [](int row) { return (row / (16 / CH)) % CH; };
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
            *(uint2*)(eb + row * (64 * MT) + (((4 * m + g) ^ ekey(row)) * 16) + 8 * (hh ^ (n >> 4))) = v;
          }
#pragma unroll
      for (int it = 0; it < NIT; it++) {
        const int c = 64 * it + lane, row = c / CH, chunk = c % CH;
        uint4 v = *(const uint4*)(eb + row * (64 * MT) + ((chunk ^ ekey(row)) * 16));
        if ((row >> 4) & 1) v = make_uint4(v.z, v.w, v.x, v.y);
        const int64_t t = tw + row, o = ow + 8 * chunk;
        if (t < T && o < O) {
          if (out.z16) store_stream_b128(out.z16 + t * out.ldz + o, v);
          if (out.act) act_max = max(act_max, fwd_act_piece(v, out, t, o));
        }
      }
    }
  }
  if (!ZF8 && out.act && out.amax_bits) {   // uniform over the workgroup
    __syncthreads();
    publish_tile_amax<NW>(act_max, 1.0f, out.amax_bits, (uint32_t*)smem);
  }
}

template <bool FP8, int WM, int WN, int MT, int NT, int KG, int NS, bool ZF8, bool AMAX>
__global__ void __launch_bounds__(64 * WM * WN * KG, 1)
k_linear_fwd_tile(const uint8_t* __restrict__ X, int64_t T, int64_t k_bytes, int64_t ldx_bytes, const uint8_t* __restrict__ vals,
                  const uint8_t* __restrict__ meta, int64_t O, FwdOut out, int m_tiles) {
  __shared__ __align__(1024) uint8_t smem[fwd_tile_smem<FP8, WM, WN, MT, NT, KG, NS>()];
  const int logical = xcd_contiguous(blockIdx.x, gridDim.x);
  fwd_tile<FP8, WM, WN, MT, NT, KG, NS, ZF8, AMAX>(smem, X, T, k_bytes, ldx_bytes, vals, meta, O, out, logical % m_tiles,
                                                   (int64_t)(logical / m_tiles) * (32 * WN * NT));
}

// Two shapes in one grid, two workgroups per CU: 128 x 128 tiles 0 .. n_big - 1, and the others as 128 x 64 halves (fwd_halves says when and why).
template <bool FP8>
constexpr int fwd_dual128_smem() {
  constexpr int BIG = fwd_tile_smem<FP8, 2, 2, 2, 2, 1, 3>(), HALF = fwd_tile_smem<FP8, 2, 2, 2, 1, 1, 4>();
  return BIG > HALF ? BIG : HALF;
}
template <bool FP8, bool ZF8, bool AMAX>
__global__ void __launch_bounds__(256, 2)
k_linear_fwd_dual128(const uint8_t* __restrict__ X, int64_t T, int64_t k_bytes, int64_t ldx_bytes, const uint8_t* __restrict__ vals,
                     const uint8_t* __restrict__ meta, int64_t O, FwdOut out, int m_tiles, int n_big) {
  __shared__ __align__(1024) uint8_t smem[fwd_dual128_smem<FP8>()];
  static_assert(2 * fwd_dual128_smem<FP8>() <= 160 * 1024, "two workgroups per CU");
  const int bid = blockIdx.x;
  if (bid < n_big) {
    const int logical = xcd_contiguous(bid, n_big);
    fwd_tile<FP8, 2, 2, 2, 2, 1, 3, ZF8, AMAX>(smem, X, T, k_bytes, ldx_bytes, vals, meta, O, out, logical % m_tiles, (int64_t)(logical / m_tiles) * 128);
  } else {
    const int h = xcd_contiguous(bid - n_big, (int)gridDim.x - n_big);
    const int tile = n_big + (h >> 1);
    const int64_t t0 = (int64_t)(tile / m_tiles) * 128 + 64 * (h & 1);
    if (t0 >= T) return;                       // second half of a ragged last token tile: nothing to do
    fwd_tile<FP8, 2, 2, 2, 1, 1, 4, ZF8, AMAX>(smem, X, T, k_bytes, ldx_bytes, vals, meta, O, out, tile % m_tiles, t0);
  }
}

// ---------------------------------------------------------------------------------------------------------
// Few tokens (a decode batch): 16 channels x 16 tokens by one workgroup whose KW waves take the k-steps in turn.  The packed
// weight is read once and every wave's operands come straight from memory into its registers (a lane's slot of a packed block and
// two pieces of an X row ARE its fragments): no LDS, no barrier until the waves' sums are added, U k-steps of loads in flight per wave.
// Bound by the load instructions a CU can take: the 16 rows of X cost more than the weight (bf16 1280 x 5120: 4.2 us with one token,
// 7.2 with 16), and so do the k-steps past the end that the last turn of KW * U asks for in vain.  Hence U = 2; us from
// U = 4 to U = 2 (T x O x I): bf16 16x1280x5120 7.50 -> 7.19, 16x768x3072 5.38 -> 5.04, 512x256x1024 5.05 -> 4.33; e4m3 16x1280x5120 5.03 -> 4.69,
// 16x5120x1280 4.29 -> 3.58, 48x3072x768 4.41 -> 3.60.  16 waves, or more k-steps in flight, are slower (8.5 and 8.3 us on the first).
template <bool FP8, int KW, int U, bool ZF8, bool AMAX>
__global__ void __launch_bounds__(64 * KW)
k_linear_fwd_skinny(const uint8_t* __restrict__ X, int64_t T, int64_t k_bytes, int64_t ldx_bytes, const uint8_t* __restrict__ vals,
                    const uint8_t* __restrict__ meta, int64_t O, FwdOut out, int m_tiles) {
  constexpr int MBLK = FP8 ? 256 : 128;
  __shared__ __align__(16) uint8_t smem[KW * 1024];
  __shared__ uint32_t red[KW];
  const int tm = blockIdx.x % m_tiles, tn = blockIdx.x / m_tiles;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int j = lane & 15, q = lane >> 4;
  const int64_t o0 = (int64_t)tm * 16, t0 = (int64_t)tn * 16;
  const int nsteps = (int)(k_bytes / 128);
  const int rows_b = (int)((T - t0) < 16 ? (T - t0) : 16);
  const BufferRsrc ra = make_rsrc(vals + (int64_t)tm * nsteps * 1024, (uint32_t)(nsteps * 1024));
  const BufferRsrc rm = make_rsrc(meta + (int64_t)tm * nsteps * MBLK, (uint32_t)(nsteps * MBLK));
  const BufferRsrc rb = make_rsrc(X + t0 * ldx_bytes, (uint32_t)((rows_b - 1) * ldx_bytes + k_bytes));
  const uint32_t offa = lane * 16, offm = lane * (MBLK / 64), offb = (uint32_t)(j * ldx_bytes + q * 16);

  f32x4 acc = (f32x4){0.f, 0.f, 0.f, 0.f};
  for (int s = wave; s < nsteps; s += KW * U) {
    uint4 fa[U], fb[U][2];
    int fi[U];
#pragma unroll
    for (int u = 0; u < U; u++) {
      // a k-step past the last one reads zeros
      const int st = s + u * KW;
      const bool live = st < nsteps;
      const uint32_t dead = live ? 0u : 0x80000000u;
      const int sc = live ? st : 0;
      fa[u] = buffer_load_b128(ra, offa + dead, (uint32_t)sc * 1024u);
      if (FP8) fi[u] = __builtin_amdgcn_raw_buffer_load_b32(rm, (int)(offm + dead), sc * MBLK, 0);
      else fi[u] = (uint16_t)__builtin_amdgcn_raw_buffer_load_b16(rm, (int)(offm + dead), sc * MBLK, 0);
      const uint32_t o = (j < rows_b ? offb : 0x80000000u) | dead;
      fb[u][0] = buffer_load_b128(rb, o, (uint32_t)sc * 128u);
      fb[u][1] = buffer_load_b128(rb, o + 64u, (uint32_t)sc * 128u);
    }
    __builtin_amdgcn_sched_barrier(0);       // the loads of all U k-steps are requested before the first use
#pragma unroll
    for (int u = 0; u < U; u++) {
      if (FP8) {
        i32x4 av;
        i32x8 bv;
        __builtin_memcpy(&av, &fa[u], 16);
        __builtin_memcpy(&bv, &fb[u][0], 32);
        acc = __builtin_amdgcn_smfmac_f32_16x16x128_fp8_fp8(av, bv, acc, fi[u], 0, 0);
      } else {
        bf16x8 av;
        bf16x16 bv;
        __builtin_memcpy(&av, &fa[u], 16);
        __builtin_memcpy(&bv, &fb[u][0], 32);
        acc = __builtin_amdgcn_smfmac_f32_16x16x64_bf16(av, bv, acc, fi[u], 0, 0);
      }
    }
  }
  *(f32x4*)(smem + wave * 1024 + lane * 16) = acc;
  __syncthreads();
  uint32_t amax = 0;
  if (wave == 0) {
    // wave 0 adds up: a lane's four values are channels 4 q .. 4 q + 3 of token j
    f32x4 v = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < KW; w++) v += *(const f32x4*)(smem + w * 1024 + lane * 16);
    const int64_t t = t0 + j, o = o0 + 4 * q;
    if (AMAX) amax = f2u(__builtin_fmaxf(__builtin_fmaxf(__builtin_fabsf(v[0]), __builtin_fabsf(v[1])), __builtin_fmaxf(__builtin_fabsf(v[2]), __builtin_fabsf(v[3]))));
    if (t < T && o < O) {
      const float sc = out.scale;
      if (ZF8) {
        int w = __builtin_amdgcn_cvt_pk_fp8_f32(clamp448(v[0] * sc), clamp448(v[1] * sc), 0, false);
        w = __builtin_amdgcn_cvt_pk_fp8_f32(clamp448(v[2] * sc), clamp448(v[3] * sc), w, true);
        *(int*)(out.z8 + t * out.ldz + o) = w;
      } else {
        const uint2 h = make_uint2(bf16_rne_pack(v[0] * sc, v[1] * sc), bf16_rne_pack(v[2] * sc, v[3] * sc));
        if (out.z16) *(uint2*)(out.z16 + t * out.ldz + o) = h;
        if (out.act) {
          const float a[4] = {gelu_tanh(bf16lo_f32(h.x)), gelu_tanh(bf16hi_f32(h.x)), gelu_tanh(bf16lo_f32(h.y)), gelu_tanh(bf16hi_f32(h.y))};
          if (out.a8) {
#pragma unroll
            for (int e = 0; e < 4; e++) amax = max(amax, f2u(a[e]) & 0x7FFFFFFFu);
            const float r = out.a_inv_scale;
            int w = __builtin_amdgcn_cvt_pk_fp8_f32(clamp448(a[0] * r), clamp448(a[1] * r), 0, false);
            w = __builtin_amdgcn_cvt_pk_fp8_f32(clamp448(a[2] * r), clamp448(a[3] * r), w, true);
            *(int*)(out.a8 + t * out.lda + o) = w;
          } else {
            *(uint2*)(out.a16 + t * out.lda + o) = make_uint2(bf16_rne_pack(a[0], a[1]), bf16_rne_pack(a[2], a[3]));
          }
        }
      }
    }
  }
  if (AMAX || (!ZF8 && out.act && out.amax_bits)) publish_tile_amax<KW>(amax, AMAX ? out.amax_scale : 1.0f, out.amax_bits, red);
}

// One tile shape for the whole grid.  Workgroups are numbered so that each XCD works on a contiguous
// range of tiles, o-tiles fastest.
template <bool FP8, int MI_, int NI_, bool ZF8, bool AMAX>
__global__ void __launch_bounds__(512, 1)
k_linear_fwd_pipe(const uint8_t* __restrict__ X, int64_t T, int64_t k_bytes, int64_t ldx_bytes,
                  const uint8_t* __restrict__ vals, const uint8_t* __restrict__ meta,
                  int64_t O, FwdOut out, int m_tiles) {
  __shared__ __align__(1024) uint8_t smem[fwd_pipe_smem<FP8, MI_, NI_>()];
  const int logical = xcd_contiguous(blockIdx.x, gridDim.x);
  const int tm = logical % m_tiles, tn = logical / m_tiles;
  fwd_pipe_tile<FP8, MI_, NI_, ZF8, AMAX>(smem, X, T, k_bytes, ldx_bytes, vals, meta, O, out, (int64_t)tm * (32 * MI_),
                                          (int64_t)tn * (64 * NI_));
}

// 256 x 256 tiles (n_big all of them), or two tile shapes in one grid, for layers whose 256 x 256 tiles fill the CUs a whole number of times plus
// a remainder of at most half a round: the first n_big workgroups take 256 x 256 tiles, the rest take
// the remaining tiles as 256 x 128 halves.  The last round then has twice as many, half as long
// workgroups instead of leaving more than half of the CUs idle for a full tile time.
template <bool FP8, bool ZF8, bool AMAX>
__global__ void __launch_bounds__(512, 1)
k_linear_fwd_dual(const uint8_t* __restrict__ X, int64_t T, int64_t k_bytes, int64_t ldx_bytes,
                  const uint8_t* __restrict__ vals, const uint8_t* __restrict__ meta,
                  int64_t O, FwdOut out, TileOrder order, int n_big) {
  __shared__ __align__(1024) uint8_t smem[fwd_pipe_smem<FP8, 8, 4>()];
  static_assert(fwd_pipe_smem<FP8, 8, 2>() <= fwd_pipe_smem<FP8, 8, 4>(), "the half tile fits in the full tile's LDS");
  const int bid = blockIdx.x;
  if (bid < n_big) {
    const int logical = xcd_contiguous(bid, n_big);
    int tm, tn;
    tile_at(order, logical, tm, tn);
    fwd_pipe_tile<FP8, 8, 4, ZF8, AMAX>(smem, X, T, k_bytes, ldx_bytes, vals, meta, O, out, (int64_t)tm * 256, (int64_t)tn * 256);
  } else {
    const int h = xcd_contiguous(bid - n_big, (int)gridDim.x - n_big);      // half-tile number
    const int tile = n_big + (h >> 1);
    int tm, tn;
    tile_at(order, tile, tm, tn);
    const int64_t t0 = (int64_t)tn * 256 + 128 * (h & 1);
    if (t0 >= T) return;                       // second half of a ragged last token tile: nothing to do
    fwd_pipe_tile<FP8, 8, 2, ZF8, AMAX>(smem, X, T, k_bytes, ldx_bytes, vals, meta, O, out, (int64_t)tm * 256, t0);
  }
}

template <bool FP8, int MI_, int NI_, bool ZF8, bool AMAX>
static void launch_fwd_pipe(const void* X, int64_t T, int64_t I, int64_t ldx, const FwdOut& out, const void* vals,
                            const void* meta, int64_t O, hipStream_t s) {
  constexpr int BM = 32 * MI_, BN = 64 * NI_;
  int m_tiles = (int)((O + BM - 1) / BM), n_tiles = (int)((T + BN - 1) / BN);
  dim3 grid((unsigned)(m_tiles * n_tiles)), block(512);
  int64_t eb = FP8 ? 1 : 2;
  SSTE_LAUNCH(SSTE_K_FWD, (k_linear_fwd_pipe<FP8, MI_, NI_, ZF8, AMAX>), grid, block, s, (const uint8_t*)X, T, I * eb, ldx * eb,
              (const uint8_t*)vals, (const uint8_t*)meta, O, out, m_tiles);
}

template <bool FP8, bool ZF8, bool AMAX>
static void launch_fwd_dual(const void* X, int64_t T, int64_t I, int64_t ldx, const FwdOut& out, const void* vals,
                            const void* meta, int64_t O, int n_big, hipStream_t s) {
  int m_tiles = (int)((O + 255) / 256), n_tiles = (int)((T + 255) / 256);
  int n_small = 2 * (m_tiles * n_tiles - n_big);
  dim3 grid((unsigned)(n_big + n_small)), block(512);
  int64_t eb = FP8 ? 1 : 2;
  SSTE_LAUNCH(SSTE_K_FWD, (k_linear_fwd_dual<FP8, ZF8, AMAX>), grid, block, s, (const uint8_t*)X, T, I * eb, ldx * eb,
              (const uint8_t*)vals, (const uint8_t*)meta, O, out, tile_order(m_tiles, n_tiles), n_big);
}

bool linear_fwd_supported(int64_t T, int64_t I, int64_t ldx, int64_t O, int dtype) {
  int64_t eb = dtype == SSTE_F8E4M3 ? 1 : 2;
  // 32-bit offsets inside a tile, 32-bit tile count
  if (product_reaches(ldx, 256 * eb, 1ll << 30) || product_reaches(I, 256 * eb, 1ll << 30)) return false;
  if (product_reaches(O / 256 + 1, T / 128 + 1, 0x80000000ll)) return false;
  return true;
}

template <bool FP8, int WM, int WN, int MT, int NT, int KG, int NS, bool ZF8, bool AMAX>
static void launch_fwd_tile(const void* X, int64_t T, int64_t I, int64_t ldx, const FwdOut& out, const void* vals,
                            const void* meta, int64_t O, hipStream_t s) {
  constexpr int BM = 32 * WM * MT, BN = 32 * WN * NT;
  int m_tiles = (int)((O + BM - 1) / BM), n_tiles = (int)((T + BN - 1) / BN);
  int64_t eb = FP8 ? 1 : 2;
  SSTE_LAUNCH(SSTE_K_FWD, (k_linear_fwd_tile<FP8, WM, WN, MT, NT, KG, NS, ZF8, AMAX>), dim3((unsigned)(m_tiles * n_tiles)), dim3(64 * WM * WN * KG), s,
              (const uint8_t*)X, T, I * eb, ldx * eb, (const uint8_t*)vals, (const uint8_t*)meta, O, out, m_tiles);
}

template <bool FP8, int KW, int U, bool ZF8, bool AMAX>
static void launch_fwd_skinny(const void* X, int64_t T, int64_t I, int64_t ldx, const FwdOut& out, const void* vals,
                              const void* meta, int64_t O, hipStream_t s) {
  int m_tiles = (int)((O + 15) / 16), n_tiles = (int)((T + 15) / 16);
  int64_t eb = FP8 ? 1 : 2;
  SSTE_LAUNCH(SSTE_K_FWD, (k_linear_fwd_skinny<FP8, KW, U, ZF8, AMAX>), dim3((unsigned)(m_tiles * n_tiles)), dim3(64 * KW), s, (const uint8_t*)X, T,
              I * eb, ldx * eb, (const uint8_t*)vals, (const uint8_t*)meta, O, out, m_tiles);
}

// Choice of the kernel.  Form of a time model in microseconds: base + store * (output bytes at 5 TB/s) + rounds, a workgroup costing F + nk *
// step with nk its k-steps (each k-group of a workgroup takes a KG-th of them) and step = max(lat, r * thr) for r workgroups sharing a CU;
// R fit a CU (LDS) and what does not fit runs in further rounds.  The two-shape grid has a row of its own: whole rounds of 256 x 256 tiles
// and one of 256 x 128 tiles, each with its F and step.  Two sets of rows:
// Weights up to 5120 wide and up to 32768 tokens: the rows rank the shapes and are no times (the terms' names say how they enter, not what
// they measure: the two-shape grid's step is 0 and its base 22 us in bf16); what they say ends with that range.  They are chosen for what the
// choice costs on 2400 random problems (1 ... 32768 tokens, 64 ... 5120 channels and features, a third of them layers of the GPT-2
// workloads), timed in every shape, and for not losing anywhere to the choice before (rows fitted without the 128 x 256 tiles): 0.9 %
// (bf16) / 0.75 % (8-bit) faster than that one on the geometric mean, by more than 3 % on a tenth of the problems, slower by more than
// 3 % on 2 / 1 % (12 / 11 % at worst).  128 x 256 tiles are there for what fills a round of them and little more than half a round of
// others: 1021 x 5120 x 1280 e4m3 11.3 -> 9.1 us.
// Wider weights or more tokens: rows fitted to the times themselves, no step below the matrix pipe's, so that they hold beyond what was
// timed.  `few`: the share of lat that a lone workgroup saves, with nobody to share L2 and memory.  2600 random problems up to 65536
// wide (1 ... 262144 tokens), on one set of buffers and on sets that rotate through 600 MB: the choice is 0.5 % slower than the best shape
// on the geometric mean, 23 / 21 % at worst; on 1500 others 0.5 %, 21 / 47 %.  The first set of rows loses 6.7 / 9.0 % there and up to
// 2.9 times the time (860 x 4192 x 63616 e4m3: 607 against 205 us), as it sends few tokens to the 64 x 32 and 32 x 32 tiles.
struct FwdShape {
  int bm, bn, kg, r, threads;
};
struct FwdCost {
  double f, lat, thr, base, store, few;
};
enum { FW_256, FW_256x128, FW_128x256, FW_128_R2, FW_128_R3, FW_128x64, FW_64, FW_64_KG2, FW_64x32_KG4, FW_32_KG4, FW_16_KG8, FW_SHAPES, FW_DUAL = FW_SHAPES, FW_DUAL128 };
static const FwdShape kFwd[FW_SHAPES] = {
  {256, 256, 1, 1, 512},
  {256, 128, 1, 2, 256},
  {128, 256, 1, 1, 512},
  {128, 128, 1, 2, 256},
  {128, 128, 1, 3, 256},
  {128, 64, 1, 2, 256},
  {64, 64, 1, 3, 256},
  {64, 64, 2, 1, 512},
  {64, 32, 4, 1, 512},
  {32, 32, 4, 1, 256},
  {16, 16, 8, 4, 512},
};
static const FwdCost kFwdCost16[FW_SHAPES] = {
  {7.033, 0.572, 0.590, 0.014, 0.681},
  {0.159, 1.290, 0.015, 3.052, 0.002},
  {2.981, 0.384, 0.000, 0.170, 1.968},
  {2.580, 0.171, 0.319, 0.803, 0.665},
  {2.798, 0.008, 0.478, 0.500, 0.000},
  {0.000, 0.201, 0.320, 3.367, 0.092},
  {0.025, 0.299, 0.315, 2.976, 0.847},
  {5.159, 0.006, 0.234, 1.318, 0.001},
  {2.681, 0.355, 0.219, 2.263, 0.000},
  {2.446, 0.090, 0.379, 1.671, 1.127},
  {0.028, 0.001, 1.049, 0.113, 0.000},
};
static const FwdCost kFwdCost8[FW_SHAPES] = {
  {0.089, 0.930, 0.024, 4.711, 1.093},
  {2.306, 0.155, 1.014, 2.827, 0.000},
  {4.175, 0.000, 0.657, 0.513, 0.289},
  {0.248, 0.001, 0.602, 4.652, 0.239},
  {0.913, 0.868, 0.435, 2.847, 0.450},
  {2.360, 0.003, 0.509, 1.932, 0.023},
  {1.157, 0.001, 0.310, 2.953, 0.185},
  {0.420, 0.457, 0.010, 3.196, 5.917},
  {3.849, 0.001, 0.287, 0.013, 17.472},
  {0.001, 0.273, 0.000, 3.727, 18.888},
  {0.002, 0.380, 1.162, 0.000, 0.003},
};
static const FwdCost kFwdWide16[FW_SHAPES] = {
  {6.667, 0.604, 0.604, 0.149, 0.736, 0.512},
  {3.881, 0.990, 0.331, 3.150, 0.203, 0.585},
  {3.783, 0.489, 0.323, 0.104, 1.395, 0.025},
  {3.320, 0.279, 0.279, 2.453, 0.206, 0.447},
  {2.401, 0.721, 0.327, 0.910, 0.912, 0.345},
  {5.510, 0.174, 0.174, 0.152, 0.896, 0.664},
  {1.917, 0.343, 0.058, 4.004, 0.878, 0.747},
  {4.436, 0.294, 0.056, 0.114, 0.217, 0.030},
  {4.409, 0.340, 0.066, 0.110, 4.462, 0.378},
  {3.581, 0.202, 0.033, 0.106, 6.000, 0.000},
  {0.304, 0.405, 0.405, 2.634, 0.205, 0.421},
};
static const FwdCost kFwdWide8[FW_SHAPES] = {
  {5.890, 0.737, 0.737, 0.140, 0.210, 0.385},
  {2.331, 1.231, 0.551, 2.599, 0.203, 0.699},
  {4.421, 0.516, 0.369, 0.105, 1.050, 0.719},
  {1.468, 0.332, 0.332, 2.848, 0.532, 0.478},
  {1.980, 0.646, 0.323, 2.047, 0.500, 0.020},
  {4.349, 0.206, 0.206, 0.260, 0.601, 0.705},
  {0.372, 0.416, 0.058, 3.468, 0.918, 0.799},
  {4.832, 0.272, 0.056, 0.112, 0.208, 0.011},
  {4.604, 0.322, 0.066, 0.106, 5.969, 0.393},
  {3.530, 0.196, 0.033, 0.108, 5.995, 0.001},
  {0.301, 0.405, 0.405, 2.178, 5.950, 0.472},
};

// the two-shape grid: F and step of a round of 256 x 256 tiles, of the last one of 256 x 128 tiles, base, store
struct FwdDual {
  double f, step, f_half, step_half, base, store;
};
static const FwdDual kFwdDual16 = {3.521, 0.000, 1.893, 0.458, 21.918, 0.003}, kFwdDual8 = {3.736, 0.003, 0.604, 1.146, 5.867, 0.830};
static const FwdDual kFwdWideDual16 = {9.943, 0.435, 3.580, 0.614, 2.986, 0.208}, kFwdWideDual8 = {7.671, 0.512, 0.673, 0.858, 1.193, 0.203};

// 128 x 128 tiles that are more than one per CU and at most one and a half: the excess runs as twice as many 128 x 64 halves, so that every CU gets
// one tile and at most one half, and not some of them two tiles (or a 128 x 256 one) and the others one or none.  On 240 + 360 random problems of
// that kind (weights up to 5120 wide; wider ones and more tokens), against the shape that the rows below choose: 7 / 6 % (bf16) and 5 / 3 % (8-bit)
// faster on the geometric mean, at worst 3 / 4 % slower.  Not taken where it lost: up to three k-steps beyond 320 tiles (up to 7 %), more than 32
// k-steps in 8 bits (up to 8 %; the 128 x 256 tiles fetch fewer bytes), and where the last tile may be mostly padding (below 512 tokens; channels
// that fill less than three quarters of their tiles: 2 ... 5 % faster, up to 7 % slower).
// (1021 x 5120 x 1280 e4m3 with the activation 16.5 -> 14.7 us.)
static bool fwd_halves(bool fp8, int64_t T, int64_t O, int64_t steps) {
  const int64_t tiles = ((O + 127) / 128) * ((T + 127) / 128);
  return T >= 512 && 4 * O >= 3 * 128 * ((O + 127) / 128) && tiles > NUM_CU && tiles <= NUM_CU * 3 / 2 && (steps >= 4 || tiles <= NUM_CU * 5 / 4) && (!fp8 || steps <= 32);
}

static int fwd_choice(bool fp8, int64_t T, int64_t O, int64_t I) {
  const bool wide = O > 5120 || I > 5120 || T > 32768;
  const FwdCost* cost = wide ? (fp8 ? kFwdWide8 : kFwdWide16) : (fp8 ? kFwdCost8 : kFwdCost16);
  const FwdDual& dual = wide ? (fp8 ? kFwdWideDual8 : kFwdWideDual16) : (fp8 ? kFwdDual8 : kFwdDual16);
  const int64_t steps = I / (fp8 ? 128 : 64);
  if (fwd_halves(fp8, T, O, steps)) return FW_DUAL128;
  const double out_us = (double)T * (double)O * 2.0 / 5e6;
  int best = FW_256;
  double best_t = 1e30;
  for (int c = 0; c < FW_SHAPES; c++) {
    const FwdShape& g = kFwd[c];
    const FwdCost& s = cost[c];
    const int64_t wgs = ((O + g.bm - 1) / g.bm) * ((T + g.bn - 1) / g.bn);
    if (c != FW_256 && wgs > 0x7FFFFFFFll) continue;                                  // grid size
    const double nk = (double)((steps + g.kg - 1) / g.kg), fixed = s.base + s.store * out_us;
    const int64_t n = (wgs + NUM_CU - 1) / NUM_CU, full = n / g.r, rem = n % g.r;      // workgroups on the busiest CU: full rounds of r, and a rest
    const double part = c == FW_16_KG8 && T < 16 ? 0.4 + 0.6 / 16.0 * (double)T : 1.0;
    const double lat = wgs < NUM_CU ? s.lat * (1.0 - s.few * (1.0 - (double)wgs / NUM_CU)) : s.lat;
    double t = fixed + (double)full * (s.f + nk * part * (lat > g.r * s.thr ? lat : g.r * s.thr));
    if (rem) t += s.f + nk * part * (lat > rem * s.thr ? lat : rem * s.thr);
    if (t < best_t) {
      best_t = t;
      best = c;
    }
    // 256 x 256 tiles whose last round is at most half full: that round as 256 x 128 tiles
    if (c == FW_256 && wgs > NUM_CU && wgs % NUM_CU != 0 && wgs % NUM_CU <= NUM_CU / 2) {
      t = dual.base + dual.store * out_us + (double)(wgs / NUM_CU) * (dual.f + nk * dual.step) + dual.f_half + nk * dual.step_half;
      if (t < best_t) {
        best_t = t;
        best = FW_DUAL;
      }
    }
  }
  return best;
}

void describe_fwd(int64_t T, int64_t O, int64_t I, int dtype, char* text, size_t n) {
  const int cfg = fwd_choice(dtype == SSTE_F8E4M3, T, O, I);
  if (cfg == FW_DUAL) {
    const int64_t big = ((O + 255) / 256) * ((T + 255) / 256);
    snprintf(text, n, "256x256+256x128 kg 1 r 1 grid %lld block 512", (long long)(big + big % NUM_CU));
    return;
  }
  if (cfg == FW_DUAL128) {
    const int64_t tiles = ((O + 127) / 128) * ((T + 127) / 128);
    snprintf(text, n, "128x128+128x64 kg 1 r 2 grid %lld block 256", (long long)(2 * tiles - NUM_CU));
    return;
  }
  const FwdShape& s = kFwd[cfg];
  snprintf(text, n, "%dx%d kg %d r %d grid %lld block %d", s.bm, s.bn, s.kg, s.r, (long long)(((O + s.bm - 1) / s.bm) * ((T + s.bn - 1) / s.bn)), s.threads);
}

// Kernel choice for one combination of operand type, output type and amax.
template <bool FP8, bool ZF8, bool AMAX>
static void launch_fwd_variant(const void* X, int64_t T, int64_t I, int64_t ldx, const FwdOut& out, const void* vals,
                               const void* meta, int64_t O, hipStream_t s) {
  const int cfg = fwd_choice(FP8, T, O, I);
#define FT(WM, WN, MT, NT, KG, NS) launch_fwd_tile<FP8, WM, WN, MT, NT, KG, NS, ZF8, AMAX>(X, T, I, ldx, out, vals, meta, O, s)
  switch (cfg) {
    case FW_256:
    case FW_DUAL: {
      const int64_t tiles = ((O + 255) / 256) * ((T + 255) / 256);
      launch_fwd_dual<FP8, ZF8, AMAX>(X, T, I, ldx, out, vals, meta, O, (int)(cfg == FW_DUAL ? tiles - tiles % NUM_CU : tiles), s);
      break;
    }
    case FW_128x256: launch_fwd_pipe<FP8, 4, 4, ZF8, AMAX>(X, T, I, ldx, out, vals, meta, O, s); break;
    case FW_256x128: {
      const int m_tiles = (int)((O + 255) / 256), n_tiles = (int)((T + 127) / 128);
      const int64_t eb = FP8 ? 1 : 2;
      SSTE_LAUNCH(SSTE_K_FWD, (k_linear_fwd_pair<FP8, 2, 8, 4, ZF8, AMAX>), dim3((unsigned)(m_tiles * n_tiles)), dim3(256), s, (const uint8_t*)X, T,
                  I * eb, ldx * eb, (const uint8_t*)vals, (const uint8_t*)meta, O, out, m_tiles);
      break;
    }
    case FW_DUAL128: {
      const int m_tiles = (int)((O + 127) / 128), tiles = m_tiles * (int)((T + 127) / 128);
      const int64_t eb = FP8 ? 1 : 2;
      SSTE_LAUNCH(SSTE_K_FWD, (k_linear_fwd_dual128<FP8, ZF8, AMAX>), dim3((unsigned)(2 * tiles - NUM_CU)), dim3(256), s, (const uint8_t*)X, T,
                  I * eb, ldx * eb, (const uint8_t*)vals, (const uint8_t*)meta, O, out, m_tiles, NUM_CU);
      break;
    }
    case FW_128_R2: FT(2, 2, 2, 2, 1, 3); break;
    case FW_128_R3: FT(2, 2, 2, 2, 1, 2); break;
    case FW_128x64: FT(2, 2, 2, 1, 1, 4); break;
    case FW_64: FT(2, 2, 1, 1, 1, 4); break;
    case FW_64_KG2: FT(2, 2, 1, 1, 2, 4); break;
    case FW_64x32_KG4: FT(2, 1, 1, 1, 4, 4); break;
    case FW_32_KG4: FT(1, 1, 1, 1, 4, 4); break;
    default: launch_fwd_skinny<FP8, 8, 2, ZF8, AMAX>(X, T, I, ldx, out, vals, meta, O, s); break;
  }
#undef FT
}

hipError_t launch_linear_fwd(const void* X, int64_t T, int64_t I, int64_t ldx, int dtype, float scale,
                             const void* vals, const void* meta, int64_t O, void* Z, int64_t ldz, int z_dtype,
                             float amax_scale, float* amax_out, hipStream_t s) {
  if (amax_out) hipLaunchKernelGGL(k_fill_u32_fwd, dim3(1), dim3(1), 0, s, (uint32_t*)amax_out, 0u);
  if (T == 0 || O == 0) return hipGetLastError();
  const bool fp8 = dtype == SSTE_F8E4M3, zf8 = z_dtype == SSTE_F8E4M3;
  FwdOut out;
  out.z16 = zf8 ? nullptr : (uint16_t*)Z;
  out.z8 = zf8 ? (uint8_t*)Z : nullptr;
  out.ldz = ldz;
  out.scale = scale;
  out.amax_scale = amax_scale;
  out.amax_bits = (uint32_t*)amax_out;
  out.act = 0;
  out.a16 = nullptr;
  out.a8 = nullptr;
  out.lda = 0;
  out.a_inv_scale = 1.0f;
  out.a_stream = 0;
  const bool amax = amax_out != nullptr;
#define FWD_CASE(F, Z8, A)                                                                \
  if (fp8 == F && zf8 == Z8 && amax == A) launch_fwd_variant<F, Z8, A>(X, T, I, ldx, out, vals, meta, O, s)
  FWD_CASE(false, false, false);
  FWD_CASE(false, false, true);
  FWD_CASE(false, true, true);          // an e4m3 output always comes with its largest magnitude (the API insists)
  FWD_CASE(true, false, false);
  FWD_CASE(true, false, true);
  FWD_CASE(true, true, true);
#undef FWD_CASE
  return hipGetLastError();
}

// Forward product with the activation in the epilogue: H = RNE_bf16(acc * scale) (stored if H != null),
// A = GELU(H) stored as bf16 or as e4m3 of A * a_inv_scale (then with the largest |A| in amax_out).
hipError_t launch_linear_fwd_act(const void* X, int64_t T, int64_t I, int64_t ldx, int dtype, float scale,
                                 const void* vals, const void* meta, int64_t O, void* H, int64_t ldh, void* A, int64_t lda,
                                 int a_dtype, float a_inv_scale, float* amax_out, hipStream_t s) {
  if (amax_out) hipLaunchKernelGGL(k_fill_u32_fwd, dim3(1), dim3(1), 0, s, (uint32_t*)amax_out, 0u);
  if (T == 0 || O == 0) return hipGetLastError();
  FwdOut out;
  out.z16 = (uint16_t*)H;
  out.z8 = nullptr;
  out.ldz = ldh;
  out.scale = scale;
  out.amax_scale = 1.0f;
  out.amax_bits = (uint32_t*)amax_out;
  out.act = 1;
  out.a16 = a_dtype == SSTE_F8E4M3 ? nullptr : (uint16_t*)A;
  out.a8 = a_dtype == SSTE_F8E4M3 ? (uint8_t*)A : nullptr;
  out.lda = lda;
  out.a_inv_scale = a_inv_scale;
  out.a_stream = a_dtype != SSTE_F8E4M3 && product_reaches(T, O * 2, (128ll << 20) + 1);
  if (dtype == SSTE_F8E4M3) launch_fwd_variant<true, false, false>(X, T, I, ldx, out, vals, meta, O, s);
  else launch_fwd_variant<false, false, false>(X, T, I, ldx, out, vals, meta, O, s);
  return hipGetLastError();
}

}  // namespace sste
