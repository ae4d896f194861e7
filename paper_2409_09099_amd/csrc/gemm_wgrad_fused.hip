// Weight-gradient GEMM of the S-STE linear layer (paper Sec. 5.1): grad_W = MVUE(grad_Z^T) X -- the kernel for small problems: one launch,
// no workspace.
//
// A workgroup owns 16 channels x 64 features and the whole token axis; its waves work alone, each on every eighth k-step (64 tokens
// bf16, 128 tokens 8-bit) through LDS slots of its own, and their sums are added at the end in a fixed order.  Small problems are a
// chain of latencies, and this keeps the chain short: no barrier before the end, and the sparse operand never leaves the registers.
// A transposing LDS read of the wave's grad_Z slot hands each lane four tokens of one channel (8-bit: eight), which is the estimator's
// group; the sparse MFMA wants from lane (row j, quarter q) the recorded values of exactly the groups 4 q .. 4 q + 3 (8-bit: 8 q ..
// 8 q + 7) of row j, so the estimator's results are the operand fragment.  The random number of a group depends only on (key, group
// id): any division of the work gives the same sparsified operand.
//
// What bounds it: the estimator is worked out once per 64 features, ~100 vector instructions per group, so the time grows with
// O T I while the packed path's does not; the host's time model takes this kernel only where that path's second launch costs more.
// Measured at 512 tokens, 256 x 1024 (bf16): 5.6 us; before, with 128 x 128 tiles, a barrier-bound loop over the tokens and the packed
// operand written to LDS, 22 us.
#include "common.h"
#include "mvue_device.h"

namespace sste {

namespace {
typedef __attribute__((address_space(3))) bf16x4 lds_bf16x4;
typedef __attribute__((address_space(3))) i32x2 lds_i32x2;
constexpr int NW = 8;                           // waves = token-axis shares of a workgroup
constexpr int DY_SLOT = 2048, X_SLOT = 8192, SLOT = DY_SLOT + X_SLOT, NS = 2;
constexpr int MAX_GRID_X = 1 << 22;             // a launch takes fewer than 2^32 threads per grid dimension

// Direct-to-LDS load from 64-bit addresses (whatever the size of the matrix): 16 bytes per lane to lds_addr + 16 lane.
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
__device__ __forceinline__ void dma_global_b128(const uint8_t* p, uint32_t lds_addr) {
  asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dwordx4 %1, off" : : "s"(lds_addr), "v"(p) : "memory", "m0");
}
#pragma clang diagnostic pop
}  // namespace

template <bool FP8, bool BF8>
__global__ void __launch_bounds__(64 * NW, 1)
k_wgrad_small(const uint8_t* __restrict__ dY, int64_t steps, int64_t O, int64_t lddy_bytes, const uint8_t* __restrict__ X, int64_t I,
              int64_t ldx_bytes, RngKey key, float scale, int accumulate, float* __restrict__ dW, int64_t lddw, int n_tiles, int tiles) {
  constexpr int EB = FP8 ? 1 : 2, KS = FP8 ? 128 : 64;
  constexpr int GROUPS = KS / 4, GPL = GROUPS / 4;      // token groups per k-step; per lane
  constexpr int CPR = 64 * EB / 16, UC = EB;            // 16-byte chunks per X row; per block of 16 features
  constexpr int LPS = (DY_SLOT + X_SLOT) / 1024;        // loads per k-step
  __shared__ __align__(1024) uint8_t smem[NW * NS * SLOT];

  const int logical = (int)blockIdx.y * MAX_GRID_X + xcd_contiguous(blockIdx.x, gridDim.x);
  if (logical >= tiles) return;
  const int64_t o0 = (int64_t)(logical / n_tiles) * 16, i0 = (int64_t)(logical % n_tiles) * 64;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int j = lane & 15, q = lane >> 4;
  uint8_t* const ring = smem + wave * NS * SLOT;
  const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_u8*)ring;

  // Channels past O and features past I are read from the tile's first ones: each row and column of the product stands alone, and
  // theirs are not stored.
  // grad_Z slot: the token rows (16 channels) one transposing read gathers lie side by side: row t of piece g of quarter q is token
  // (KS / 4) q + P g + t with P rows per piece (4, 8-bit 8).
  constexpr int P = FP8 ? 8 : 4, RCH = EB;              // 16-byte chunks per row of 16 channels
  const uint8_t* pdy[2];
#pragma unroll
  for (int i = 0; i < 2; i++) {
    const int d = 64 * i + lane, pos = d / RCH, c = d % RCH;
    const int g = pos / (4 * P), qq = (pos / P) % 4, t = pos % P;
    pdy[i] = dY + ((KS / 4) * qq + P * g + t) * lddy_bytes + (o0 + (o0 + c * (16 / EB) < O ? c * (16 / EB) : 0)) * EB;
  }
  // X slot: rows of 64 features; block u of 16 features of token row r lies at u ^ xkey(r), which spreads the rows and columns of one
  // transposing read (per 32 lanes: 8 rows x 32 B, 8-bit 16 rows x 16 B) over all banks
  auto xkey = [](int r) { return FP8 ? ((r >> 2) & 1) | ((r >> 3) & 2) : ((r >> 1) & 1) | ((r >> 2) & 2); };
  const uint8_t* px[8];
#pragma unroll
  for (int i = 0; i < 8; i++) {
    const int d = 64 * i + lane, r = d / CPR, cs = d % CPR;
    const int c = ((cs / UC) ^ xkey(r)) * UC + cs % UC;
    px[i] = X + r * ldx_bytes + (i0 + (i0 + c * (16 / EB) < I ? c * (16 / EB) : 0)) * EB;
  }
  auto issue = [&](int64_t st, int slot) {
#pragma unroll
    for (int i = 0; i < 2; i++) dma_global_b128(pdy[i] + st * KS * lddy_bytes, lds0 + slot * SLOT + i * 1024);
#pragma unroll
    for (int i = 0; i < 8; i++) dma_global_b128(px[i] + st * KS * ldx_bytes, lds0 + slot * SLOT + DY_SLOT + i * 1024);
  };

  f32x4 acc[4];
#pragma unroll
  for (int ni = 0; ni < 4; ni++) acc[ni] = (f32x4){0.f, 0.f, 0.f, 0.f};
  const uint64_t gid0 = (key.first_group + (uint64_t)(GPL * q)) * (uint64_t)O + (uint64_t)(o0 + j);

  if (wave < steps) issue(wave, 0);
  if (wave + NW < steps) issue(wave + NW, 1);
  int slot = 0;
  for (int64_t st = wave; st < steps; st += NW) {
    if (st + NW < steps) wait_vmcnt<LPS>();
    else wait_vmcnt<0>();
    const uint8_t* sl = ring + slot * SLOT;
    uint32_t fa[4], idx = 0;
#pragma unroll
    for (int g = 0; g < 4; g++) {
      const uint64_t gid = gid0 + ((uint64_t)st * GROUPS + (FP8 ? 2 : 1) * g) * (uint64_t)O;
      const uint32_t x0 = draw_u32(key.k0, key.k1, (uint32_t)gid, (uint32_t)(gid >> 32));
      uint32_t m;
      if (FP8) {
        const i32x2 v = __builtin_amdgcn_ds_read_tr8_b64_v2i32((lds_i32x2*)(sl + (g * 32 + q * 8 + (j >> 1)) * 16 + 8 * (j & 1)));
        const uint64_t gid1 = gid + (uint64_t)O;
        fa[g] = mvue_pair_f8<BF8>((uint32_t)v[0], (uint32_t)v[1], x0, draw_u32(key.k0, key.k1, (uint32_t)gid1, (uint32_t)(gid1 >> 32)), m);
        idx |= m << (8 * g);
      } else {
        const bf16x4 v = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4*)(sl + (g * 16 + q * 4 + (j >> 2)) * 32 + 8 * (j & 3)));
        uint2 w;
        __builtin_memcpy(&w, &v, 8);
        fa[g] = mvue_group_bf16(w.x, w.y, x0, m);
        idx |= m << (4 * g);
      }
    }
    if (!FP8) idx = 0xEEEEu - idx;
#pragma unroll
    for (int ni = 0; ni < 4; ni++) {
      uint2 fb[4];
#pragma unroll
      for (int r = 0; r < 4; r++) {
        const int row = FP8 ? 16 * q + 8 * (r & 1) + 64 * (r >> 1) + (j >> 1) : 8 * q + 4 * (r & 1) + 32 * (r >> 1) + (j >> 2);
        const uint8_t* p = sl + DY_SLOT + row * (64 * EB) + ((ni ^ xkey(row)) * 16 * EB) + (FP8 ? 8 * (j & 1) : 8 * (j & 3));
        if (FP8) {
          const i32x2 v = __builtin_amdgcn_ds_read_tr8_b64_v2i32((lds_i32x2*)p);
          fb[r] = make_uint2((uint32_t)v[0], (uint32_t)v[1]);
        } else {
          const bf16x4 v = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4*)p);
          __builtin_memcpy(&fb[r], &v, 8);
        }
      }
      if (FP8) {
        i32x4 av;
        i32x8 bv;
        __builtin_memcpy(&av, fa, 16);
        __builtin_memcpy(&bv, fb, 32);
        if (BF8) acc[ni] = __builtin_amdgcn_smfmac_f32_16x16x128_bf8_fp8(av, bv, acc[ni], (int)idx, 0, 0);
        else acc[ni] = __builtin_amdgcn_smfmac_f32_16x16x128_fp8_fp8(av, bv, acc[ni], (int)idx, 0, 0);
      } else {
        bf16x8 av;
        bf16x16 bv;
        __builtin_memcpy(&av, fa, 16);
        __builtin_memcpy(&bv, fb, 32);
        acc[ni] = __builtin_amdgcn_smfmac_f32_16x16x64_bf16(av, bv, acc[ni], (int)idx, 0, 0);
      }
    }
    if (st + 2 * NW < steps) {
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");     // the slot has been read
      issue(st + 2 * NW, slot);
    }
    slot ^= 1;
  }

  // sums of the waves that had a k-step, wave 0 first: each leaves its own in its slots (which nobody else reads before the barrier)
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
  for (int ni = 0; ni < 4; ni++) *(float4*)(ring + ni * 1024 + lane * 16) = make_float4(acc[ni][0], acc[ni][1], acc[ni][2], acc[ni][3]);
  __syncthreads();
  // wave w adds up and stores the rows 4 q + 2 (w % 2) + {0, 1} of the feature block w / 2
  const int ni = wave >> 1, r0 = 2 * (wave & 1);
  const int shares = (int)(steps < NW ? steps : NW);
  float2 sum = make_float2(0.f, 0.f);
  for (int w = 0; w < shares; w++) {
    const float2 v = *(const float2*)(smem + w * NS * SLOT + ni * 1024 + lane * 16 + r0 * 4);
    sum.x += v.x;
    sum.y += v.y;
  }
  const int64_t i = i0 + 16 * ni + j;
#pragma unroll
  for (int r = 0; r < 2; r++) {
    const int64_t o = o0 + 4 * q + r0 + r;
    if (o < O && i < I) {
      const float v = (r ? sum.y : sum.x) * scale;
      float* p = dW + o * lddw + i;
      *p = accumulate ? (*p + v) : v;
    }
  }
}

hipError_t launch_wgrad_fused(const void* dY, int64_t T, int64_t O, int64_t lddy, int dtype, const void* X, int64_t I, int64_t ldx,
                              RngKey key, float scale, int accumulate, float* dW, int64_t lddw, hipStream_t s) {
  const bool fp8 = dtype != SSTE_BF16;
  const int eb = fp8 ? 1 : 2, n_tiles = (int)((I + 63) / 64);
  const int tiles = (int)((O + 15) / 16) * n_tiles;
  const dim3 grid((unsigned)(tiles < MAX_GRID_X ? tiles : MAX_GRID_X), (unsigned)((tiles + MAX_GRID_X - 1) / MAX_GRID_X)), block(64 * NW);
#define WS_CASE(F8, B8)                                                                                                             \
  SSTE_LAUNCH(SSTE_K_WGRAD, (k_wgrad_small<F8, B8>), grid, block, s, (const uint8_t*)dY, T / (F8 ? 128 : 64), O, lddy * eb,           \
              (const uint8_t*)X, I, ldx * eb, key, scale, accumulate, dW, lddw, n_tiles, tiles)
  if (dtype == SSTE_F8E5M2) WS_CASE(true, true);
  else if (fp8) WS_CASE(true, false);
  else WS_CASE(false, false);
#undef WS_CASE
  return hipGetLastError();
}

}  // namespace sste
