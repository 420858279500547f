// Weight gradients of experts with few rows, or with few output tiles: 128 x 128 tiles, three workgroups per compute unit, both
// products in one launch.  Part of the bf16 expert-FFN kernels; included by ffn_bf16.hip only (one translation unit).
#pragma once
#include "common.h"
#include "ffn_bf16_tile.h"
#include "ffn_bf16_dma.h"
#include "ffn_bf16_small.h"
#include "ffn_bf16_wgrad.h"
namespace flexmoe {
// =============================================================================================
// wgrad_gemm_small: the products of wgrad_gemm_dma where an output tile's contraction is a few 32-token K tiles.  Then a tile is
// its job's look-up, its first loads' trip from memory and its stores, and the single workgroup per compute unit of the
// 256 x 256 kernels has nothing to put beside them.  So
//  * four waves own 128 x 128 outputs (64 x 64 each, 64 accumulator registers) and three stages of 16 KB, which leaves room for
//    three workgroups per compute unit: one stores while another waits for its operands;
//  * one workgroup per tile, dispatched by the hardware as compute units become free, dW2's tiles before dW1's in the
//    same launch: the second product fills the compute units that the first one's last tiles leave;
//  * a K tile lies in LDS as in memory (32 tokens x 256 bytes), transposed on the way out by ds_read_tr16_b64 (chunk swizzle as in
//    dmat_chunk); outputs go through a wave-private patch, so that a store instruction fills whole 128-byte lines.
// What bounds it: 1500 tokens (k 2) of d 1024, f 4096, 32 experts: the 537 MB of both gradients' stores (109 us at the rate of a
// large copy).  Whole backward pass there 382 -> 366 us; d 256, f 1024, 8 experts, 3200 rows 97 -> 66; d 128, f 512, 16 experts, 4096 rows
// 79 -> 54, with dXp in the same launch 44 (two launches instead of four, six times as many tiles in flight).
// Work list, segments and the order of the sums are those of the 256 x 256 kernels (the same instruction, K tiles in the same
// order): the same bits.
// =============================================================================================
constexpr int GT = 128;                                  // edge of an output tile
constexpr int kGradThreads = 4 * kWave;
constexpr int kGradStages = 3;
constexpr int kGradOpBytes = DK * GT * 2;                // one operand's K tile: 8 KB
constexpr int kGradStageBytes = 2 * kGradOpBytes;
constexpr int kGradLds = kGradStages * kGradStageBytes;
constexpr int kGradLoads = 4;                            // direct loads per wave and stage: two of either operand

struct WgradSmallArgs {
  WgradDmaArgs p[2];             // dW2, dW1 (m_tiles, n_tiles: of GT)
  unsigned grid0;                // workgroups of dW2, a multiple of kXcds * kPatch
};

typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// smem: kGradLds bytes
__device__ __forceinline__ void wgrad_small_block(const WgradSmallArgs& a, unsigned char* smem, unsigned block) {
  lds_byte_t* const sm = (lds_byte_t*)smem;
  const unsigned lds0 = __builtin_amdgcn_readfirstlane((unsigned)(uintptr_t)sm);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int fr = lane & 15, fg = lane >> 4;
  const bool second = block >= a.grid0;
  const WgradDmaArgs& p = a.p[second ? 1 : 0];
  const int M = p.M, NC = p.NC;
  int grow, nt;
  if (!patched_tile(block - (second ? a.grid0 : 0u), p.seg_rows_max * p.m_tiles, p.n_tiles, &grow, &nt)) return;
  const i32x4_t job = ((ConstInt4Ptr)p.plan.jobs)[grow / p.m_tiles];
  const int e = job[0], seg = job[1], nseg = job[2];
  if (e < 0) return;
  const int m0 = (grow % p.m_tiles) * GT, n0 = nt * GT;
  const int mvalid = min(GT, M - m0), nvalid = min(GT, NC - n0);

  // the job's K tiles [lo, hi) of the expert's sequence, and the bucket / offset where they start
  const ConstIntPtr boff = (ConstIntPtr)p.plan.boff, bstart = (ConstIntPtr)p.plan.bstart, brows = (ConstIntPtr)p.plan.brows;
  const int b0 = boff[e], b1 = boff[e + 1], Te = ((ConstIntPtr)p.plan.etiles)[e];
  const int lo = nseg > 1 ? seg * p.seg_tiles : 0;
  const int T = (nseg > 1 ? min(Te, lo + p.seg_tiles) : Te) - lo;
  const bf16_t *lp = p.L + m0, *rp = p.R + n0;           // token row 0 of the next K tile, first column of the tile
  int b = b0, rows_left = 0;                             // rows of bucket b from that row on
  auto seek = [&](int skip) {
    const int start = bstart[b] + skip;
    rows_left = brows[b] - skip;
    lp = p.L + (size_t)start * M + m0;
    rp = p.R + (size_t)start * NC + n0;
  };
  if (T > 0) {
    int skip = lo;
    for (int n; b < b1 - 1 && skip >= (n = (brows[b] + DK - 1) / DK); ++b) skip -= n;
    seek(skip * DK);
  }

  // load q of either operand: K rows 4 (2 wave + q) .. + 3, columns past the matrix repeat its last chunk
  uint32_t loff[2], roff[2];
  int krow[2];
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    krow[q] = (wave * 2 + q) * 4 + fg;
    const int c = fr ^ ((krow[q] & 3) << 2) ^ ((krow[q] & 8) >> 2);
    loff[q] = (uint32_t)(krow[q] * M + min(c, mvalid / 8 - 1) * 8) * 2;
    roff[q] = (uint32_t)(krow[q] * NC + min(c, nvalid / 8 - 1) * 8) * 2;
  }
  int issued = 0;
  unsigned to = lds0;                                    // stage of the next K tile to load
  auto issue = [&]() {
    const unsigned at = to + (unsigned)wave * 2048;
    if (rows_left >= DK) {
#pragma unroll
      for (int q = 0; q < 2; ++q) small_load(lp, loff[q], at + q * 1024);
#pragma unroll
      for (int q = 0; q < 2; ++q) small_load(rp, roff[q], at + kGradOpBytes + q * 1024);
    } else {                                             // tokens past the bucket: zeros on both sides
      const bf16_t* z = (const bf16_t*)kZeroRow + fr * 8;
#pragma unroll
      for (int q = 0; q < 2; ++q)
        small_load_at(krow[q] < rows_left ? (const bf16_t*)((const char*)lp + loff[q]) : z, at + q * 1024);
#pragma unroll
      for (int q = 0; q < 2; ++q)
        small_load_at(krow[q] < rows_left ? (const bf16_t*)((const char*)rp + roff[q]) : z, at + kGradOpBytes + q * 1024);
    }
    to = to + kGradStageBytes == lds0 + kGradStages * kGradStageBytes ? lds0 : to + kGradStageBytes;
    if (++issued < T) {
      rows_left -= DK;
      lp += (size_t)DK * M;
      rp += (size_t)DK * NC;
      if (rows_left <= 0) {
        ++b;                                             // (a tile is left, so the expert has another bucket)
        seek(0);
      }
    }
  };

  const int wm = wave >> 1, wn = wave & 1;
  uint32_t lane_at;
  {
    const int k = 8 * fg + (fr >> 2), x = ((fr >> 2) << 2) ^ ((fg & 1) << 1);
    lane_at = k * 256 + 8 * (fr & 1) + ((((fr & 3) >> 1) ^ x) << 4);
  }
  auto frag = [&](const lds_byte_t* tile, int unit) {    // columns 16 unit .. of the tile
    const lds_byte_t* at = tile + (lane_at ^ (uint32_t)(unit << 5));
    const s16x4 f0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)at);
    const s16x4 f1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(at + 4 * 256));
    typedef short s16x8 __attribute__((ext_vector_type(8)));
    return __builtin_bit_cast(bf16x8, (s16x8)__builtin_shufflevector(f0, f1, 0, 1, 2, 3, 4, 5, 6, 7));
  };
  f32x4 acc[4][4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

  if (T > 0) issue();
  if (T > 1) issue();
  unsigned st = 0;
  for (int kt = 0; kt < T; ++kt) {
    if (kt + 1 < T) wait_vmcnt<kGradLoads>();
    else wait_vmcnt<0>();
    lds_barrier();
    if (kt + 2 < T) issue();                             // into the stage every wave has just left
    const lds_byte_t* tile = sm + st;
    bf16x8 l[4], r[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) l[i] = frag(tile, wm * 4 + i);
#pragma unroll
    for (int j = 0; j < 4; ++j) r[j] = frag(tile + kGradOpBytes, wn * 4 + j);
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(r[j], l[i], acc[i][j], 0, 0, 0);
    st = st + kGradStageBytes == kGradStages * kGradStageBytes ? 0 : st + kGradStageBytes;
  }

  // lane: row fr of 16-row block i, columns 4 fg .. of 16-column block j
  if (nseg == 1) {
    __syncthreads();                                     // every wave has left the last stage
    lds_byte_t* const patch = sm + wave * 8192;          // 64 rows of 128 bytes, chunk XOR row & 7
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const f32x4 c = acc[i][j];
        *(__attribute__((address_space(3))) u32x2*)(patch + (i * 16 + fr) * 128 + (((j * 2 + (fg >> 1)) ^ (fr & 7)) << 4) + (fg & 1) * 8) =
            u32x2{pack_bf16x2(c[0], c[1]), pack_bf16x2(c[2], c[3])};
      }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
    bf16_t* const out = p.dw + (size_t)e * M * NC;
    const int col = n0 + wn * 64 + (lane & 7) * 8;
#pragma unroll
    for (int it = 0; it < 8; ++it) {
      const int row = it * 8 + (lane >> 3);
      const u32x4 v = *(const __attribute__((address_space(3))) u32x4*)(patch + row * 128 + (((lane & 7) ^ (row & 7)) << 4));
      if (m0 + wm * 64 + row < M && col < NC)
        __builtin_nontemporal_store(v, (u32x4*)(out + (size_t)(m0 + wm * 64 + row) * NC + col));      // written once
    }
  } else {
    // one of several segments: the fp32 tile goes to the workspace for wgrad_reduce_kernel
    float* const out = p.partial + (size_t)(job[3] + seg) * M * NC;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int row = m0 + wm * 64 + i * 16 + fr;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int col = n0 + wn * 64 + j * 16 + fg * 4;
        if (row < M && col < NC) *(f32x4*)(out + (size_t)row * NC + col) = acc[i][j];
      }
    }
  }
}

__global__ __launch_bounds__(kGradThreads, 3) void wgrad_gemm_small_bf16(const WgradSmallArgs a) {
  __shared__ __align__(1024) unsigned char smem[kGradLds];
  wgrad_small_block(a, smem, blockIdx.x);
}

// dXp and both weight gradients, which depend on nothing of each other: the first `rows_grid` workgroups (a multiple of kXcds) walk
// dXp's tiles, and the weight gradients' fill the compute units as they finish.
// (Backward pass of d 128, f 512, 16 experts, 1536 rows 47 -> 34 us.)
template <int BM> __global__ __launch_bounds__(kGradThreads, 2) void bwd_products_small_bf16(const SmallArgs p, const WgradSmallArgs a, unsigned rows_grid) {
  __shared__ __align__(1024) unsigned char smem[SmallCfg<BM>::kLds > kGradLds ? SmallCfg<BM>::kLds : kGradLds];
  if (blockIdx.x < rows_grid) rows_small_block<BM, true, EPI_PLAIN, false>(p, smem, blockIdx.x, rows_grid);
  else wgrad_small_block(a, smem, blockIdx.x - rows_grid);
}

}  // namespace flexmoe
