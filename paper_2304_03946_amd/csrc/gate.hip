// Top-k gate (paper Eq. 3): logits l = x . W_g, keep the k largest per token, softmax over them.
//
// bf16 path: HBM-bound streaming of x.  The logits come from MFMA so that the 2*d*E flops per
// token do not cap the kernel below the memory roofline: the gate weights act as the MFMA
// row operand (32 experts per tile) and 32 tokens as the column operand, hence after the
// K loop every lane holds half of one token's logits and its partner lane (lane ^ 32) the
// other half -- the top-k selection is a register scan plus one cross-lane exchange per pick.
// x and W_g travel global -> LDS with direct loads that fetch whole 128-byte lines, and the fragments are read from LDS, those of W_g
// transposed on the way.
// From 32768 tokens with up to 64 experts (gate_dma_kernel) every wave owns 32 tokens and the whole contraction, several 64-wide K
// tiles in flight per workgroup.  Otherwise (gate_quarters_kernel) there is one workgroup per 32 tokens, the contraction split over its
// four waves and the partial logits summed in a fixed order through LDS.
// The order of a logit's sum is part of the result: logits that differ by fp32 rounding alone decide a near tie, and with
// it a token's experts.  gate_quarters_kernel adds in quarters: quarter q holds
// the 64-wide K chunks q, q + 4, .., summed in ascending order, and the logit is q0 + (q1 + (q2 + q3)).  gate_dma_kernel: one sum over
// all chunks, from a first chunk that depends on the token's workgroup.
//
// fp32 path: a group of lanes per token, sequential fp32 FMA per logit out of LDS, butterfly arg-max per pick.
#include <algorithm>

#include "common.h"

namespace flexmoe {

constexpr int kGateThreads = 256;
constexpr float kNegInf = -__builtin_huge_valf();

constexpr int kGateDK = 64;                          // K tile of the direct-to-LDS gate kernel
static int gate_dpad(int d) { return (int)align_up((size_t)d, kGateDK); }

size_t gate_ws_bytes(int d, int E, int dtype) {
  if (dtype != FLEXMOE_BF16) return 0;
  int nt = 1;
  while (nt * 32 < E) nt <<= 1;
  return align_up((size_t)nt * 32 * gate_dpad(d) * sizeof(bf16_t), 256);
}

// wgt[e, i] = wg[i, e] for e < E, i < d; zero in the padding (rows up to epad, columns up to ld)
__global__ void gate_transpose_wg_kernel(const bf16_t* __restrict__ wg, int d, int E, int epad, int ld,
                                         bf16_t* __restrict__ wgt) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;   // feature
  const int e = blockIdx.y;                              // expert row of the transposed copy
  if (i < ld && e < epad) wgt[(size_t)e * ld + i] = (e < E && i < d) ? wg[(size_t)i * E + e] : (bf16_t)0;
}

union Frag {
  uint4 u;
  bf16x8 v;
  bf16_t h[8];
};

// Top-k selection and softmax for one tile of 32 tokens whose logits sit in MFMA layout:
// lane (j = lane%32, h = lane/32) holds, for token j, experts r*32 + 8*(n/4) + 4*h + n%4.
template <int NT>
__device__ __forceinline__ void gate_select_store(f32x16 (&acc)[NT], int t, int N, int E, int k,
                                                  int32_t* __restrict__ topk_idx, float* __restrict__ topk_w) {
  const int h = (threadIdx.x % kWave) >> 5;
#pragma unroll
  for (int r = 0; r < NT; ++r)
#pragma unroll
    for (int n = 0; n < 16; ++n)
      if (r * 32 + 8 * (n / 4) + 4 * h + (n % 4) >= E) acc[r][n] = kNegInf;

  float sel_v[FLEXMOE_MAX_TOPK];
  int sel_e[FLEXMOE_MAX_TOPK];
#pragma unroll
  for (int p = 0; p < FLEXMOE_MAX_TOPK; ++p) {
    sel_v[p] = kNegInf;
    sel_e[p] = 0;
    if (p < k) {
      float bv = kNegInf;
      int be = 0x7fffffff;
#pragma unroll
      for (int r = 0; r < NT; ++r)
#pragma unroll
        for (int n = 0; n < 16; ++n) {          // ascending expert id: strict > keeps the lowest id on ties
          const int e = r * 32 + 8 * (n / 4) + 4 * h + (n % 4);
          if (acc[r][n] > bv) {
            bv = acc[r][n];
            be = e;
          }
        }
      const float ov = __shfl_xor(bv, 32);
      const int oe = __shfl_xor(be, 32);
      const bool mine = (bv > ov) || (bv == ov && be < oe);
      const float wv = mine ? bv : ov;
      const int we = mine ? be : oe;
#pragma unroll
      for (int r = 0; r < NT; ++r)
#pragma unroll
        for (int n = 0; n < 16; ++n)
          if (r * 32 + 8 * (n / 4) + 4 * h + (n % 4) == we) acc[r][n] = kNegInf;
      sel_v[p] = wv;
      sel_e[p] = we;
    }
  }
  if (h == 0 && t < N) {
    float ex[FLEXMOE_MAX_TOPK];
    float sum = 0.f;
#pragma unroll
    for (int p = 0; p < FLEXMOE_MAX_TOPK; ++p) {
      ex[p] = (p < k) ? expf(sel_v[p] - sel_v[0]) : 0.f;
      sum += ex[p];
    }
    const float inv = 1.f / sum;
#pragma unroll
    for (int p = 0; p < FLEXMOE_MAX_TOPK; ++p)
      if (p < k) {
        topk_idx[(size_t)t * k + p] = sel_e[p];
        topk_w[(size_t)t * k + p] = ex[p] * inv;
      }
  }
}

// ---------------------------------------------------------------------------------------------
// Direct-to-LDS gate for up to 64 experts.  One workgroup = WAVES waves x 32 tokens; K tiles of 64
// through S LDS stages (x tile [32*WAVES][64], W_g^T tile [32*NT][64], rows of 128 bytes whose
// 16-byte chunks are XORed with row & 7: conflict-free fragment reads).  A direct load writes lane
// i's 16 bytes at M0 + 16*i, i.e. eight lanes fill one row, so the swizzle is applied by choosing
// which chunk of the row a lane fetches.  Chunks past d come from a row of zeros (x) or from the
// zero padding of the transposed weights; token rows past N are clamped (their results are dropped).
// STORED: `wgt` is W_g itself, [d, E], E a multiple of four: its K tile is one contiguous piece of memory, transposed on the way out of
// LDS as in gate_quarters_kernel (no launch that writes a transposed copy: 5 us).
// S: as many stages as leave room for a second workgroup on a compute unit (65536 x 2048, 64 experts: six stages, one workgroup 49.1,
// three, two workgroups and no transposing launch 42.6 us; 32768 x 2048 38.7, 26.2; from the transposed copy, up to 32 experts the same
// as before: 40000 x 1024, 30 24.7, 24.7, 50000 x 512, 30 16.0, 16.3; more 40000 x 1024, 61 33.7, 27.2).
// ---------------------------------------------------------------------------------------------
__device__ const uint4 kGateZeroRow[8] = {};
typedef __attribute__((address_space(3))) unsigned char gate_lds_t;

// s_waitcnt vmcnt(L * tiles) only (the other counters left at "no wait"): returns once at most
// `tiles` K tiles of L direct loads each are still in flight.  The immediate must be a constant.
constexpr int gate_vmcnt_imm(int n) { return 0x0F70 | (n & 15) | ((n >> 4) << 14); }
template <int L>
__device__ __forceinline__ void gate_wait_tiles(int tiles) {   // callers keep L * tiles below 64

  switch (tiles) {
    case 0: __builtin_amdgcn_s_waitcnt(gate_vmcnt_imm(0)); break;
    case 1: __builtin_amdgcn_s_waitcnt(gate_vmcnt_imm(L)); break;
    case 2: __builtin_amdgcn_s_waitcnt(gate_vmcnt_imm(2 * L)); break;
    case 3: __builtin_amdgcn_s_waitcnt(gate_vmcnt_imm(3 * L)); break;
    case 4: __builtin_amdgcn_s_waitcnt(gate_vmcnt_imm(4 * L)); break;
    case 5: __builtin_amdgcn_s_waitcnt(gate_vmcnt_imm(5 * L)); break;
    default: __builtin_amdgcn_s_waitcnt(gate_vmcnt_imm(6 * L)); break;
  }
}

// W_g[k0 .. k0 + 7, 32 r + lane % 32] of a K tile as stored ([64][E] in LDS, rows of whole 8-byte pieces); what experts past E get is
// other rows' values, and past the tile's end the ring's: their logits are discarded.
__device__ __forceinline__ bf16x8 gate_w_tr(const gate_lds_t* tile, int k0, int r, int E, int lane) {
  typedef short s16x4 __attribute__((ext_vector_type(4)));
  typedef short s16x8 __attribute__((ext_vector_type(8)));
  const gate_lds_t* at = tile + ((k0 + ((lane & 15) >> 2)) * E + r * 32 + (lane & 16) + (lane & 3) * 4) * 2;
  const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)at);
  const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(at + 8 * E));
  return __builtin_bit_cast(bf16x8, (s16x8)__builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
}

// Quarters kernel: one workgroup per 32 tokens, wave q takes the 64-wide K chunks q, q + 4, ..  A chunk is 32 rows of x (128 bytes
// each) and 64 rows of W_g as stored, one contiguous piece of memory; both go global -> LDS with direct loads into a ring of S chunks
// of the wave's own, so nothing waits for another wave and no registers limit what is in flight.  The fragments of W_g are
// transposed on the way out of LDS, TR: by ds_read_tr16_b64 (rows of W_g are whole 8-byte pieces), else with 2-byte reads.
// What bounds it: the chunks' trips from L2, S at a time, and for the smallest batches what comes after them (sum over the
// quarters, selection).  In us, the fragments gathered from global memory with 2-byte loads (more than 64 experts: read from a transposed
// copy that a launch of its own made), and now; tokens x features, experts:
//   16 x 1024, 32 6.3, 5.1; 1500 x 1024, 32 7.3, 5.4; 256 x 2048, 64 15.6, 10.0; 8192 x 768, 16 6.5, 5.2; 16384 x 1024, 32 10.9, 6.8;
//   4096 x 512, 128 14.9, 11.1; 60000 x 2048, 100 183, 85; 4000 x 1024, 256 32.6, 23.1
// and with experts in no whole groups of four (2-byte reads) 16 x 1024, 61 8.3, 8.4; 300 x 64, 61 5.0, 5.2; 1500 x 1024, 30 7.2, 6.0; 3000 x 4096, 61 27.0,
//   21.3; 8192 x 768, 13 6.5, 5.7; 16384 x 1024, 6 11.0, 7.2; 40000 x 1024, 101 72, 40; 1500 x 1024, 250 28.2, 22.1
// and where the streaming kernel below served fewer than 32768 tokens: 12000 x 2048, 64 23.1, 14.5; 32000 x 512, 64 18.8, 12.3; 30000 x
// 2048, 32 25.1, 22.1.
template <int NT, int S, bool TR>
__global__ __launch_bounds__(4 * kWave) void gate_quarters_kernel(const bf16_t* __restrict__ x, const bf16_t* __restrict__ wg, int N,
                                                                  int d, int E, int k, int32_t* __restrict__ topk_idx,
                                                                  float* __restrict__ topk_w) {
  constexpr int kXBytes = 32 * 128, kWBytes = NT * 32 * 128, kChunk = kXBytes + kWBytes;
  constexpr int kWLoads = kWBytes / 1024, L = 4 + kWLoads;
  constexpr int kPieces = NT * 4;                       // float4 pieces of a lane's logits
  static_assert((S - 1) * L < 64, "the wait count has six bits");
  // (the fragments of experts past E reach up to 64 NT bytes past their rows)
  constexpr int kRing = 4 * S * kChunk, kSums = 4 * kPieces * kWave * 16;
  __shared__ __align__(1024) unsigned char smem[kRing > kSums ? kRing : kSums];
  const int lane = threadIdx.x % kWave, q = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int j = lane & 31, h = lane >> 5;
  const int t0 = blockIdx.x * 32;
  const int nchunks = (d + 63) / 64, n = (nchunks - q + 3) / 4;      // chunks of the wave
  const gate_lds_t* const ring = (const gate_lds_t*)smem + q * (S * kChunk);
  const unsigned lds0 = __builtin_amdgcn_readfirstlane((unsigned)(uintptr_t)ring);

  // x: instruction i covers rows 8 i .. 8 i + 7, 16-byte pieces XORed with row & 7
  const int lrow = lane >> 3, lpiece = (lane & 7) ^ lrow;
  const bf16_t* xsrc[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) xsrc[i] = x + (size_t)min(t0 + 8 * i + lrow, N - 1) * d + lpiece * 8;
  const bf16_t* const zero = (const bf16_t*)kGateZeroRow + (lane & 7) * 8;
  const long long w_all = (long long)d * E;             // (whole 16-byte pieces: d is a multiple of 8)
  auto issue = [&](int i) {
    const int c = q + 4 * i;
    const unsigned st = lds0 + i % S * kChunk;
    const bool x_ok = c * 64 + lpiece * 8 < d;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const bf16_t* g = x_ok ? xsrc[r] + c * 64 : zero;
      asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" ::"v"(g), "s"(st + r * 1024) : "memory");
    }
    const long long w0 = (long long)c * 64 * E + lane * 8;
#pragma unroll
    for (int r = 0; r < kWLoads; ++r) {
      const long long at = w0 + r * 512;
      const bf16_t* g = at < w_all ? wg + at : zero;    // past d: zeros, as in x
      asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" ::"v"(g), "s"(st + kXBytes + r * 1024) : "memory");
    }
  };

  f32x16 acc[NT];
#pragma unroll
  for (int r = 0; r < NT; ++r)
#pragma unroll
    for (int m = 0; m < 16; ++m) acc[r][m] = 0.f;
#pragma unroll
  for (int i = 0; i < S; ++i)
    if (i < n) issue(i);
  for (int i = 0; i < n; ++i) {
    gate_wait_tiles<L>(min(S - 1, n - 1 - i));
    const gate_lds_t* xs = ring + i % S * kChunk;
    const gate_lds_t* ws = xs + kXBytes;
    Frag xb[4];
#pragma unroll
    for (int s = 0; s < 4; ++s) xb[s].v = *(const __attribute__((address_space(3))) bf16x8*)(xs + j * 128 + (((s + 4 * h) ^ (j & 7)) << 4));
#pragma unroll
    for (int r = 0; r < NT; ++r) {
      Frag wa[4];                                       // W_g[64 c + 32 h + 8 s + 0..7, 32 r + j]
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        if (TR) {
          wa[s].v = gate_w_tr(ws, 32 * h + 8 * s, r, E, lane);
        } else {
          const gate_lds_t* at = ws + ((32 * h + 8 * s) * E + min(r * 32 + j, E - 1)) * 2;
#pragma unroll
          for (int m = 0; m < 8; ++m) wa[s].h[m] = *(const __attribute__((address_space(3))) bf16_t*)(at + m * 2 * E);
        }
      }
#pragma unroll
      for (int s = 0; s < 4; ++s) acc[r] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wa[s].v, xb[s].v, acc[r], 0, 0, 0);
    }
    if (i + S < n) {
      __builtin_amdgcn_s_waitcnt(0xC07F);               // lgkmcnt(0): the slot has been read
      issue(i + S);
    }
  }

  // quarter 0 + (1 + (2 + 3)), the pieces dealt to the waves
  float4(*partial)[kPieces][kWave] = (float4(*)[kPieces][kWave])smem;
  __syncthreads();                                      // every wave has left its ring
#pragma unroll
  for (int r = 0; r < NT; ++r)
#pragma unroll
    for (int m = 0; m < 4; ++m)
      partial[q][r * 4 + m][lane] = make_float4(acc[r][4 * m], acc[r][4 * m + 1], acc[r][4 * m + 2], acc[r][4 * m + 3]);
  __syncthreads();
  for (int i = q; i < kPieces; i += 4) {
    float4 v = partial[3][i][lane];
#pragma unroll
    for (int m = 2; m >= 0; --m) {
      const float4 o = partial[m][i][lane];
      v.x = o.x + v.x; v.y = o.y + v.y; v.z = o.z + v.z; v.w = o.w + v.w;
    }
    partial[0][i][lane] = v;
  }
  __syncthreads();
  if (q != 0) return;
  f32x16 l[NT];
#pragma unroll
  for (int r = 0; r < NT; ++r)
#pragma unroll
    for (int m = 0; m < 4; ++m) {
      const float4 o = partial[0][r * 4 + m][lane];
      l[r][4 * m] = o.x; l[r][4 * m + 1] = o.y; l[r][4 * m + 2] = o.z; l[r][4 * m + 3] = o.w;
    }
  gate_select_store<NT>(l, t0 + j, N, E, k, topk_idx, topk_w);
}

template <int NT, int WAVES, int S, bool STORED>
__global__ __launch_bounds__(WAVES * kWave) void gate_dma_kernel(const bf16_t* __restrict__ x,
                                                                 const bf16_t* __restrict__ wgt, int N, int d,
                                                                 int dpad, int E, int k,
                                                                 int32_t* __restrict__ topk_idx,
                                                                 float* __restrict__ topk_w) {
  constexpr int kXBytes = WAVES * 32 * 128;          // x tile
  constexpr int kWBytes = NT * 32 * 128;             // W_g^T tile
  constexpr int kStage = kXBytes + kWBytes;
  constexpr int L = 4 + (NT * 4 + WAVES - 1) / WAVES;   // direct loads per wave per K tile (x: 4, W: its share)
  static_assert(S >= 3 && S - 2 <= 6 && (S - 2) * L <= 63, "the wait count has six bits");
  __shared__ __align__(1024) unsigned char smem[S * kStage];
  const int lane = threadIdx.x % kWave, wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int j = lane & 31, h = lane >> 5;
  const int t0 = blockIdx.x * (32 * WAVES) + wave * 32;
  const int KT = dpad / kGateDK;

  // x: this wave loads its own 32 token rows: instruction q covers rows 8q .. 8q+7, lane -> (row, chunk)
  const int lrow = lane >> 3, lchunk = (lane & 7) ^ (lrow & 7);
  const bf16_t* xsrc[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) xsrc[q] = x + (size_t)min(t0 + 8 * q + lrow, N - 1) * d + lchunk * 8;
  // W: the NT*4 instructions of a tile are dealt round-robin to the waves
  constexpr int kWLoads = (NT * 4 + WAVES - 1) / WAVES;
  const bf16_t* wsrc[kWLoads];
#pragma unroll
  for (int q = 0; q < kWLoads; ++q) {
    const int instr = min(q * WAVES + wave, NT * 4 - 1);      // surplus slots repeat the last instruction (same bytes)
    wsrc[q] = STORED ? wgt + instr * 512 + lane * 8 : wgt + (size_t)(instr * 8 + lrow) * dpad + lchunk * 8;
  }
  const long long w_all = (long long)d * E;
  const bf16_t* zsrc = (const bf16_t*)kGateZeroRow + (lane & 7) * 8;
  const unsigned lds_base = __builtin_amdgcn_readfirstlane((unsigned)(uintptr_t)(gate_lds_t*)smem);

  // Workgroups start their contraction at different K tiles and wrap around, so that the requests in flight on the
  // chip are not all at the same column offset of their rows (measured: -7 % on 65536 tokens x 2048 features).
  // The order of a token's sum then depends on its workgroup, i.e. on the token's index only: still reproducible.
  const int kshift = (int)((blockIdx.x * 5u) % (unsigned)KT);
  auto issue = [&](int kt) {
    const unsigned st = lds_base + (kt % S) * kStage;
    const int ktr = kt + kshift < KT ? kt + kshift : kt + kshift - KT;
    const int k0 = ktr * kGateDK;
    const bool x_ok = k0 + lchunk * 8 < d;                    // whole 16-byte chunks: d is a multiple of 8
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const bf16_t* g = x_ok ? xsrc[q] + k0 : zsrc;
      asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" ::"v"(g), "s"(st + (wave * 4 + q) * 1024) : "memory");
    }
#pragma unroll
    for (int q = 0; q < kWLoads; ++q) {
      const int instr = min(q * WAVES + wave, NT * 4 - 1);
      const bf16_t* g;
      if (STORED) g = (long long)k0 * E + instr * 512 + lane * 8 < w_all ? wsrc[q] + (size_t)k0 * E : zsrc;      // past d: zeros
      else g = wsrc[q] + k0;
      asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" ::"v"(g), "s"(st + kXBytes + instr * 1024) : "memory");
    }
  };

  f32x16 acc[NT];
#pragma unroll
  for (int r = 0; r < NT; ++r)
#pragma unroll
    for (int n = 0; n < 16; ++n) acc[r][n] = 0.f;

#pragma unroll
  for (int p = 0; p < S - 1; ++p)
    if (p < KT) issue(p);
  for (int kt = 0; kt < KT; ++kt) {
    // tile kt has landed once at most the younger tiles are still in flight
    gate_wait_tiles<L>(min(S - 2, KT - 1 - kt));
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
    if (kt + S - 1 < KT) issue(kt + S - 1);                   // into the stage every wave has just left
    const gate_lds_t* xs = (const gate_lds_t*)smem + (kt % S) * kStage + wave * 32 * 128;
    const gate_lds_t* wsm = (const gate_lds_t*)smem + (kt % S) * kStage + kXBytes;
#pragma unroll
    for (int ks = 0; ks < kGateDK / 16; ++ks) {
      const int chunk = ((2 * ks + h) ^ (j & 7)) << 4;
      Frag xb;
      xb.v = *(const __attribute__((address_space(3))) bf16x8*)(xs + j * 128 + chunk);
#pragma unroll
      for (int r = 0; r < NT; ++r) {
        Frag wa;
        if (STORED) wa.v = gate_w_tr(wsm, 16 * ks + 8 * h, r, E, lane);
        else wa.v = *(const __attribute__((address_space(3))) bf16x8*)(wsm + (r * 32 + j) * 128 + chunk);
        acc[r] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wa.v, xb.v, acc[r], 0, 0, 0);
      }
    }
  }
  if (t0 < N) gate_select_store<NT>(acc, t0 + j, N, E, k, topk_idx, topk_w);
}

// fp32: LPT lanes per token, lane l of a token's group owns experts l, l + LPT, ... (LPT = the experts rounded up to a
// power of two, at most a wave; PER = experts per lane).  A workgroup holds up to 16 tokens; x and W_g pass through LDS in
// pieces of KC features, so that the serial FMA chain of a logit (features in ascending order) waits for LDS and not for
// memory: a wave per token that fetched each feature's weights as it needed them took 47 us on 1000 tokens x 256 features,
// 8 experts.
constexpr int kGateF32Tokens = 16;
template <int PER> struct GateF32 { static constexpr int KC = PER == 1 ? 128 : 32; };      // W_g piece: at most 32 KB
template <int PER>
__global__ __launch_bounds__(kGateThreads) void gate_f32_kernel(const float* __restrict__ x,
                                                                const float* __restrict__ wg, int N, int d, int E,
                                                                int k, int lpt, int32_t* __restrict__ topk_idx,
                                                                float* __restrict__ topk_w) {
  constexpr int KC = GateF32<PER>::KC, XS = KC + 4;      // padded x row: tokens of a wave in different banks
  __shared__ float4 xs4[kGateF32Tokens * XS / 4];
  __shared__ float4 ws4[KC * (PER == 1 ? kWave : FLEXMOE_MAX_EXPERTS) / 4];
  float* const xs = (float*)xs4;
  float* const ws = (float*)ws4;
  const int toks = blockDim.x / lpt;
  const int lane = threadIdx.x & (lpt - 1), tok = threadIdx.x / lpt;
  const int t0 = blockIdx.x * toks, t = t0 + tok;
  float l[PER];
#pragma unroll
  for (int q = 0; q < PER; ++q) l[q] = 0.f;
  for (int i0 = 0; i0 < d; i0 += KC) {
    const int kc = min(KC, d - i0);                      // a multiple of 8
    __syncthreads();
    const float4* wsrc = (const float4*)(wg + (size_t)i0 * E);
    for (int i = threadIdx.x; i < kc * E / 4; i += blockDim.x) ws4[i] = wsrc[i];
    for (int i = threadIdx.x; i < toks * (KC / 4); i += blockDim.x) {
      const int r = i / (KC / 4), c = i % (KC / 4);
      if (c * 4 < kc) xs4[r * (XS / 4) + c] = *(const float4*)(x + (size_t)min(t0 + r, N - 1) * d + i0 + c * 4);
    }
    __syncthreads();
#pragma unroll 2
    for (int i = 0; i < kc; i += 4) {
      const float4 xv = xs4[tok * (XS / 4) + i / 4];
      const float xq[4] = {xv.x, xv.y, xv.z, xv.w};
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int q = 0; q < PER; ++q) l[q] = fmaf(xq[j], ws[(i + j) * E + min(lane + q * lpt, E - 1)], l[q]);
    }
  }
#pragma unroll
  for (int q = 0; q < PER; ++q)
    if (lane + q * lpt >= E) l[q] = kNegInf;

  float sel_v[FLEXMOE_MAX_TOPK];
  int sel_e[FLEXMOE_MAX_TOPK];
#pragma unroll
  for (int p = 0; p < FLEXMOE_MAX_TOPK; ++p) {
    sel_v[p] = kNegInf;
    sel_e[p] = 0;
    if (p < k) {
      float bv = kNegInf;
      int be = 0x7fffffff;
#pragma unroll
      for (int q = 0; q < PER; ++q)
        if (l[q] > bv) {
          bv = l[q];
          be = lane + q * lpt;
        }
      for (int o = lpt / 2; o >= 1; o >>= 1) {
        const float ov = __shfl_xor(bv, o);
        const int oe = __shfl_xor(be, o);
        if (ov > bv || (ov == bv && oe < be)) {
          bv = ov;
          be = oe;
        }
      }
#pragma unroll
      for (int q = 0; q < PER; ++q)
        if (lane + q * lpt == be) l[q] = kNegInf;
      sel_v[p] = bv;
      sel_e[p] = be;
    }
  }
  if (lane == 0 && t < N) {
    float ex[FLEXMOE_MAX_TOPK];
    float sum = 0.f;
#pragma unroll
    for (int p = 0; p < FLEXMOE_MAX_TOPK; ++p) {
      ex[p] = (p < k) ? expf(sel_v[p] - sel_v[0]) : 0.f;
      sum += ex[p];
    }
    const float inv = 1.f / sum;
#pragma unroll
    for (int p = 0; p < FLEXMOE_MAX_TOPK; ++p)
      if (p < k) {
        topk_idx[(size_t)t * k + p] = sel_e[p];
        topk_w[(size_t)t * k + p] = ex[p] * inv;
      }
  }
}

hipError_t launch_gate(const void* x, const void* wg, int N, int d, int E, int k, int dtype, int32_t* idx, float* w,
                       void* ws, hipStream_t s) {
  if (N == 0) return hipSuccess;
  if (dtype == FLEXMOE_F32) {
    int lpt = 1;
    while (lpt < E && lpt < kWave) lpt <<= 1;
    const int toks = std::min(kGateF32Tokens, kGateThreads / lpt);
    const dim3 grid((N + toks - 1) / toks), block(toks * lpt);
    if (E <= kWave)
      hipLaunchKernelGGL(gate_f32_kernel<1>, grid, block, 0, s, (const float*)x, (const float*)wg, N, d, E, k, lpt, idx, w);
    else
      hipLaunchKernelGGL(gate_f32_kernel<FLEXMOE_MAX_EXPERTS / kWave>, grid, block, 0, s, (const float*)x, (const float*)wg, N, d,
                         E, k, lpt, idx, w);
    return hipGetLastError();
  }
  int nt = 1;
  while (nt * 32 < E) nt <<= 1;
  const int epad = nt * 32;
  bf16_t* wgt = (bf16_t*)ws;
  const bf16_t* xb = (const bf16_t*)x;
  if (N >= 32768 && nt <= 2) {
    // direct-to-LDS streaming, four waves (two below 65536 tokens) share a weight tile
    const int dpad = gate_dpad(d);
    const bool stored = E % 4 == 0;
    if (!stored)
      hipLaunchKernelGGL(gate_transpose_wg_kernel, dim3((dpad + 255) / 256, epad), dim3(256), 0, s, (const bf16_t*)wg, d,
                         E, epad, dpad, wgt);
#define FLEXMOE_GATE_LAUNCH(NT_, WAVES_, S_)                                                                        \
  if (stored)                                                                                                       \
    hipLaunchKernelGGL((gate_dma_kernel<NT_, WAVES_, S_, true>), dim3((N + 32 * WAVES_ - 1) / (32 * WAVES_)),        \
                       dim3(WAVES_* kWave), 0, s, xb, (const bf16_t*)wg, N, d, dpad, E, k, idx, w);                 \
  else                                                                                                              \
    hipLaunchKernelGGL((gate_dma_kernel<NT_, WAVES_, S_, false>), dim3((N + 32 * WAVES_ - 1) / (32 * WAVES_)),       \
                       dim3(WAVES_* kWave), 0, s, xb, wgt, N, d, dpad, E, k, idx, w)
    if (N >= 65536) {
      if (nt == 1) { FLEXMOE_GATE_LAUNCH(1, 4, 4); }
      else { FLEXMOE_GATE_LAUNCH(2, 4, 3); }
    } else {
      if (nt == 1) { FLEXMOE_GATE_LAUNCH(1, 2, 6); }
      else { FLEXMOE_GATE_LAUNCH(2, 2, 5); }
    }
#undef FLEXMOE_GATE_LAUNCH
    return hipGetLastError();
  }
  // One chunk per wave and ring where that is all there is, or where more workgroups than compute units (8192 tokens) hide each other's
  // trips; else as many as fit.  In us, one chunk and more: 9000 x 2048, 64 13.6, 19.7; 16500 x 1024, 64 11.9, 19.8; 32000 x 1024, 32 13.4,
  // 14.6; 20000 x 512, 128 17.6, 23.8; at most 8192 tokens the same or fewer with more chunks (4096 x 512, 128 11.2, 11.1).
  const dim3 grid((N + 31) / 32);
  const bool one = d <= 256 || N > 8192;
#define FLEXMOE_GATE_LAUNCH(NT_, S_)                                                                                                     \
  if (E % 4 == 0)                                                                                                                        \
    hipLaunchKernelGGL((gate_quarters_kernel<NT_, S_, true>), grid, dim3(4 * kWave), 0, s, xb, (const bf16_t*)wg, N, d, E, k, idx, w);   \
  else                                                                                                                                   \
    hipLaunchKernelGGL((gate_quarters_kernel<NT_, S_, false>), grid, dim3(4 * kWave), 0, s, xb, (const bf16_t*)wg, N, d, E, k, idx, w)
  if (nt == 1) {
    if (one) { FLEXMOE_GATE_LAUNCH(1, 1); }
    else { FLEXMOE_GATE_LAUNCH(1, 4); }
  } else if (nt == 2) {
    if (one) { FLEXMOE_GATE_LAUNCH(2, 1); }
    else { FLEXMOE_GATE_LAUNCH(2, 3); }
  } else if (nt == 4) {
    if (one) { FLEXMOE_GATE_LAUNCH(4, 1); }
    else { FLEXMOE_GATE_LAUNCH(4, 2); }
  } else { FLEXMOE_GATE_LAUNCH(8, 1); }
#undef FLEXMOE_GATE_LAUNCH
  return hipGetLastError();
}

}  // namespace flexmoe
