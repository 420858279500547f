// Top-k gate (paper Eq. 3): logits l = x . W_g, keep the k largest per token, softmax over them.
//
// bf16 path: HBM-bound streaming of x.  The logits come from MFMA so that the 2*d*E flops per
// token do not cap the kernel below the memory roofline: the gate weights act as the MFMA
// row operand (32 experts per tile) and 32 tokens as the column operand, hence after the
// K loop every lane holds half of one token's logits and its partner lane (lane ^ 32) the
// other half -- the top-k selection is a register scan plus one cross-lane exchange per pick.
// W_g is first transposed to [E_pad, d_pad] in the workspace (tiny, stays in L2), except in the
// small-batch kernel with up to 64 experts, which gathers its fragments from W_g as stored.
// Large batches with up to 64 experts (gate_dma_kernel): every wave owns 32 tokens and the whole contraction; x and
// W_g^T travel global -> LDS with direct loads that fetch whole 128-byte lines of a row (eight
// rows per instruction), several 64-wide K tiles in flight per workgroup, and the MFMA fragments
// are read from LDS.  Otherwise (gate_bf16_kernel): one workgroup per 32 tokens, operands read
// straight into the MFMA register layout, the contraction split over four waves (or four pairs) and the
// partial logits summed in a fixed order through LDS.
// The order of a logit's sum is part of the result: logits that differ by fp32 rounding alone decide a near tie, and with
// it a token's experts.  Below 32768 tokens, and with more than 64 experts, every kernel adds in quarters: quarter q holds
// the 64-wide K chunks q, q + 4, .., summed in ascending order, and the logit is q0 + (q1 + (q2 + q3)).  From 32768
// tokens with up to 64 experts: one sum over all chunks, from a first chunk that depends on the token's workgroup.
//
// fp32 path: a group of lanes per token, sequential fp32 FMA per logit out of LDS, butterfly arg-max per pick.
#include <algorithm>

#include "common.h"

namespace flexmoe {

constexpr int kGateThreads = 256;
constexpr float kNegInf = -__builtin_huge_valf();

static int gate_epad(int E) { return (int)align_up((size_t)E, 32); }

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

// One workgroup = 32 tokens.  The contraction is split over four wavefronts (wave w % 4 takes the 64-wide K chunks of
// quarter w % 4); with G > 1 there are G waves per quarter, each with NT / G of the expert tiles.  Then every partial logit
// is summed over the quarters through LDS, the pieces dealt to all waves, and wave 0 selects.  What bounds it is the latency
// of the chunks' round trips, one after another in a wave: where the fragments of W_g are many, a second wave per quarter
// has half of them to fetch and room for more chunks in flight (launch_gate).
// DIRECT: `wgt` is W_g itself, [d, E]: a lane gathers the eight values of a fragment with 2-byte
// loads (stride E) instead of reading a transposed copy -- 32 NT small loads per chunk from a
// matrix that sits in L2, which saves the launch that writes the copy.  Lanes of experts >= E
// re-read expert E-1 (their logits are discarded) and rows past d re-read row d-1 (x is zero there).
template <int NT, int G, bool DIRECT>   // NT tiles of 32 experts, G waves per quarter
__global__ __launch_bounds__(4 * G * kWave) void gate_bf16_kernel(const bf16_t* __restrict__ x,
                                                                 const bf16_t* __restrict__ wgt, int N, int d,
                                                                 int E, int k, int32_t* __restrict__ topk_idx,
                                                                 float* __restrict__ topk_w) {
  constexpr int W = 4, NTW = NT / G;                    // quarters; expert tiles of a wave
  constexpr int kPieces = NT * 4;                       // float4 pieces of a lane's logits
  __shared__ float4 partial[W][kPieces][kWave];
  const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave, quarter = wave % W, r0 = wave / W * NTW;
  const int j = lane & 31, h = lane >> 5;
  const int t0 = blockIdx.x * 32;

  f32x16 acc[NTW];
#pragma unroll
  for (int r = 0; r < NTW; ++r)
#pragma unroll
    for (int n = 0; n < 16; ++n) acc[r][n] = 0.f;

  const bf16_t* xrow = x + (size_t)min(t0 + j, N - 1) * d + 32 * h;   // clamp the ragged last tile
  const bf16_t* wrow = wgt + (size_t)(r0 * 32 + j) * d + 32 * h;
  const int nchunks = (d + 63) / 64;
  // DIRECT: column of W_g for the lane's expert in tile r, at row 32 h
  const bf16_t* wcol[NTW];
#pragma unroll
  for (int r = 0; r < NTW; ++r) wcol[r] = wgt + (size_t)(32 * h) * E + min((r0 + r) * 32 + j, E - 1);
  auto gather_w = [&](int r, int k0, bool full) -> uint4 {        // W_g[k0 + 32 h + 0..7, expert]
    Frag f;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int kk = full ? k0 + i : min(k0 + i, d - 1 - 32 * h);
      f.h[i] = wcol[r][(size_t)kk * E];
    }
    return f.u;
  };

  // lane reads k = 64c + 32h + 8s .. +8 of its row for s = 0..3 (64 contiguous bytes); pieces past d are zero
  auto load_chunk = [&](int c, Frag (&xb)[4], Frag (&wa)[NTW][4]) {
    if (c * 64 + 64 <= d) {
#pragma unroll
      for (int s = 0; s < 4; ++s) xb[s].u = *(const uint4*)(xrow + c * 64 + s * 8);
#pragma unroll
      for (int r = 0; r < NTW; ++r)
#pragma unroll
        for (int s = 0; s < 4; ++s)
          wa[r][s].u = DIRECT ? gather_w(r, c * 64 + s * 8, true) : *(const uint4*)(wrow + (size_t)r * 32 * d + c * 64 + s * 8);
    } else {
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        const bool ok = c * 64 + 32 * h + s * 8 < d;
        xb[s].u = ok ? *(const uint4*)(xrow + c * 64 + s * 8) : make_uint4(0, 0, 0, 0);
#pragma unroll
        for (int r = 0; r < NTW; ++r) {
          if (DIRECT) wa[r][s].u = gather_w(r, c * 64 + s * 8, false);
          else wa[r][s].u = ok ? *(const uint4*)(wrow + (size_t)r * 32 * d + c * 64 + s * 8) : make_uint4(0, 0, 0, 0);
        }
      }
    }
  };
  auto mma_chunk = [&](const Frag (&xb)[4], const Frag (&wa)[NTW][4]) {
#pragma unroll
    for (int r = 0; r < NTW; ++r)
#pragma unroll
      for (int s = 0; s < 4; ++s) acc[r] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wa[r][s].v, xb[s].v, acc[r], 0, 0, 0);
  };

  // chunks of loads in flight per wave (register sets used in rotation), as many as the registers hold
  constexpr int kSets = NTW == 8 ? 1 : NTW == 4 ? 2 : 3;
  Frag xb[kSets][4], wa[kSets][NTW][4];
  int c = quarter;
#pragma unroll
  for (int q = 0; q < kSets; ++q)
    if (c + W * q < nchunks) load_chunk(c + W * q, xb[q], wa[q]);
  for (; c < nchunks; c += W * kSets) {
#pragma unroll
    for (int q = 0; q < kSets; ++q)
      if (c + W * q < nchunks) {
        mma_chunk(xb[q], wa[q]);
        if (c + W * (q + kSets) < nchunks) load_chunk(c + W * (q + kSets), xb[q], wa[q]);
      }
  }

  // quarter 0 + (1 + (2 + 3)), the pieces dealt to the waves
#pragma unroll
  for (int r = 0; r < NTW; ++r)
#pragma unroll
    for (int q = 0; q < 4; ++q)
      partial[quarter][(r0 + r) * 4 + q][lane] = make_float4(acc[r][4 * q], acc[r][4 * q + 1], acc[r][4 * q + 2], acc[r][4 * q + 3]);
  __syncthreads();
  for (int i = wave; i < kPieces; i += W * G) {
    float4 v = partial[W - 1][i][lane];
#pragma unroll
    for (int q = W - 2; q >= 0; --q) {
      const float4 o = partial[q][i][lane];
      v.x = o.x + v.x; v.y = o.y + v.y; v.z = o.z + v.z; v.w = o.w + v.w;
    }
    partial[0][i][lane] = v;
  }
  __syncthreads();
  if (wave != 0) return;
  f32x16 l[NT];
#pragma unroll
  for (int r = 0; r < NT; ++r)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const float4 o = partial[0][r * 4 + q][lane];
      l[r][4 * q] = o.x; l[r][4 * q + 1] = o.y; l[r][4 * q + 2] = o.z; l[r][4 * q + 3] = o.w;
    }
  gate_select_store<NT>(l, t0 + j, N, E, k, topk_idx, topk_w);
}

// ---------------------------------------------------------------------------------------------
// Direct-to-LDS gate for up to 64 experts.  One workgroup = WAVES waves x 32 tokens; K tiles of 64
// through S LDS stages (x tile [32*WAVES][64], W_g^T tile [32*NT][64], rows of 128 bytes whose
// 16-byte chunks are XORed with row & 7: conflict-free fragment reads).  A direct load writes lane
// i's 16 bytes at M0 + 16*i, i.e. eight lanes fill one row, so the swizzle is applied by choosing
// which chunk of the row a lane fetches.  Chunks past d come from a row of zeros (x) or from the
// zero padding of the transposed weights; token rows past N are clamped (their results are dropped).
// QUARTERS: one accumulator per quarter of the chunks and gate_bf16_kernel's fragments, so that a token's logits are the
// same bits in either kernel.
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

template <int NT, int WAVES, int S, bool QUARTERS>
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
    wsrc[q] = wgt + (size_t)(instr * 8 + lrow) * dpad + lchunk * 8;
  }
  const bf16_t* zsrc = (const bf16_t*)kGateZeroRow + (lane & 7) * 8;
  const unsigned lds_base = __builtin_amdgcn_readfirstlane((unsigned)(uintptr_t)(gate_lds_t*)smem);

  // Workgroups start their contraction at different K tiles and wrap around, so that the requests in flight on the
  // chip are not all at the same column offset of their rows (measured: -7 % on 65536 tokens x 2048 features).
  // The order of a token's sum then depends on its workgroup, i.e. on the token's index only: still reproducible.
  const int kshift = QUARTERS ? 0 : (int)((blockIdx.x * 5u) % (unsigned)KT);
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
      const bf16_t* g = wsrc[q] + k0;
      asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" ::"v"(g), "s"(st + kXBytes + instr * 1024) : "memory");
    }
  };

  constexpr int Q = QUARTERS ? 4 : 1;
  f32x16 acc[Q][NT];
#pragma unroll
  for (int q = 0; q < Q; ++q)
#pragma unroll
    for (int r = 0; r < NT; ++r)
#pragma unroll
      for (int n = 0; n < 16; ++n) acc[q][r][n] = 0.f;

#pragma unroll
  for (int p = 0; p < S - 1; ++p)
    if (p < KT) issue(p);
  for (int kt0 = 0; kt0 < KT; kt0 += Q) {
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const int kt = kt0 + q;
      if (kt >= KT) break;
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
        const int chunk = ((QUARTERS ? ks + 4 * h : 2 * ks + h) ^ (j & 7)) << 4;
        Frag xb;
        xb.v = *(const __attribute__((address_space(3))) bf16x8*)(xs + j * 128 + chunk);
#pragma unroll
        for (int r = 0; r < NT; ++r) {
          Frag wa;
          wa.v = *(const __attribute__((address_space(3))) bf16x8*)(wsm + (r * 32 + j) * 128 + chunk);
          acc[q][r] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wa.v, xb.v, acc[q][r], 0, 0, 0);
        }
      }
    }
  }
  f32x16 l[NT];
#pragma unroll
  for (int r = 0; r < NT; ++r)
#pragma unroll
    for (int n = 0; n < 16; ++n)
      l[r][n] = QUARTERS ? acc[0][r][n] + (acc[1 % Q][r][n] + (acc[2 % Q][r][n] + acc[3 % Q][r][n])) : acc[0][r][n];
  if (t0 < N) gate_select_store<NT>(l, t0 + j, N, E, k, topk_idx, topk_w);
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

// From which size the streaming kernel is ahead: where the split-K kernel needs another round.  Its registers leave a compute
// unit one workgroup with 33 to 64 experts (8192 tokens a round), three below (24576; the second workgroup of a compute unit
// already costs as much as streaming from 2048 features on).  Below 256 features the launch that transposes W_g eats it up.  In us,
// split-K and streaming, tokens x features:
//   64 experts: 9000 x 64 7.6, 6.8; 9000 x 2048 30.8, 22.5; 17000 x 1024 26.6, 25.1; 32000 x 64 14.1, 10.3; but 17000 x 512 17.3, 17.2
//   32 experts: 25000 x 256 7.4, 7.1; 25000 x 1024 17.1, 13.4; 32000 x 512 11.5, 9.5; 17000 x 2048 22.2, 20.2;
//               past the line: 25000 x 128 6.1, 6.2; 32000 x 64 5.7, 5.9; 17000 x 1024 12.7, 12.9; 20000 x 512 7.8, 10.1; 17000 x 64 4.3, 5.7
static bool gate_streams(int N, int d, int nt) {
  if (nt > 2) return false;
  return N >= 32768 || (nt == 2 ? N > 8192 : d >= 2048 ? N > 16384 : d >= 256 && N > 24576);
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
  if (gate_streams(N, d, nt)) {
    // large batches: direct-to-LDS streaming, four waves (two below 65536 tokens) share a weight tile
    const int dpad = gate_dpad(d);
    hipLaunchKernelGGL(gate_transpose_wg_kernel, dim3((dpad + 255) / 256, epad), dim3(256), 0, s, (const bf16_t*)wg, d,
                       E, epad, dpad, wgt);
#define FLEXMOE_GATE_LAUNCH(NT_, WAVES_, S_, Q_)                                                                   \
  hipLaunchKernelGGL((gate_dma_kernel<NT_, WAVES_, S_, Q_>), dim3((N + 32 * WAVES_ - 1) / (32 * WAVES_)),            \
                     dim3(WAVES_* kWave), 0, s, xb, wgt, N, d, dpad, E, k, idx, w)
    if (N >= 65536) {
      if (nt == 1) FLEXMOE_GATE_LAUNCH(1, 4, 6, false);
      else FLEXMOE_GATE_LAUNCH(2, 4, 6, false);
    } else if (N >= 32768) {
      if (nt == 1) FLEXMOE_GATE_LAUNCH(1, 2, 6, false);
      else FLEXMOE_GATE_LAUNCH(2, 2, 6, false);
    } else {
      if (nt == 1) FLEXMOE_GATE_LAUNCH(1, 2, 6, true);
      else FLEXMOE_GATE_LAUNCH(2, 2, 6, true);
    }
#undef FLEXMOE_GATE_LAUNCH
    return hipGetLastError();
  }
  // small batches (a few waves per compute unit at most) and more than 64 experts: split-K kernel.
  // Two waves per quarter with 33 to 64 experts and several rounds of chunks (one, two; us; 64 experts): 256 x 2048 20.6,
  // 15.6; 12000 x 2048 49.8, 32.9; 32000 x 1024 42.5, 36.2; but 16000 x 512 13.2, 13.4.  With more experts two waves lose what the
  // smaller fragments win: 4096 x 1024, 128 experts 19.6, 20.7; 2000 x 2048, 100 experts 26.3, 29.2.
  const dim3 grid((N + 31) / 32);
  const int g = d >= 512 && nt == 2 ? 2 : 1;
  const bool direct = nt <= 2;      // the fragments of W_g are gathered from the matrix as stored (one launch)
  if (!direct)
    hipLaunchKernelGGL(gate_transpose_wg_kernel, dim3((d + 255) / 256, epad), dim3(256), 0, s, (const bf16_t*)wg, d, E, epad, d, wgt);
  const bf16_t* wgb = direct ? (const bf16_t*)wg : wgt;
#define FLEXMOE_GATE_LAUNCH(NT_, G_, DIRECT_) \
  hipLaunchKernelGGL((gate_bf16_kernel<NT_, G_, DIRECT_>), grid, dim3(4 * G_ * kWave), 0, s, xb, wgb, N, d, E, k, idx, w)
  switch (nt * 10 + g) {
    case 11: FLEXMOE_GATE_LAUNCH(1, 1, true); break;
    case 21: FLEXMOE_GATE_LAUNCH(2, 1, true); break;
    case 22: FLEXMOE_GATE_LAUNCH(2, 2, true); break;
    case 41: FLEXMOE_GATE_LAUNCH(4, 1, false); break;
    default: FLEXMOE_GATE_LAUNCH(8, 1, false); break;
  }
#undef FLEXMOE_GATE_LAUNCH
  return hipGetLastError();
}

}  // namespace flexmoe
