// fp32 expert FFN (paper Eq. 2) forward and backward per vExpert bucket, on the fp32 matrix instruction
// v_mfma_f32_16x16x4_f32 (fp32 operands, products and sums).
//
// One workgroup of four waves per tile of outputs.  64 x 64: a wave per 32 x 32 (four independent accumulators).  32 x 64, where 64 x 64
// tiles would leave most of the chip without work: two waves per 32 x 32, one for the even 32-wide K tiles and one for the odd, whose
// sums are added at the end.  K tiles travel global -> LDS with direct loads through four (three) stages; two workgroups per compute
// unit.  Within sixteen k an instruction's lane groups hold four consecutive ones each, so that a K-contiguous operand is read
// from LDS as 16-byte vectors.  Every sum is that of the even K tiles in ascending order plus that of the odd ones, whichever tile it
// belongs to: a row's outputs do not depend on how many other rows there are.
//
// What bounds it: 1024 cycles of matrix instructions per K tile and wave where the chip is full (4352 tiles: 207 us for [8192, 512] x
// [512, 2048], 83 TFLOP/s of 157), else what a workgroup does before its first K tile, the K tiles' latency, and workgroups that do not
// come out even over the compute units.  With 64 x 64 tiles alone, loads behind a branch each and two trips to memory before the first
// one: fp32 training step of 1000 tokens (d 256, f 1024, 8 experts) 30, 29, 31, 27 us for its rows products and 28, 28 for its weight
// gradients, now 26, 25, 25, 24 and 22, 21; 8192 rows of 8 experts (d 512, f 2048) 215, 216, 226, 219, 204, 203 -> 206, 203, 216, 197, 197, 195; 200
// rows of that layer 24, 50, 25, 48, 18, 17 -> 16, 26, 15, 25, 18, 18; weight gradients of one expert with 8192 rows (d 128, f 512) 216 -> 111.
#include <algorithm>
#include <type_traits>

#include "common.h"

namespace flexmoe {

constexpr int kF32Threads = 256;
constexpr int FN = 64, FK = 32;                      // columns of a tile, contraction indices of a K tile

enum { EPI_FWD1 = 0, EPI_PLAIN = 1, EPI_DH = 2 };

typedef __attribute__((address_space(3))) unsigned char lds_t;
__device__ const float4 kF32Zero = {0.f, 0.f, 0.f, 0.f};

__device__ __forceinline__ void f32_load(const float* p, unsigned lds) {
  asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" ::"v"(p), "s"(lds) : "memory");
}
template <int N> __device__ __forceinline__ void f32_wait_vmcnt() { __builtin_amdgcn_s_waitcnt(0x0F70 | (N & 15) | ((N >> 4) << 14)); }

// One operand's K tile in LDS, W outputs wide.  KC (K-contiguous): [W][32 k], rows of eight 16-byte chunks, chunk index XOR row & 7.
// K-strided: [32 k][W]; an instruction's four lane groups read rows four apart, 16 outputs (64 bytes) each, which must lie in different
// banks: 64 wide, chunk index XOR 4 ((k / 4) % 4); 32 wide (half the banks), chunk index XOR 4 ((k / 4) % 2), neighbouring rows swapped
// where k & 8.
template <bool KC, int W> struct F32Op {
  static constexpr int kBytes = W * FK * 4;
  static constexpr int kPieces = kBytes / 1024;      // direct loads
  // output (row or column) and k that the lane fetches in piece i, four of the contiguous ones from there
  static __device__ __forceinline__ int out(int i, int lane) {
    if (KC) return i * 8 + (lane >> 3);
    if (W == 64) return ((lane & 15) ^ (((k(i, lane) >> 2) & 3) << 2)) * 4;
    return ((lane & 7) ^ (((k(i, lane) >> 2) & 1) << 2)) * 4;
  }
  static __device__ __forceinline__ int k(int i, int lane) {
    if (KC) return ((lane & 7) ^ (lane >> 3)) * 4;
    if (W == 64) return i * 4 + (lane >> 4);
    const int p = i * 8 + (lane >> 3);
    return p ^ ((p >> 3) & 1);
  }
  // four k of output base + lane % 16: k = 16 kk + 4 (lane / 16) ..
  static __device__ __forceinline__ void frag(float (&f)[4], const lds_t* tile, int base, int kk, int lane) {
    const int r = base + (lane & 15), g = lane >> 4;
    if (KC) {
      const f32x4 v = *(const __attribute__((address_space(3))) f32x4*)(tile + r * 128 + (((4 * kk + g) ^ (r & 7)) << 4));
#pragma unroll
      for (int j = 0; j < 4; ++j) f[j] = v[j];
    } else {
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int kr = 16 * kk + 4 * g + j;
        const lds_t* at = W == 64 ? tile + kr * 256 + (((r >> 2) ^ (g << 2)) << 4) + (r & 3) * 4
                                  : tile + (kr ^ (g >> 1)) * 128 + (((r >> 2) ^ ((g & 1) << 2)) << 4) + (r & 3) * 4;
        f[j] = *(const __attribute__((address_space(3))) float*)at;
      }
    }
  }
};

typedef f32x4 F32Acc[2][2];                          // a wave's 32 x 32 outputs: 16-row and 16-column blocks

// A workgroup's K loop: MT 32-row blocks x 64 columns.  MT == 2: a wave per 32 x 32 outputs.  MT == 1: two waves per 32 x 32 outputs,
// one for the even K tiles, one for the odd ones.  A stage holds 3 - MT K tiles.
template <int MT, bool KC0, bool KC1> struct F32Loop {
  typedef F32Op<KC0, MT * 32> Op0;
  typedef F32Op<KC1, FN> Op1;
  static constexpr int kSub = 3 - MT;                // K tiles of a stage
  static constexpr int kSubBytes = Op0::kBytes + Op1::kBytes;
  static constexpr int kStageBytes = kSub * kSubBytes;
  static constexpr int S = MT == 2 ? 4 : 3;
  static constexpr int kL0 = kSub * Op0::kPieces / 4, kL1 = kSub * Op1::kPieces / 4, kLoads = kL0 + kL1;      // direct loads per wave and stage
  static constexpr int kLds = S * kStageBytes;
  // the wave's q-th load of either operand: K tile of the stage, piece
  static __device__ __forceinline__ int sub0(int wave, int q) { return (wave * kL0 + q) / Op0::kPieces; }
  static __device__ __forceinline__ int piece0(int wave, int q) { return (wave * kL0 + q) % Op0::kPieces; }
  static __device__ __forceinline__ int sub1(int wave, int q) { return (wave * kL1 + q) / Op1::kPieces; }
  static __device__ __forceinline__ int piece1(int wave, int q) { return (wave * kL1 + q) % Op1::kPieces; }
  static __device__ __forceinline__ unsigned dst0(int wave, int q) { return sub0(wave, q) * kSubBytes + piece0(wave, q) * 1024; }
  static __device__ __forceinline__ unsigned dst1(int wave, int q) { return sub1(wave, q) * kSubBytes + Op0::kBytes + piece1(wave, q) * 1024; }

  // stage kt is in LDS, and every wave has left the one before it
  static __device__ __forceinline__ void ready(int kt, int KT) {
    switch (min(S - 2, KT - 1 - kt)) {               // younger stages in flight
      case 0: f32_wait_vmcnt<0>(); break;
      case 1: f32_wait_vmcnt<kLoads>(); break;
      default: f32_wait_vmcnt<2 * kLoads>(); break;
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
  }
  static __device__ __forceinline__ void multiply(const lds_t* st, F32Acc& acc, int wave, int lane) {
#pragma unroll
    for (int kk = 0; kk < FK / 16; ++kk) {
      float a[2][4], b[2][4];
#pragma unroll
      for (int i = 0; i < 2; ++i) Op0::frag(a[i], st, (MT == 2 ? (wave >> 1) * 32 : 0) + i * 16, kk, lane);
#pragma unroll
      for (int j = 0; j < 2; ++j) Op1::frag(b[j], st + Op0::kBytes, (wave & 1) * 32 + j * 16, kk, lane);
#pragma unroll
      for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int j = 0; j < 2; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(b[j][q], a[i][q], acc[i][j], 0, 0, 0);
    }
  }

  // KT stages; issue(s, lds address) starts the wave's loads of one.
  // acc[i][j]: row 16 i + lane % 16, columns 16 j + 4 (lane / 16) .. of the wave's block.  MT == 1: on return the wave with the even K tiles
  // has the sums of the block's first 16 columns, the other one of the rest.
  // Either way a sum is that of the even K tiles, ascending, plus that of the odd ones: MT == 2 keeps the two in accumulators of their own.
  template <typename Issue>
  static __device__ __forceinline__ void run(lds_t* sm, F32Acc& acc, int KT, Issue issue) {
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const unsigned lds0 = __builtin_amdgcn_readfirstlane((unsigned)(uintptr_t)sm);
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
    for (int s = 0; s < min(S - 1, KT); ++s) issue(s, lds0 + s * kStageBytes);
    if (MT == 2) {
      F32Acc odd;
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) odd[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
      for (int kt = 0; kt < KT; kt += 2) {
        ready(kt, KT);
        if (kt + S - 1 < KT) issue(kt + S - 1, lds0 + (kt + S - 1) % S * kStageBytes);
        multiply(sm + kt % S * kStageBytes, acc, wave, lane);
        if (kt + 1 == KT) break;
        ready(kt + 1, KT);
        if (kt + S < KT) issue(kt + S, lds0 + (kt + S) % S * kStageBytes);
        multiply(sm + (kt + 1) % S * kStageBytes, odd, wave, lane);
      }
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] += odd[i][j];
    } else {
      for (int kt = 0; kt < KT; ++kt) {
        ready(kt, KT);
        if (kt + S - 1 < KT) issue(kt + S - 1, lds0 + (kt + S - 1) % S * kStageBytes);
        multiply(sm + kt % S * kStageBytes + (wave >> 1) * kSubBytes, acc, wave, lane);
      }
    }
    if (MT == 1) {
      // the two waves of a block trade the halves they do not keep (even K tiles + odd K tiles, in either)
      __syncthreads();
      typedef __attribute__((address_space(3))) f32x4* Ptr;
      const int keep = wave >> 1;
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const f32x4 first = acc[i][0], second = acc[i][1];
        *(Ptr)(sm + ((wave * 2 + i) * kWave + lane) * 16) = keep ? first : second;
      }
      __syncthreads();
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const f32x4 v = *(Ptr)(sm + (((wave ^ 2) * 2 + i) * kWave + lane) * 16);      // (even K tiles + odd ones, in either wave)
        acc[i][0] += v;
        acc[i][1] += v;
      }
    }
  }
};

// Workgroup -> {first row, rows, expert} of an FM-row tile of the bucket list, and column tile; one wave scans the buckets'
// tile counts (all that it needs of them in one trip to memory).  False (for the whole workgroup): beyond the last tile.
// Workgroups are dealt round-robin to the XCDs; XCD x takes the x-th eighth of the tiles, row tile by row tile, so that rows and
// weights come into one L2 or two and not into all eight.
constexpr unsigned kF32Xcds = 8;
template <int FM>
__device__ __forceinline__ bool f32_tile(const int32_t* __restrict__ voff, const int32_t* __restrict__ owner, int V, int col_tiles,
                                         int* s_tile, int* row0, int* rows, int* e, int* ct) {
  if (threadIdx.x < kWave) {
    const int lane = threadIdx.x;
    if (lane == 0) s_tile[0] = -1;
    const unsigned x = blockIdx.x % kF32Xcds;
    auto scan = [&](auto per_lane) {                 // buckets per lane
      constexpr int kPer = decltype(per_lane)::value;
      int lo[kPer], hi[kPer], own[kPer], sum = 0;
#pragma unroll
      for (int q = 0; q < kPer; ++q) {
        const int v = lane * kPer + q;
        lo[q] = voff[min(v, V)];
        hi[q] = voff[min(v + 1, V)];
        own[q] = owner[min(v, V - 1)];
      }
#pragma unroll
      for (int q = 0; q < kPer; ++q) sum += (hi[q] - lo[q] + FM - 1) / FM;
      int incl = sum;
#pragma unroll
      for (int o = 1; o < kWave; o <<= 1) {
        const int up = __shfl_up(incl, o);
        if (lane >= o) incl += up;
      }
      const unsigned long long tiles = (unsigned long long)(unsigned)__builtin_amdgcn_readlane(incl, kWave - 1) * (unsigned)col_tiles;
      const unsigned t = (unsigned)(tiles * x / kF32Xcds) + blockIdx.x / kF32Xcds;
      const int rt = t < (unsigned)(tiles * (x + 1) / kF32Xcds) ? (int)(t / (unsigned)col_tiles) : -1;
      if (lane == 0) s_tile[3] = (int)(t % (unsigned)col_tiles);
      int start = incl - sum;
#pragma unroll
      for (int q = 0; q < kPer; ++q) {
        const int n = (hi[q] - lo[q] + FM - 1) / FM;
        if (rt >= start && rt < start + n) {
          s_tile[0] = lo[q] + (rt - start) * FM;
          s_tile[1] = min(FM, hi[q] - s_tile[0]);
          s_tile[2] = own[q];
        }
        start += n;
      }
    };
    if (V <= kWave) scan(std::integral_constant<int, 1>{});
    else scan(std::integral_constant<int, FLEXMOE_MAX_VEXPERTS / kWave>{});
  }
  __syncthreads();
  *row0 = __builtin_amdgcn_readfirstlane(s_tile[0]);
  *rows = __builtin_amdgcn_readfirstlane(s_tile[1]);
  *e = __builtin_amdgcn_readfirstlane(s_tile[2]);
  *ct = __builtin_amdgcn_readfirstlane(s_tile[3]);
  return *row0 >= 0;
}

// C[p, n] = sum_k In[p, k] * W_e[k, n]   (WT == false, W_e is [K, NC])
//         = sum_k In[p, k] * W_e[n, k]   (WT == true,  W_e is [NC, K])
// for `col_tiles` tiles of 64 columns from tile ct0 on.
template <int MT, bool WT, int EPI>
__global__ __launch_bounds__(kF32Threads, 2) void rows_gemm_f32(const float* __restrict__ in, const float* __restrict__ w,
                                                                const float* __restrict__ bias,
                                                                const int32_t* __restrict__ voff,
                                                                const int32_t* __restrict__ owner, int V, int K, int NC,
                                                                int ct0, int col_tiles, int act, const float* __restrict__ hpre_in,
                                                                float* __restrict__ out0, float* __restrict__ out1) {
  typedef F32Loop<MT, true, WT> Loop;
  __shared__ __align__(1024) unsigned char smem[Loop::kLds];
  __shared__ int s_tile[4];
  int row0, rows, e, ct;
  if (!f32_tile<MT * 32>(voff, owner, V, col_tiles, s_tile, &row0, &rows, &e, &ct)) return;
  const int n0 = (ct0 + ct) * FN, cols = min(FN, NC - n0);
  const float* we = w + (size_t)e * K * NC;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;

  // the lane's loads, from the tile's first row and column on
  const float* const a_base = in + (size_t)row0 * K;
  const float* const w_base = we + (WT ? (size_t)n0 * K : (size_t)n0);
  size_t aoff[Loop::kL0], woff[Loop::kL1];
  int ak[Loop::kL0], wk[Loop::kL1];                  // k (in the stage) of the lane's first element
#pragma unroll
  for (int q = 0; q < Loop::kL0; ++q) {
    const int i = Loop::piece0(wave, q);
    ak[q] = Loop::sub0(wave, q) * FK + Loop::Op0::k(i, lane);
    aoff[q] = (uint64_t)(uint32_t)min(Loop::Op0::out(i, lane), rows - 1) * (uint32_t)K + ak[q];
  }
#pragma unroll
  for (int q = 0; q < Loop::kL1; ++q) {
    const int i = Loop::piece1(wave, q);
    wk[q] = Loop::sub1(wave, q) * FK + Loop::Op1::k(i, lane);
    woff[q] = WT ? (uint64_t)(uint32_t)min(Loop::Op1::out(i, lane), cols - 1) * (uint32_t)K + wk[q]
                 : (uint64_t)(uint32_t)wk[q] * (uint32_t)NC + min(Loop::Op1::out(i, lane), cols - 4);
  }
  constexpr int kStep = Loop::kSub * FK;
  auto issue = [&](int s, unsigned lds) {
    const int k0 = s * kStep;
    const float *ab = a_base + k0, *wb = w_base + (WT ? (size_t)k0 : (size_t)k0 * NC);
    if (k0 + kStep <= K) {
#pragma unroll
      for (int q = 0; q < Loop::kL0; ++q) f32_load(ab + aoff[q], lds + Loop::dst0(wave, q));
#pragma unroll
      for (int q = 0; q < Loop::kL1; ++q) f32_load(wb + woff[q], lds + Loop::dst1(wave, q));
    } else {                                         // past K: zeros
#pragma unroll
      for (int q = 0; q < Loop::kL0; ++q) f32_load(k0 + ak[q] < K ? ab + aoff[q] : (const float*)&kF32Zero, lds + Loop::dst0(wave, q));
#pragma unroll
      for (int q = 0; q < Loop::kL1; ++q) f32_load(k0 + wk[q] < K ? wb + woff[q] : (const float*)&kF32Zero, lds + Loop::dst1(wave, q));
    }
  };
  F32Acc acc;
  Loop::run((lds_t*)smem, acc, (K + kStep - 1) / kStep, issue);

  auto row_at = [&](int x) { return (MT == 2 ? (wave >> 1) * 32 : 0) + (x >> 1) * 16 + (lane & 15); };
  auto col_at = [&](int x) { return n0 + (wave & 1) * 32 + (x & 1) * 16 + 4 * (lane >> 4); };
  auto stored = [&](int x) { return row_at(x) < rows && col_at(x) < NC && (MT == 2 || (x & 1) == (wave >> 1)); };
  float4 hp[4];
  if (EPI == EPI_DH) {              // (one trip to memory, not one after another)
#pragma unroll
    for (int x = 0; x < 4; ++x)
      if (stored(x)) hp[x] = *(const float4*)(hpre_in + (size_t)(row0 + row_at(x)) * NC + col_at(x));
  }
#pragma unroll
  for (int x = 0; x < 4; ++x) {
    if (!stored(x)) continue;
    const int i = x >> 1, j = x & 1, col = col_at(x);
    const size_t o = (size_t)(row0 + row_at(x)) * NC + col;
    float c[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) c[q] = acc[i][j][q];
    if (bias) {
      const float4 b = *(const float4*)(bias + (size_t)e * NC + col);
      c[0] += b.x; c[1] += b.y; c[2] += b.z; c[3] += b.w;
    }
    if (EPI == EPI_FWD1) {          // out0 = pre-activation (kept), out1 = activation
      if (out0) *(float4*)(out0 + o) = make_float4(c[0], c[1], c[2], c[3]);
      *(float4*)(out1 + o) = make_float4(act_apply(c[0], act), act_apply(c[1], act), act_apply(c[2], act), act_apply(c[3], act));
    } else if (EPI == EPI_PLAIN) {
      *(float4*)(out0 + o) = make_float4(c[0], c[1], c[2], c[3]);
    } else {                        // out0 = dHpre, out1 = act(Hpre) unless the forward pass kept it
      const float4 z = hp[x];
      *(float4*)(out0 + o) = make_float4(c[0] * act_deriv(z.x, act), c[1] * act_deriv(z.y, act), c[2] * act_deriv(z.z, act),
                                         c[3] * act_deriv(z.w, act));
      if (out1) *(float4*)(out1 + o) = make_float4(act_apply(z.x, act), act_apply(z.y, act), act_apply(z.z, act), act_apply(z.w, act));
    }
  }
}

// dW_e[m, n] = sum over the vExperts v of e (ascending v), rows p of v: L[p, m] * R[p, n].  The rows of all of the
// expert's buckets are one contraction: K tile kt holds rows 32 kt .. of the buckets laid behind each other.  Output rows from m_first on.
template <int MT>
__global__ __launch_bounds__(kF32Threads, 2) void wgrad_f32(const float* __restrict__ L, const float* __restrict__ R,
                                                            const int32_t* __restrict__ voff,
                                                            const int32_t* __restrict__ owner, int V, int M, int NC,
                                                            int m_first, float* __restrict__ dw) {
  typedef F32Loop<MT, false, false> Loop;
  __shared__ __align__(1024) unsigned char smem[Loop::kLds];
  __shared__ int s_first[FLEXMOE_MAX_VEXPERTS], s_end[FLEXMOE_MAX_VEXPERTS];      // first row - rows before it, rows up to its end
  __shared__ int s_n;
  const int e = blockIdx.z, m0 = m_first + (int)blockIdx.y * (MT * 32), n0 = blockIdx.x * FN;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (wave == 0) {                  // the expert's non-empty buckets, ascending
    int n = 0, total = 0;
    for (int v0 = 0; v0 < V; v0 += kWave) {
      const int v = v0 + lane;
      const bool mine = v < V && owner[v] == e;
      const int lo = mine ? voff[v] : 0, len = mine ? voff[v + 1] - lo : 0;
      int incl = len;
#pragma unroll
      for (int o = 1; o < kWave; o <<= 1) {
        const int up = __shfl_up(incl, o);
        if (lane >= o) incl += up;
      }
      const unsigned long long has = __ballot(len > 0);
      if (len > 0) {
        const int at = n + __popcll(has & ((1ull << lane) - 1));
        s_first[at] = lo - (total + incl - len);
        s_end[at] = total + incl;
      }
      n += __popcll(has);
      total += __shfl(incl, kWave - 1);
    }
    if (lane == 0) s_n = n;
  }
  __syncthreads();
  const int nb = s_n, T = nb ? s_end[nb - 1] : 0;

  constexpr int kStep = Loop::kSub * FK;
  size_t loff[Loop::kL0], roff[Loop::kL1];           // the lane's loads, from a stage's first row
#pragma unroll
  for (int q = 0; q < Loop::kL0; ++q) {
    const int i = Loop::piece0(wave, q), k = Loop::sub0(wave, q) * FK + Loop::Op0::k(i, lane);
    loff[q] = (uint64_t)(uint32_t)k * (uint32_t)M + min(m0 + Loop::Op0::out(i, lane), M - 4);
  }
#pragma unroll
  for (int q = 0; q < Loop::kL1; ++q) {
    const int i = Loop::piece1(wave, q), k = Loop::sub1(wave, q) * FK + Loop::Op1::k(i, lane);
    roff[q] = (uint64_t)(uint32_t)k * (uint32_t)NC + min(n0 + Loop::Op1::out(i, lane), NC - 4);
  }
  int bu = 0, bu_end = 0, bu_first = 0;              // bucket of a stage's first row
  if (nb) {
    bu_end = __builtin_amdgcn_readfirstlane(s_end[0]);
    bu_first = __builtin_amdgcn_readfirstlane(s_first[0]);
  }
  auto issue = [&](int s, unsigned lds) {
    const int p0 = s * kStep;
    while (p0 >= bu_end) {
      ++bu;
      bu_end = __builtin_amdgcn_readfirstlane(s_end[bu]);
      bu_first = __builtin_amdgcn_readfirstlane(s_first[bu]);
    }
    if (p0 + kStep <= bu_end) {                      // all rows of the stage in one bucket
      const float *lb = L + (size_t)(bu_first + p0) * M, *rb = R + (size_t)(bu_first + p0) * NC;
#pragma unroll
      for (int q = 0; q < Loop::kL0; ++q) f32_load(lb + loff[q], lds + Loop::dst0(wave, q));
#pragma unroll
      for (int q = 0; q < Loop::kL1; ++q) f32_load(rb + roff[q], lds + Loop::dst1(wave, q));
      return;
    }
    if (bu == nb - 1) {                              // .. and the end of the last one: zeros
      const float *lb = L + (size_t)(bu_first + p0) * M, *rb = R + (size_t)(bu_first + p0) * NC;
      const int left = T - p0;
#pragma unroll
      for (int q = 0; q < Loop::kL0; ++q)
        f32_load(Loop::sub0(wave, q) * FK + Loop::Op0::k(Loop::piece0(wave, q), lane) < left ? lb + loff[q] : (const float*)&kF32Zero,
                 lds + Loop::dst0(wave, q));
#pragma unroll
      for (int q = 0; q < Loop::kL1; ++q)
        f32_load(Loop::sub1(wave, q) * FK + Loop::Op1::k(Loop::piece1(wave, q), lane) < left ? rb + roff[q] : (const float*)&kF32Zero,
                 lds + Loop::dst1(wave, q));
      return;
    }
    // rows of several buckets: a lane's loads each look for theirs among the stage's buckets
    int pl[Loop::kL0], pr[Loop::kL1], fl[Loop::kL0], fr[Loop::kL1];      // row of the contraction; what leads from there to the row of L and R
#pragma unroll
    for (int q = 0; q < Loop::kL0; ++q) {
      pl[q] = p0 + Loop::sub0(wave, q) * FK + Loop::Op0::k(Loop::piece0(wave, q), lane);
      fl[q] = bu_first;
    }
#pragma unroll
    for (int q = 0; q < Loop::kL1; ++q) {
      pr[q] = p0 + Loop::sub1(wave, q) * FK + Loop::Op1::k(Loop::piece1(wave, q), lane);
      fr[q] = bu_first;
    }
    for (int b = bu, end = bu_end; end < p0 + kStep && ++b < nb;) {
      const int first = __builtin_amdgcn_readfirstlane(s_first[b]), next = __builtin_amdgcn_readfirstlane(s_end[b]);
#pragma unroll
      for (int q = 0; q < Loop::kL0; ++q) fl[q] = pl[q] >= end ? first : fl[q];
#pragma unroll
      for (int q = 0; q < Loop::kL1; ++q) fr[q] = pr[q] >= end ? first : fr[q];
      end = next;
    }
#pragma unroll
    for (int q = 0; q < Loop::kL0; ++q) {
      const float* l = L + (size_t)(fl[q] + pl[q]) * M + min(m0 + Loop::Op0::out(Loop::piece0(wave, q), lane), M - 4);
      f32_load(pl[q] < T ? l : (const float*)&kF32Zero, lds + Loop::dst0(wave, q));
    }
#pragma unroll
    for (int q = 0; q < Loop::kL1; ++q) {
      const float* r = R + (size_t)(fr[q] + pr[q]) * NC + min(n0 + Loop::Op1::out(Loop::piece1(wave, q), lane), NC - 4);
      f32_load(pr[q] < T ? r : (const float*)&kF32Zero, lds + Loop::dst1(wave, q));
    }
  };
  F32Acc acc;
  Loop::run((lds_t*)smem, acc, (T + kStep - 1) / kStep, issue);

#pragma unroll
  for (int x = 0; x < 4; ++x) {
    const int i = x >> 1, j = x & 1;
    const int m = m0 + (MT == 2 ? (wave >> 1) * 32 : 0) + i * 16 + (lane & 15);
    const int col = n0 + (wave & 1) * 32 + j * 16 + 4 * (lane >> 4);
    if (m < M && col < NC && (MT == 2 || j == (wave >> 1)))
      *(float4*)(dw + (size_t)e * M * NC + (size_t)m * NC + col) = make_float4(acc[i][j][0], acc[i][j][1], acc[i][j][2], acc[i][j][3]);
  }
}

static unsigned tiles_of(int n, int t) { return (unsigned)((n + t - 1) / t); }

// 32-row blocks of a workgroup's tile: two (64 x 64 tiles) where there are enough tiles for the chip, else one, with the contraction
// over two waves.
// Rows products: two from 280 tiles of 64 x 64 on where the contraction is short (a 32-row tile's first loads and its sum over two
// waves weigh more), from 1200 otherwise; and always one where buckets are so short that 32-row tiles are hardly more.  In us, one and two:
//   K 32, NC 128: 208 tiles 8.8, 9.2;              past the line: 408 12.0, 8.4; 1502 28.4, 18.4
//   K 128, NC 512: 256 9.4, 11.8;                                 408 13.8, 13.0; 1508 38.7, 31.7
//   K 256, NC 1024: 512 18.8, 24.8; 1088 33.9, 34.3;              1508 45.9, 42.7
//   K 1024, NC 1024: 608 61, 82;                                  1504 136, 128
//   short buckets (16 rows, 512 of them, K 256, NC 256)  2048 tiles 41, 60
// Weight gradients: one for fewer than 1024 tiles of 64 x 64 over all experts and from 30 (300 tiles and more: 120) rows per expert on, by
// rows per expert, one over two:  below 120 tiles  8 rows 1.04, 20 0.93, 60 0.83, 200 0.67;  300 - 500  20 1.23, 60 1.05, 130 0.85;
// 800 - 1024  60 1.17, 130 0.99, 300 0.75;  past the line: 1024 - 2000  60 1.31, 300 1.09
static int f32_rows_blocks(const FfnArgs& a, int K, int NC) {
  const long long one = std::max(a.V, a.A / 32 + a.V / 2), two = std::max(a.V, a.A / 64 + a.V / 2);      // row tiles of that many blocks
  return two * tiles_of(NC, FN) >= (K <= 224 ? 280 : 1200) && 10 * one >= 16 * two ? 2 : 1;
}
static int f32_wgrad_blocks(const FfnArgs& a, int M, int NC) {
  const long long tiles = (long long)a.E * tiles_of(M, 64) * tiles_of(NC, FN);
  return tiles >= 1024 || a.A < (tiles < 300 ? 30 : 120) * a.E ? 2 : 1;
}

template <bool WT, int EPI>
static void launch_rows_f32(const FfnArgs& a, const void* in, const void* w, const void* bias, int K, int NC, const void* hpre_in,
                            void* out0, void* out1, hipStream_t s) {
  const int mt = f32_rows_blocks(a, K, NC), cols = (int)tiles_of(NC, FN);
  // row tiles: at most one ragged one per bucket; an eighth of the tiles per XCD, rounded up.  Fewer than 2^32 threads in a launch (of
  // more, HIP runs what is left modulo 2^32, and reports nothing): layers of millions of columns take several.
  const long long row_tiles = a.A / (mt * 32) + a.V;
  const int most = (int)std::max((((1ll << 32) / kF32Threads - 1) / kF32Xcds * kF32Xcds) / row_tiles, 1ll);
  for (int ct0 = 0; ct0 < cols; ct0 += most) {
    const int n = std::min(most, cols - ct0);
    const dim3 grid((unsigned)((row_tiles * n + kF32Xcds - 1) / kF32Xcds * kF32Xcds));
    if (mt == 2)
      hipLaunchKernelGGL((rows_gemm_f32<2, WT, EPI>), grid, dim3(kF32Threads), 0, s, (const float*)in, (const float*)w, (const float*)bias,
                         a.voff, a.owner, a.V, K, NC, ct0, n, a.act, (const float*)hpre_in, (float*)out0, (float*)out1);
    else
      hipLaunchKernelGGL((rows_gemm_f32<1, WT, EPI>), grid, dim3(kF32Threads), 0, s, (const float*)in, (const float*)w, (const float*)bias,
                         a.voff, a.owner, a.V, K, NC, ct0, n, a.act, (const float*)hpre_in, (float*)out0, (float*)out1);
  }
}

static void launch_wgrad_f32(const FfnArgs& a, const void* L, const void* R, int M, int NC, void* dw, hipStream_t s) {
  const int mt = f32_wgrad_blocks(a, M, NC);
  // a grid's second dimension ends at 65535 workgroups: layers of millions of columns take several launches
  const int m_tiles = (int)tiles_of(M, mt * 32), most = 65535;
  for (int m0 = 0; m0 < m_tiles; m0 += most) {
    const dim3 grid(tiles_of(NC, FN), (unsigned)std::min(most, m_tiles - m0), a.E);
    if (mt == 2)
      hipLaunchKernelGGL(wgrad_f32<2>, grid, dim3(kF32Threads), 0, s, (const float*)L, (const float*)R, a.voff, a.owner, a.V, M, NC, m0 * 64, (float*)dw);
    else
      hipLaunchKernelGGL(wgrad_f32<1>, grid, dim3(kF32Threads), 0, s, (const float*)L, (const float*)R, a.voff, a.owner, a.V, M, NC, m0 * 32, (float*)dw);
  }
}

hipError_t launch_ffn_fwd_f32(const FfnArgs& a, const void* xp, const void* w1, const void* b1, const void* w2,
                              const void* b2, void* hpre, void* h_keep, void* yp, void* ws, hipStream_t s) {
  if (a.A == 0) return hipSuccess;
  void* h = h_keep ? h_keep : ws;
  launch_rows_f32<false, EPI_FWD1>(a, xp, w1, b1, a.d, a.f, nullptr, hpre, h, s);
  launch_rows_f32<false, EPI_PLAIN>(a, h, w2, b2, a.f, a.d, nullptr, yp, nullptr, s);
  return hipGetLastError();
}

hipError_t launch_ffn_bwd_f32(const FfnArgs& a, const void* dyp, const void* xp, const void* hpre, const void* h_kept,
                              const void* w1, const void* w2, void* dxp, void* dw1, void* dw2, void* ws, hipStream_t s) {
  float* dhpre = (float*)ws;
  float* h_ws = (float*)((char*)ws + align_up((size_t)a.A * a.f * sizeof(float), 256));
  if (a.A > 0) {
    // dH = dYp . W2^T (W2_e is [f, d]: contraction over its second index), fused with act'
    launch_rows_f32<true, EPI_DH>(a, dyp, w2, nullptr, a.d, a.f, hpre, dhpre, h_kept ? nullptr : h_ws, s);
    // dXp = dHpre . W1^T (W1_e is [d, f])
    launch_rows_f32<true, EPI_PLAIN>(a, dhpre, w1, nullptr, a.f, a.d, nullptr, dxp, nullptr, s);
  }
  const float* h = h_kept ? (const float*)h_kept : h_ws;
  launch_wgrad_f32(a, h, dyp, a.f, a.d, dw2, s);
  launch_wgrad_f32(a, xp, dhpre, a.d, a.f, dw1, s);
  return hipGetLastError();
}

}  // namespace flexmoe
