// fp32 expert FFN (paper Eq. 2) forward and backward per vExpert bucket, on the fp32 matrix instruction
// v_mfma_f32_32x32x2_f32 (fp32 operands, products and sums).
//
// One workgroup of four waves per 64 x 64 outputs, a wave per 32 x 32.  32-wide K tiles travel global -> LDS with direct
// loads through four stages (64 KB: two workgroups per compute unit); three tiles are in flight while one is multiplied.
// The contraction index inside a K tile is dealt to the instruction's two halves four at a time, so that a
// K-contiguous operand is read from LDS as 16-byte vectors.  Every sum runs over its K tiles in ascending order in one
// accumulator: results are reproducible.
//
// What bounds it: a workgroup's K tile is 1024 cycles of matrix instructions per wave against 16 KB of operands; with
// 100 - 600 workgroups (the sizes fp32 layers are used at) the K tiles' latency.  One thread per output, reading its
// operands with scalar loads, took 255 us for [2000, 256] x [256, 1024] and 1680 us where the weights are read along their
// rows (dH, dXp: every lane in a cache line of its own); these take 31 us each (34 TFLOP/s of 157), the weight gradients
// of that layer 26 us instead of 317, and the whole fp32 training step 237 us instead of 4920.
#include "common.h"

namespace flexmoe {

constexpr int kF32Threads = 256;
constexpr int FM = 64, FN = 64, FK = 32;             // tile of outputs, K tile
constexpr int kF32Stages = 4;
constexpr int kF32OpBytes = 64 * FK * 4;             // one operand's K tile: 8 KB
constexpr int kF32StageBytes = 2 * kF32OpBytes;
constexpr int kF32Loads = 4;                         // direct loads per wave and K tile: two per operand

enum { EPI_FWD1 = 0, EPI_PLAIN = 1, EPI_DH = 2 };

typedef __attribute__((address_space(3))) unsigned char lds_t;
__device__ const float4 kF32Zero = {0.f, 0.f, 0.f, 0.f};

__device__ __forceinline__ void f32_load(const float* p, unsigned lds) {
  asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" ::"v"(p), "s"(lds) : "memory");
}
template <int N> __device__ __forceinline__ void f32_wait_vmcnt() { __builtin_amdgcn_s_waitcnt(0x0F70 | (N & 15) | ((N >> 4) << 14)); }
__device__ __forceinline__ void f32_wait_tiles(int tiles) {      // at most `tiles` younger K tiles in flight
  switch (tiles) {
    case 0: f32_wait_vmcnt<0>(); break;
    case 1: f32_wait_vmcnt<kF32Loads>(); break;
    default: f32_wait_vmcnt<2 * kF32Loads>(); break;
  }
}

// LDS tile of a K-contiguous operand: [64][32 k], rows of eight 16-byte chunks, chunk index XOR row & 7 (conflict-free
// 16-byte reads of 32 rows).  Direct load q of wave w fills rows 8 (2 w + q) ..: the lane's row and first k:
__device__ __forceinline__ int kc_row(int wave, int q, int lane) { return (wave * 2 + q) * 8 + (lane >> 3); }
__device__ __forceinline__ int kc_k(int lane) { return ((lane & 7) ^ (lane >> 3)) * 4; }
// LDS tile of a K-strided operand: [32 k][64], rows of sixteen chunks, chunk index XOR 8 where k & 4 (the
// instruction's halves read rows four apart: 32 banks apart).  The lane's k row and first column:
__device__ __forceinline__ int ks_k(int wave, int q, int lane) { return (wave * 2 + q) * 4 + (lane >> 4); }
__device__ __forceinline__ int ks_col(int k, int lane) { return ((lane & 15) ^ ((k & 4) << 1)) * 4; }

// Four k of one operand's 32 outputs (lane % 32 + base): k = 8 kk + 4 (lane / 32) ..
template <bool KC> __device__ __forceinline__ void f32_frag(float (&f)[4], const lds_t* tile, int base, int kk, int lane) {
  const int r = base + (lane & 31), h = lane >> 5;
  if (KC) {
    const f32x4 v = *(const __attribute__((address_space(3))) f32x4*)(tile + r * 128 + (((2 * kk + h) ^ (r & 7)) << 4));
#pragma unroll
    for (int j = 0; j < 4; ++j) f[j] = v[j];
  } else {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int k = 8 * kk + 4 * h + j;
      f[j] = *(const __attribute__((address_space(3))) float*)(tile + k * 256 + (((r >> 2) ^ (h << 3)) << 4) + (r & 3) * 4);
    }
  }
}

// KT K tiles through the stages; issue(kt, lds address of the stage) starts the wave's kF32Loads loads of one.
// First operand = output rows, second = columns; acc[q]: row lane % 32, column 8 (q / 4) + 4 (lane / 32) + q % 4 of the wave's block.
template <bool KC0, bool KC1, typename Issue>
__device__ __forceinline__ void f32_mainloop(lds_t* sm, f32x16& acc, int KT, Issue issue) {
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const unsigned lds0 = __builtin_amdgcn_readfirstlane((unsigned)(uintptr_t)sm);
#pragma unroll
  for (int s = 0; s < kF32Stages - 1; ++s)
    if (s < KT) issue(s, lds0 + s * kF32StageBytes);
  for (int kt = 0; kt < KT; ++kt) {
    f32_wait_tiles(min(kF32Stages - 2, KT - 1 - kt));
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
    if (kt + kF32Stages - 1 < KT) issue(kt + kF32Stages - 1, lds0 + (kt + kF32Stages - 1) % kF32Stages * kF32StageBytes);
    const lds_t* st = sm + kt % kF32Stages * kF32StageBytes;
#pragma unroll
    for (int kk = 0; kk < FK / 8; ++kk) {
      float a[4], b[4];
      f32_frag<KC0>(a, st, (wave >> 1) * 32, kk, lane);
      f32_frag<KC1>(b, st + kF32OpBytes, (wave & 1) * 32, kk, lane);
#pragma unroll
      for (int j = 0; j < 4; ++j) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(b[j], a[j], acc, 0, 0, 0);
    }
  }
}

// flat row-tile index -> {first row, rows, expert} of a 64-row tile of the bucket list; one wave scans the buckets'
// tile counts.  False (for the whole workgroup): beyond the last tile.
__device__ __forceinline__ bool f32_row_tile(const int32_t* __restrict__ voff, const int32_t* __restrict__ owner, int V, int rt,
                                             int* s_tile, int* row0, int* rows, int* e) {
  if (threadIdx.x < kWave) {
    const int lane = threadIdx.x;
    if (lane == 0) s_tile[0] = -1;
    const int per = (V + kWave - 1) / kWave;
    int sum = 0;
    for (int q = 0; q < per; ++q) {
      const int v = lane * per + q;
      if (v < V) sum += (voff[v + 1] - voff[v] + FM - 1) / FM;
    }
    int incl = sum;
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
      const int up = __shfl_up(incl, o);
      if (lane >= o) incl += up;
    }
    int start = incl - sum;
    if (rt >= start && rt < incl)
      for (int q = 0; q < per; ++q) {
        const int v = lane * per + q;
        if (v >= V) break;
        const int lo = voff[v], n = (voff[v + 1] - lo + FM - 1) / FM;
        if (rt < start + n) {
          s_tile[0] = lo + (rt - start) * FM;
          s_tile[1] = min(FM, voff[v + 1] - s_tile[0]);
          s_tile[2] = owner[v];
          break;
        }
        start += n;
      }
  }
  __syncthreads();
  *row0 = __builtin_amdgcn_readfirstlane(s_tile[0]);
  *rows = __builtin_amdgcn_readfirstlane(s_tile[1]);
  *e = __builtin_amdgcn_readfirstlane(s_tile[2]);
  return *row0 >= 0;
}

// C[p, n] = sum_k In[p, k] * W_e[k, n]   (WT == false, W_e is [K, NC])
//         = sum_k In[p, k] * W_e[n, k]   (WT == true,  W_e is [NC, K])
template <bool WT, int EPI>
__global__ __launch_bounds__(kF32Threads, 2) void rows_gemm_f32(const float* __restrict__ in, const float* __restrict__ w,
                                                                const float* __restrict__ bias,
                                                                const int32_t* __restrict__ voff,
                                                                const int32_t* __restrict__ owner, int V, int K, int NC,
                                                                int act, const float* __restrict__ hpre_in,
                                                                float* __restrict__ out0, float* __restrict__ out1) {
  __shared__ __align__(1024) unsigned char smem[kF32Stages * kF32StageBytes];
  __shared__ int s_tile[3];
  int row0, rows, e;
  if (!f32_row_tile(voff, owner, V, blockIdx.x, s_tile, &row0, &rows, &e)) return;
  const int n0 = blockIdx.y * FN, cols = min(FN, NC - n0);
  const float* we = w + (size_t)e * K * NC;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;

  const float* ap[2];
  const float* wp[2];
  int wk[2];
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    ap[q] = in + (size_t)(row0 + min(kc_row(wave, q, lane), rows - 1)) * K + kc_k(lane);
    if (WT) {
      wk[q] = kc_k(lane);
      wp[q] = we + (size_t)(n0 + min(kc_row(wave, q, lane), cols - 1)) * K + wk[q];
    } else {
      wk[q] = ks_k(wave, q, lane);
      wp[q] = we + (size_t)wk[q] * NC + n0 + min(ks_col(wk[q], lane), cols - 4);
    }
  }
  auto issue = [&](int kt, unsigned lds) {
    const int k0 = kt * FK;
#pragma unroll
    for (int q = 0; q < 2; ++q) f32_load(k0 + kc_k(lane) < K ? ap[q] + k0 : (const float*)&kF32Zero, lds + (wave * 2 + q) * 1024);
#pragma unroll
    for (int q = 0; q < 2; ++q)
      f32_load(k0 + wk[q] < K ? wp[q] + (WT ? (size_t)k0 : (size_t)k0 * NC) : (const float*)&kF32Zero,
               lds + kF32OpBytes + (wave * 2 + q) * 1024);
  };
  f32x16 acc;
#pragma unroll
  for (int q = 0; q < 16; ++q) acc[q] = 0.f;
  f32_mainloop<true, WT>((lds_t*)smem, acc, (K + FK - 1) / FK, issue);

  const int row = (wave >> 1) * 32 + (lane & 31);
  if (row >= rows) return;
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    const int col = n0 + (wave & 1) * 32 + 8 * g + 4 * (lane >> 5);
    if (col >= NC) continue;
    const size_t o = (size_t)(row0 + row) * NC + col;
    float c[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) c[q] = acc[4 * g + q];
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
      const float4 z = *(const float4*)(hpre_in + o);
      *(float4*)(out0 + o) = make_float4(c[0] * act_deriv(z.x, act), c[1] * act_deriv(z.y, act), c[2] * act_deriv(z.z, act),
                                         c[3] * act_deriv(z.w, act));
      if (out1) *(float4*)(out1 + o) = make_float4(act_apply(z.x, act), act_apply(z.y, act), act_apply(z.z, act), act_apply(z.w, act));
    }
  }
}

// dW_e[m, n] = sum over the vExperts v of e (ascending v), rows p of v: L[p, m] * R[p, n].  The rows of all of the
// expert's buckets are one contraction: K tile kt holds rows 32 kt .. of the buckets laid behind each other.
__global__ __launch_bounds__(kF32Threads, 2) void wgrad_f32(const float* __restrict__ L, const float* __restrict__ R,
                                                            const int32_t* __restrict__ voff,
                                                            const int32_t* __restrict__ owner, int V, int M, int NC,
                                                            float* __restrict__ dw) {
  __shared__ __align__(1024) unsigned char smem[kF32Stages * kF32StageBytes];
  __shared__ int s_first[FLEXMOE_MAX_VEXPERTS], s_end[FLEXMOE_MAX_VEXPERTS];      // first row - rows before it, rows up to its end
  __shared__ int s_n;
  const int e = blockIdx.z;
  const int m0 = blockIdx.y * FM, n0 = blockIdx.x * FN;
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

  // the wave's loads of a K tile: k rows ks_k(wave, 0) and ks_k(wave, 1); a lane's k rows only grow, so its bucket does too
  int b[2] = {0, 0};
  auto issue = [&](int kt, unsigned lds) {
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const int k = ks_k(wave, q, lane), p = kt * FK + k;
      const float* l = (const float*)&kF32Zero;
      const float* r = l;
      if (p < T) {
        while (p >= s_end[b[q]]) ++b[q];
        const size_t row = (size_t)(s_first[b[q]] + p);
        l = L + row * M + min(m0 + ks_col(k, lane), M - 4);
        r = R + row * NC + min(n0 + ks_col(k, lane), NC - 4);
      }
      f32_load(l, lds + (wave * 2 + q) * 1024);
      f32_load(r, lds + kF32OpBytes + (wave * 2 + q) * 1024);
    }
  };
  f32x16 acc;
#pragma unroll
  for (int q = 0; q < 16; ++q) acc[q] = 0.f;
  f32_mainloop<false, false>((lds_t*)smem, acc, (T + FK - 1) / FK, issue);

  const int m = m0 + (wave >> 1) * 32 + (lane & 31);
  if (m >= M) return;
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    const int col = n0 + (wave & 1) * 32 + 8 * g + 4 * (lane >> 5);
    if (col < NC)
      *(float4*)(dw + (size_t)e * M * NC + (size_t)m * NC + col) = make_float4(acc[4 * g], acc[4 * g + 1], acc[4 * g + 2], acc[4 * g + 3]);
  }
}

static unsigned tiles_of(int n, int t) { return (unsigned)((n + t - 1) / t); }

template <bool WT, int EPI>
static void launch_rows_f32(const FfnArgs& a, const void* in, const void* w, const void* bias, int K, int NC, const void* hpre_in,
                            void* out0, void* out1, hipStream_t s) {
  const dim3 grid((unsigned)(a.A / FM + a.V), tiles_of(NC, FN));      // row tiles: at most one ragged one per bucket
  hipLaunchKernelGGL((rows_gemm_f32<WT, EPI>), grid, dim3(kF32Threads), 0, s, (const float*)in, (const float*)w,
                     (const float*)bias, a.voff, a.owner, a.V, K, NC, a.act, (const float*)hpre_in, (float*)out0, (float*)out1);
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
  hipLaunchKernelGGL(wgrad_f32, dim3(tiles_of(a.d, FN), tiles_of(a.f, FM), a.E), dim3(kF32Threads), 0, s, h, (const float*)dyp,
                     a.voff, a.owner, a.V, a.f, a.d, (float*)dw2);
  hipLaunchKernelGGL(wgrad_f32, dim3(tiles_of(a.f, FN), tiles_of(a.d, FM), a.E), dim3(kF32Threads), 0, s, (const float*)xp,
                     (const float*)dhpre, a.voff, a.owner, a.V, a.d, a.f, (float*)dw1);
  return hipGetLastError();
}

}  // namespace flexmoe
