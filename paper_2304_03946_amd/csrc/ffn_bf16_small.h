// Rows GEMMs for buckets that do not fill 256-row tiles: decode steps, short prompts, small training batches, many
// small experts.  Part of the bf16 expert-FFN kernels; included by ffn_bf16.hip only (one translation unit).
#pragma once
#include "common.h"
#include "ffn_bf16_tile.h"
#include "ffn_bf16_dma.h"
#include "ffn_bf16_persist.h"
namespace flexmoe {
// =============================================================================================
// rows_gemm_small: with a few rows per expert the product is a pass over the weights, bound by HBM.  So
//  * a row tile holds BM = 32 or 64 rows of one EXPERT, not of one bucket: the plan lists the rows of all of an
//    expert's vExperts behind each other (rowmap), so that replicas do not read the expert's weights again;
//  * a workgroup of four waves owns BM x 128 outputs; 64-wide K tiles travel HBM -> LDS with direct loads that
//    fetch whole 128-byte lines of either operand (a K-strided operand: 256-byte pieces of 64 rows), S stages of
//    them, two workgroups per compute unit (measured for the loads alone: 5.6 - 6.2 TB/s of 8);
//  * where there are fewer tiles than workgroups the contraction is cut into segments; the last workgroup
//    to finish a tile adds the fp32 partial tiles in segment order (a fixed order: the same call gives the same bits) and
//    runs the epilogue, so there is no second launch.  How many segments there are follows from the row tiles in use
//    (small_segments), so the last bits of a row can depend on how many experts the other rows of the batch went to;
//  * where K is a multiple of 128, products are summed by the same instruction in the same order as in the 256 x 256
//    kernels: a row without segments here and outside a split last round there has the same bits in either.
// K and NC are any multiples of 8: the last, partial K tile reads zeros past K.
// =============================================================================================
constexpr int SN = 128, SK = 64;                         // columns of a tile, contraction indices of a stage
constexpr int kSmallWaves = 4;
constexpr int kSmallThreads = kSmallWaves * kWave;
constexpr int kSmallWBytes = SN * SK * 2;
constexpr int kSmallSplitMax = 16;                       // segments of a contraction
constexpr int kSmallSplitTarget = 512;                   // workgroups a launch wants: two per compute unit
constexpr int kSmallSplitKTiles = 4;                     // a segment is at least this many K tiles
constexpr int kSmallSlots = kSmallSplitTarget;           // tiles x segments where there are segments (small_segments)
template <int BM> struct SmallCfg {
  static constexpr int kABytes = BM * SK * 2;
  static constexpr int kStage = kABytes + kSmallWBytes;
  static constexpr int S = 81920 / kStage;               // stages: half of a compute unit's LDS
  static constexpr int kLds = S * kStage;
  static constexpr int kALoads = BM / 8 / kSmallWaves;   // direct loads per wave and stage: rows operand ...
  static constexpr int kWLoads = kSmallWBytes / 1024 / kSmallWaves;      // ... and weights
  static constexpr int kLoads = kALoads + kWLoads;
  static_assert(BM % 32 == 0 && S >= 3 && (S - 2) * kLoads < 64, "the wait count has six bits");
};

__device__ const uint4 kSmallZero[8] = {};

struct SmallArgs {
  const bf16_t* in;
  const bf16_t* w;
  const bf16_t* bias;
  const i32x4* tab;              // tab[0][0] row tiles; tab[1 + t] = {first position in rowmap, rows, expert, 0}
  const int32_t* rowmap;         // position in expert order -> bucket row
  int K, NC, col_tiles;
  const bf16_t* hpre_in;
  bf16_t* out0;
  bf16_t* out1;
  const int32_t* gsrc;           // gathered rows of `in`: row gsrc[bucket row] / gk; or null
  int gk;
  const int32_t* scatter_rows;   // bucket row p is stored as row scatter_rows[p] of out0; or null
  int act, lut;                  // activation (EVAL); which of g_act_lut's tables it is read from, -1: ReLU
  float* partial;                // kSmallSlots partial tiles
  int* counters;                 // one per tile that is cut into segments, zeroed by the plan
};

// Segments of a product with `tiles` output tiles and k_tiles K tiles.
__host__ __device__ inline int small_segments(int tiles, int k_tiles) {
  int s = 1;
  while (s < kSmallSplitMax && tiles * s * 2 <= kSmallSplitTarget && k_tiles >= 2 * s * kSmallSplitKTiles) s *= 2;
  return s;
}

// ---- plan: expert-major row list and row tiles ----------------------------------------------
// Every workgroup derives the prefixes.  The first writes the experts' first row tiles, a thread per expert, and all of them
// together the further ones; the others write the row list, bucket by bucket (an expert's buckets in ascending vExpert id),
// plan.parts waves to a bucket.  (With one wave per bucket and one thread per expert the plan was the longest launch where
// few experts have many rows: whole forward passes, d = f = 8, 1.6 million rows of 4 experts 485 -> 319 us; d 64, f 128, 112000 rows
// 121 -> 101; d 128, f 512, 22400 rows 64 -> 61.)
struct SmallPlan {
  i32x4* tab;
  int32_t* rowmap;
  int* counters;
  int bm;                        // 0: the product does not use these kernels
  int parts;                     // waves that write a bucket's rows
};
__device__ __forceinline__ void small_plan_block(const int32_t* __restrict__ voff, const int32_t* __restrict__ owner, int E, int V,
                                                 const SmallPlan& plan, int block, int nblocks) {
  const int bm = plan.bm;
  __shared__ int rows_e[FLEXMOE_MAX_EXPERTS], start_e[FLEXMOE_MAX_EXPERTS], tile_e[FLEXMOE_MAX_EXPERTS], wsum[2][kGemmThreads / kWave];
  __shared__ int2 bucket[FLEXMOE_MAX_VEXPERTS];          // {expert, rows}
  __shared__ int pos0[FLEXMOE_MAX_VEXPERTS], off[FLEXMOE_MAX_VEXPERTS];
  static_assert(kGemmThreads == FLEXMOE_MAX_EXPERTS && 2 * kGemmThreads == FLEXMOE_MAX_VEXPERTS, "a thread per expert, two buckets per thread");
  const int t = threadIdx.x, lane = t & (kWave - 1), wave = t / kWave;
  int own[2], cnt[2];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int v = t + h * kGemmThreads;
    own[h] = -1;
    cnt[h] = 0;
    if (v < V) {
      own[h] = owner[v];
      off[v] = voff[v];
      cnt[h] = voff[v + 1] - off[v];
    }
    bucket[v] = make_int2(own[h], cnt[h]);
  }
  rows_e[t] = 0;
  __syncthreads();
#pragma unroll
  for (int h = 0; h < 2; ++h)
    if (own[h] >= 0) atomicAdd(&rows_e[own[h]], cnt[h]);      // integer sums: order does not matter
  __syncthreads();
  // exclusive prefixes over the experts: rows, row tiles
  const int r = t < E ? rows_e[t] : 0, n = (r + bm - 1) / bm;
  int ir = r, in = n;
#pragma unroll
  for (int o = 1; o < kWave; o <<= 1) {
    const int ur = __shfl_up(ir, o), un = __shfl_up(in, o);
    if (lane >= o) {
      ir += ur;
      in += un;
    }
  }
  if (lane == kWave - 1) {
    wsum[0][wave] = ir;
    wsum[1][wave] = in;
  }
  __syncthreads();
  int row0 = ir - r, tile0 = in - n;
  for (int w = 0; w < wave; ++w) {
    row0 += wsum[0][w];
    tile0 += wsum[1][w];
  }
  constexpr int kFirst = 16;                             // row tiles of an expert that its thread writes
  if (block == 0) {
    for (int i = 0; i < min(n, kFirst); ++i) plan.tab[1 + tile0 + i] = i32x4{row0 + i * bm, min(bm, r - i * bm), t, 0};
    if (t == kGemmThreads - 1) plan.tab[0] = i32x4{tile0 + n, 0, 0, 0};
    for (int i = t; i < kSmallSlots; i += kGemmThreads) plan.counters[i] = 0;
  }
  start_e[t] = row0;
  tile_e[t] = tile0;
  if (__syncthreads_or(n > kFirst)) {
    const int total = tile_e[kGemmThreads - 1] + (rows_e[kGemmThreads - 1] + bm - 1) / bm;
    for (int rt = block * kGemmThreads + t; rt < total; rt += nblocks * kGemmThreads) {
      int e = 0;                                         // the last expert with tile_e <= rt (one without tiles shares its successor's value)
#pragma unroll
      for (int step = kGemmThreads / 2; step; step >>= 1)
        if (tile_e[e + step] <= rt) e += step;
      const int i = rt - tile_e[e];
      if (i >= kFirst) plan.tab[1 + rt] = i32x4{start_e[e] + i * bm, min(bm, rows_e[e] - i * bm), e, 0};
    }
  }
  if (block == 0) return;
  {
    int before[2] = {0, 0};      // rows of the same expert in earlier buckets
#pragma unroll 8
    for (int u = 0; u < V; ++u) {
      const int2 b = bucket[u];
#pragma unroll
      for (int h = 0; h < 2; ++h)
        if (b.x == own[h] && u < t + h * kGemmThreads) before[h] += b.y;
    }
#pragma unroll
    for (int h = 0; h < 2; ++h)
      if (own[h] >= 0) pos0[t + h * kGemmThreads] = start_e[own[h]] + before[h];
  }
  __syncthreads();
  constexpr int kWaves = kGemmThreads / kWave;
  for (int w = (block - 1) * kWaves + wave; w < V * plan.parts; w += (nblocks - 1) * kWaves) {
    const int v = w / plan.parts, lo = off[v], len = bucket[v].y, to = pos0[v];
    for (int i = w % plan.parts * kWave + lane; i < len; i += plan.parts * kWave) plan.rowmap[to + i] = lo + i;
  }
}
__global__ __launch_bounds__(kGemmThreads) void small_plan_kernel(const int32_t* __restrict__ voff,
                                                                  const int32_t* __restrict__ owner, int E, int V, SmallPlan plan) {
  small_plan_block(voff, owner, E, V, plan, blockIdx.x, gridDim.x);
}

// ---- loads of one stage ---------------------------------------------------------------------
__device__ __forceinline__ void small_load(const bf16_t* base, uint32_t off, unsigned lds) {
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(off), "s"(base), "s"(lds) : "memory");
}
__device__ __forceinline__ void small_load_at(const bf16_t* p, unsigned lds) {
  asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" ::"v"(p), "s"(lds) : "memory");
}
// Activation and derivative without a table.
template <bool EVAL> __device__ __forceinline__ void small_act(int act, float z, float* a, float* da) {
  if (!EVAL) act_both<FLEXMOE_RELU>(z, a, da);
  else if (act == FLEXMOE_GELU_ERF) act_both<FLEXMOE_GELU_ERF>(z, a, da);
  else act_both<FLEXMOE_GELU_TANH>(z, a, da);
}
template <int L> __device__ __forceinline__ void small_wait(int tiles) {
  switch (tiles) {
    case 0: wait_vmcnt<0>(); break;
    case 1: wait_vmcnt<L>(); break;
    default: wait_vmcnt<2 * L>(); break;
  }
}

// EPI as in rows_epilogue_t.  WT: W_e is [NC, K] (else [K, NC]).  EVAL: GELU is evaluated, not read from a table (kernels of their
// own: with both in one, the 1500-token step of d 1024 took 658 us instead of 650).
// `block` of `blocks` that walk the product's tiles; smem: SmallCfg<BM>::kLds bytes.
template <int BM, bool WT, int EPI, bool EVAL>
__device__ __forceinline__ void rows_small_block(const SmallArgs& p, unsigned char* smem, unsigned block, unsigned blocks) {
  typedef SmallCfg<BM> C;
  constexpr int S = C::S, RB = BM / 16, NB2 = SN / kSmallWaves / 16;      // 16-row and 16-column blocks of a wave
  lds_byte_t* const sm = (lds_byte_t*)smem;
  const unsigned lds0 = __builtin_amdgcn_readfirstlane((unsigned)(uintptr_t)sm);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  const int fr = lane & 15, fg = lane >> 4;              // fragment row (or column), group of eight k
  const RowTabPtr tab = (RowTabPtr)p.tab;
  const int K = p.K, NC = p.NC;
  const int rows_act = tab[0][0];
  const int k_tiles = (K + SK - 1) / SK;
  const int tiles = rows_act * p.col_tiles;
  const int nseg = small_segments(tiles, k_tiles);
  // without segments: the XCD-aware patch order; with them: tile-major, a tile's segments side by side
  const unsigned total = nseg > 1 ? (unsigned)(tiles * nseg) : patched_grid(rows_act, p.col_tiles);

  // lane parts of the LDS fragment addresses
  uint32_t la, lw;
  la = fr * 128 + ((fg ^ (fr & 7)) << 4);                // second half of a stage: chunk index XOR 4
  if (WT) {
    lw = C::kABytes + wave * (NB2 * 2048) + la;
  } else {
    const int k = 8 * fg + (fr >> 2);
    const int x = ((fr >> 2) << 2) ^ ((fg & 1) << 1);
    lw = C::kABytes + k * 256 + (((wave * (NB2 * 2) + ((fr & 3) >> 1)) ^ x) << 4) + 8 * (fr & 1);
  }

  for (unsigned idx = block; idx < total; idx += blocks) {
    int rt, ct, seg = 0;
    if (nseg > 1) {
      seg = (int)(idx % nseg);
      const int tile = (int)(idx / nseg);
      rt = tile / p.col_tiles;
      ct = tile % p.col_tiles;
    } else if (!patched_tile(idx, rows_act, p.col_tiles, &rt, &ct)) {
      continue;
    }
    const i32x4 d = tab[1 + rt];
    const int first = d[0], rows = d[1], e = d[2];
    const int n0 = ct * SN, cols = min(SN, NC - n0);
    const int kt0 = (int)((long long)k_tiles * seg / nseg), kt1 = (int)((long long)k_tiles * (seg + 1) / nseg);
    const bf16_t* w_e = p.w + (size_t)e * K * NC + (WT ? (size_t)n0 * K : (size_t)n0);

    // bucket rows of the wave's loads (rows past the tile repeat its last row) and of its outputs
    uint32_t aoff[C::kALoads];
    int akc;                                             // the lane's chunk of a row, in elements
    {
      const int lr = lane >> 3;
      akc = ((lane & 7) ^ lr) * 8;
#pragma unroll
      for (int q = 0; q < C::kALoads; ++q) {
        int r = p.rowmap[first + min((wave * C::kALoads + q) * 8 + lr, rows - 1)];
        if (p.gsrc) r = p.gsrc[r] / p.gk;
        aoff[q] = ((uint32_t)r * (uint32_t)K + akc) * 2;
      }
    }
    int orow[RB];
#pragma unroll
    for (int b = 0; b < RB; ++b) orow[b] = p.rowmap[first + min(b * 16 + fr, rows - 1)];
    uint32_t woff[C::kWLoads];
    int wk[C::kWLoads];                                  // k (in the stage) of the lane's first element
#pragma unroll
    for (int q = 0; q < C::kWLoads; ++q) {
      const int i = wave * C::kWLoads + q;
      if (WT) {
        const int row = i * 8 + (lane >> 3);
        wk[q] = ((lane & 7) ^ (row & 7)) * 8;
        woff[q] = (uint32_t)(min(row, cols - 1) * K + wk[q]) * 2;
      } else {
        const int kr = i * 4 + (lane >> 4);
        wk[q] = kr;
        const int c = min((lane & 15) ^ ((kr & 3) << 2) ^ ((kr & 8) >> 2), cols / 8 - 1);
        woff[q] = (uint32_t)(kr * NC + c * 8) * 2;
      }
    }
    auto issue = [&](int kt) {
      const unsigned st = lds0 + (unsigned)((kt - kt0) % S) * C::kStage;
      const int k0 = kt * SK;
      const bf16_t* wb = w_e + (WT ? (size_t)k0 : (size_t)k0 * NC);
      if (k0 + SK <= K) {
#pragma unroll
        for (int q = 0; q < C::kALoads; ++q) small_load(p.in + k0, aoff[q], st + (wave * C::kALoads + q) * 1024);
#pragma unroll
        for (int q = 0; q < C::kWLoads; ++q) small_load(wb, woff[q], st + C::kABytes + (wave * C::kWLoads + q) * 1024);
      } else {                                           // past K: zeros on both sides
        const bf16_t* z = (const bf16_t*)kSmallZero + (lane & 7) * 8;
#pragma unroll
        for (int q = 0; q < C::kALoads; ++q)
          small_load_at(k0 + akc < K ? (const bf16_t*)((const char*)(p.in + k0) + aoff[q]) : z, st + (wave * C::kALoads + q) * 1024);
#pragma unroll
        for (int q = 0; q < C::kWLoads; ++q)
          small_load_at(k0 + wk[q] < K ? (const bf16_t*)((const char*)wb + woff[q]) : z,
                        st + C::kABytes + (wave * C::kWLoads + q) * 1024);
      }
    };

    f32x4 acc[RB][NB2];
#pragma unroll
    for (int i = 0; i < RB; ++i)
#pragma unroll
      for (int j = 0; j < NB2; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

    __syncthreads();                                     // the previous tile's epilogue has left the stages
#pragma unroll
    for (int q = 0; q < S - 1; ++q)
      if (kt0 + q < kt1) issue(kt0 + q);
    for (int kt = kt0; kt < kt1; ++kt) {
      small_wait<C::kLoads>(min(S - 2, kt1 - 1 - kt));
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
      __builtin_amdgcn_s_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
      if (kt + S - 1 < kt1) issue(kt + S - 1);           // into the stage every wave has just left
      const lds_byte_t* st = sm + ((kt - kt0) % S) * C::kStage;
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) {
        bf16x8 a[RB], w[NB2];
#pragma unroll
        for (int j = 0; j < NB2; ++j) {
          if (WT) {
            w[j] = *(const __attribute__((address_space(3))) bf16x8*)(st + (lw ^ (ks << 6)) + j * 2048);
          } else {
            const lds_byte_t* at = st + (lw ^ (uint32_t)(j << 5)) + ks * (32 * 256);
            const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)at);
            const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(at + 4 * 256));
            typedef short s16x8 __attribute__((ext_vector_type(8)));
            w[j] = __builtin_bit_cast(bf16x8, (s16x8)__builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
          }
        }
#pragma unroll
        for (int i = 0; i < RB; ++i) a[i] = *(const __attribute__((address_space(3))) bf16x8*)(st + (la ^ (ks << 6)) + i * 2048);
#pragma unroll
        for (int i = 0; i < RB; ++i)
#pragma unroll
          for (int j = 0; j < NB2; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[j], a[i], acc[i][j], 0, 0, 0);
      }
    }
    __syncthreads();                                     // every wave has left the last stage

    if (nseg > 1) {
      // Partial tiles cross XCDs: stores and loads at agent scope go past the L2s; every wave waits for its stores before the
      // counter is advanced, and the last workgroup's loads stay behind one thread's acquire.  (Decode step of 16 tokens 76 us; with an
      // acquire in every wave 82, with an add that also releases, i.e. writes the L2 back for every segment, 94.)
      const int tile = rt * p.col_tiles + ct;
      typedef unsigned long long u64;
      u64* part = (u64*)(p.partial + (size_t)tile * nseg * (BM * SN));
#pragma unroll
      for (int i = 0; i < RB; ++i)
#pragma unroll
        for (int j = 0; j < NB2; ++j) {
          u64* dst = part + (size_t)seg * (BM * SN / 2) + (i * NB2 + j) * (2 * kSmallThreads) + threadIdx.x;
          const u64 lo = (u64)__float_as_uint(acc[i][j][0]) | (u64)__float_as_uint(acc[i][j][1]) << 32;
          const u64 hi = (u64)__float_as_uint(acc[i][j][2]) | (u64)__float_as_uint(acc[i][j][3]) << 32;
          __hip_atomic_store(dst, lo, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          __hip_atomic_store(dst + kSmallThreads, hi, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
      __builtin_amdgcn_s_waitcnt(0x0F70);                // vmcnt(0): the stores have arrived
      __syncthreads();
      if (threadIdx.x == 0) {
        const int before = __hip_atomic_fetch_add(&p.counters[tile], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (before == nseg - 1) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
        *(volatile __attribute__((address_space(3))) int*)sm = before;
      }
      __syncthreads();
      const bool last = __builtin_amdgcn_readfirstlane(*(volatile __attribute__((address_space(3))) int*)sm) == nseg - 1;
      if (!last) continue;
      if (threadIdx.x == 0) p.counters[tile] = 0;        // as the plan left it: the call's next product counts there too
#pragma unroll
      for (int i = 0; i < RB; ++i)
#pragma unroll
        for (int j = 0; j < NB2; ++j) {
          f32x4 s = f32x4{0.f, 0.f, 0.f, 0.f};
          for (int g = 0; g < nseg; ++g) {
            u64* from = part + (size_t)g * (BM * SN / 2) + (i * NB2 + j) * (2 * kSmallThreads) + threadIdx.x;
            const u64 lo = __hip_atomic_load(from, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            const u64 hi = __hip_atomic_load(from + kSmallThreads, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            s[0] += __uint_as_float((uint32_t)lo);
            s[1] += __uint_as_float((uint32_t)(lo >> 32));
            s[2] += __uint_as_float((uint32_t)hi);
            s[3] += __uint_as_float((uint32_t)(hi >> 32));
          }
          acc[i][j] = s;
        }
      __syncthreads();                                   // the flag has been read
    }

    const bool use_lut = EPI != EPI_PLAIN && !EVAL && p.lut >= 0;
    if (use_lut) {
      // the stages are free: the activation table (14 KB, EPI_DH 28, from L2) goes there
      const unsigned char* g = lut_source<EPI>(p.lut) + lane * 16;
      for (int i = wave; i < lut_lds_bytes<EPI>() / 1024; i += kSmallWaves) small_load_at((const bf16_t*)(g + i * 1024), lds0 + i * 1024);
      __builtin_amdgcn_s_waitcnt(0x0F70);
      __syncthreads();
    }
#pragma unroll
    for (int i = 0; i < RB; ++i) {
      if (i * 16 + fr < rows) {
        const size_t row = p.scatter_rows ? (size_t)p.scatter_rows[orow[i]] : (size_t)orow[i];
#pragma unroll
        for (int j = 0; j < NB2; ++j) {
          const int col = n0 + wave * (NB2 * 16) + j * 16 + fg * 4;
          if (col < NC) {
            f32x4 c = acc[i][j];
            if (EPI == EPI_FWD1 || EPI == EPI_PLAIN) {
              if (p.bias) {
                float b[4];
                unpack4(*(const uint2*)(p.bias + (size_t)e * NC + col), b);
#pragma unroll
                for (int q = 0; q < 4; ++q) c[q] += b[q];
              }
            }
            const size_t o = row * NC + col;
            if (EPI == EPI_PLAIN) {
              *(uint2*)(p.out0 + o) = pack4(c[0], c[1], c[2], c[3]);
            } else if (EPI == EPI_FWD1) {
              const uint2 pre = pack4(c[0], c[1], c[2], c[3]);
              float z[4], a[4];
              unpack4(pre, z);
#pragma unroll
              for (int q = 0; q < 4; ++q) {
                const uint32_t zu = __float_as_uint(z[q]);
                float da;
                if (use_lut) a[q] = lut_act(sm, zu);
                else small_act<EVAL>(p.act, z[q], &a[q], &da);
              }
              if (p.out0) *(uint2*)(p.out0 + o) = pre;
              *(uint2*)(p.out1 + o) = pack4(a[0], a[1], a[2], a[3]);
            } else {
              float z[4], a[4], dv[4];
              unpack4(*(const uint2*)(p.hpre_in + o), z);
#pragma unroll
              for (int q = 0; q < 4; ++q) {
                const uint32_t zu = __float_as_uint(z[q]);
                if (use_lut) {
                  if (EPI == EPI_DHQ) dv[q] = lut_act_d(sm, zu);
                  else lut_act_both(sm, zu, &a[q], &dv[q]);
                } else {
                  small_act<EVAL>(p.act, z[q], &a[q], &dv[q]);
                }
              }
              *(uint2*)(p.out0 + o) = pack4(c[0] * dv[0], c[1] * dv[1], c[2] * dv[2], c[3] * dv[3]);
              if (EPI == EPI_DH) *(uint2*)(p.out1 + o) = pack4(a[0], a[1], a[2], a[3]);
            }
          }
        }
      }
    }
  }
}

template <int BM, bool WT, int EPI, bool EVAL>
__global__ __launch_bounds__(kSmallThreads, 2) void rows_gemm_small_bf16(const SmallArgs p) {
  __shared__ __align__(1024) unsigned char smem[SmallCfg<BM>::kLds];
  rows_small_block<BM, WT, EPI, EVAL>(p, smem, blockIdx.x, gridDim.x);
}

}  // namespace flexmoe
