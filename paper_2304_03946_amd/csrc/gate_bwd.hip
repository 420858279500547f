// The rest of a trainable layer: the gradient through the gate (paper Eq. 3-4) and the bias
// gradients of the expert FFN (Eq. 2).
//
//   dg[t,j] = <dY_t, Yp[dest[t*k+j]]>                          (Eq. 4 is linear in the gate values)
//   dl[t,j] = g[t,j] * (dg[t,j] - sum_i g[t,i] dg[t,i])         (softmax over the k kept logits, Eq. 3)
//   dX_t   += sum_j dl[t,j] * W_g[:, e_j]                       (logits l = x.W_g)
//   dW_g[:,e] = sum over the assignments routed to e of dl * x  (same sum, seen from the weights)
//   db2_e = sum of the rows of dYp in e's buckets, db1_e = the same for dHpre
//
// All of it is HBM-bound row traffic, on small layers the latency of a few dependent loads per launch.  The
// per-expert sums run over the bucketed layout (an expert's rows are contiguous per vExpert), in two stages with a
// fixed summation order, so results are reproducible: no atomics.  What does not depend on each other shares a
// launch: both bias gradients (two launches in all); the logit gradients and the transposed copy of W_g; then the
// gate's share of dX and the partial sums of dW_g; then their final sums.  Eight launches of 4.6 - 15 us became five:
// 5003 tokens (d 192, f 768, E 12) 49.2 -> 29.0 us, 1500 tokens (d 1024, f 4096, E 32) 47.2 -> 30.7 (replayed from a graph).
#include "common.h"

namespace flexmoe {

constexpr int kBwdThreads = 256;
constexpr int kBwdWaves = kBwdThreads / kWave;
constexpr int kChunkRows = 128;                    // rows of one bucket summed by one workgroup
constexpr int kSumThreads = 512;                   // of the partial sums: every wave has its 16 rows in flight at once
constexpr int kSumWaves = kSumThreads / kWave;
constexpr int kSumChains = 4;                      // sums per column: rows w, w + 4, ..
constexpr int kMaxGridY = 65535;
constexpr int kChunkCols = 512;                    // columns per workgroup: 64 lanes x 16 bytes of bf16

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int o = kWave / 2; o > 0; o >>= 1) v += __shfl_xor(v, o);
  return v;
}

// First launch of the gate's backward pass.  Workgroups below token_blocks, a wave per token: the k gate-value
// gradients and the logit gradients.  The others: wgT = W_g transposed ([E, d]), so that an expert's column is a row
// (the gate weights are small: no tiling).
template <typename T>
__global__ __launch_bounds__(kBwdThreads) void gate_bwd_logits_kernel(
    const T* __restrict__ dy, const T* __restrict__ yp, const int32_t* __restrict__ dest, const float* __restrict__ w,
    int N, int k, int d, float* __restrict__ dl, int token_blocks, const T* __restrict__ wg, int E, T* __restrict__ wgT) {
  constexpr int VN = Vec16<T>::n;
  if ((int)blockIdx.x >= token_blocks) {
    const int n = d * E, stride = (gridDim.x - token_blocks) * kBwdThreads;
    for (int i = (blockIdx.x - token_blocks) * kBwdThreads + threadIdx.x; i < n; i += stride) {
      const int e = i / d, r = i % d;              // consecutive threads write consecutive outputs
      wgT[i] = wg[(size_t)r * E + e];
    }
    return;
  }
  const int lane = threadIdx.x % kWave;
  const int wave = blockIdx.x * kBwdWaves + threadIdx.x / kWave;
  const int nwaves = token_blocks * kBwdWaves;
  const int vec_per_row = d / VN;
  for (int t = wave; t < N; t += nwaves) {
    const uint4* dy_row = (const uint4*)(dy + (size_t)t * d);
    float dg[FLEXMOE_MAX_TOPK], g[FLEXMOE_MAX_TOPK];
    int row[FLEXMOE_MAX_TOPK];
    float inner = 0.f;
#pragma unroll
    for (int j = 0; j < FLEXMOE_MAX_TOPK; ++j) {
      row[j] = j < k ? dest[t * k + j] : 0;
      g[j] = j < k ? w[t * k + j] : 0.f;
    }
#pragma unroll
    for (int j = 0; j < FLEXMOE_MAX_TOPK; ++j) {
      dg[j] = 0.f;
      if (j < k) {
        const uint4* yp_row = (const uint4*)(yp + (size_t)row[j] * d);
        float acc = 0.f;
        for (int c = lane; c < vec_per_row; c += kWave) {
          float u[VN], v[VN];
          Vec16<T>::unpack(dy_row[c], u);
          Vec16<T>::unpack(yp_row[c], v);
#pragma unroll
          for (int q = 0; q < VN; ++q) acc = fmaf(u[q], v[q], acc);
        }
        dg[j] = wave_sum(acc);
        inner = fmaf(g[j], dg[j], inner);
      }
    }
#pragma unroll
    for (int j = 0; j < FLEXMOE_MAX_TOPK; ++j)
      if (j < k && lane == 0) dl[t * k + j] = g[j] * (dg[j] - inner);
  }
}

// The gate path's share of dX, added in place: a wave per token, wave `wave` of `nwaves`.
template <typename T>
__device__ __forceinline__ void gate_bwd_dx(const float* __restrict__ dl, const int32_t* __restrict__ idx,
                                            const T* __restrict__ wgT, int N, int k, int d, T* __restrict__ dx, int wave,
                                            int nwaves) {
  constexpr int VN = Vec16<T>::n;
  const int lane = threadIdx.x % kWave;
  const int vec_per_row = d / VN;
  for (int t = wave; t < N; t += nwaves) {
    float dlv[FLEXMOE_MAX_TOPK];
    int e[FLEXMOE_MAX_TOPK];
#pragma unroll
    for (int j = 0; j < FLEXMOE_MAX_TOPK; ++j) {
      dlv[j] = j < k ? dl[t * k + j] : 0.f;
      e[j] = j < k ? idx[t * k + j] : 0;
    }
    uint4* dx_row = (uint4*)(dx + (size_t)t * d);
    for (int c = lane; c < vec_per_row; c += kWave) {
      float acc[VN];
      Vec16<T>::unpack(dx_row[c], acc);
#pragma unroll
      for (int j = 0; j < FLEXMOE_MAX_TOPK; ++j)
        if (j < k) {
          float v[VN];
          Vec16<T>::unpack(((const uint4*)(wgT + (size_t)e[j] * d))[c], v);
#pragma unroll
          for (int q = 0; q < VN; ++q) acc[q] = fmaf(dlv[j], v[q], acc[q]);
        }
      dx_row[c] = Vec16<T>::pack(acc);
    }
  }
}

// Chunks: every bucket is cut into pieces of kChunkRows rows; flat chunk ids run over the buckets
// in ascending vExpert id.  chunk_start[v] = id of bucket v's first chunk (one wave's scan).
__device__ __forceinline__ void chunk_starts(const int32_t* __restrict__ voff, int V, int* chunk_start) {
  if (threadIdx.x < kWave) {
    const int lane = threadIdx.x;
    const int per = (V + kWave - 1) / kWave;
    int cnt[FLEXMOE_MAX_VEXPERTS / kWave];
    int sum = 0;
#pragma unroll
    for (int q = 0; q < FLEXMOE_MAX_VEXPERTS / kWave; ++q) {
      const int v = lane * per + q;
      cnt[q] = 0;
      if (q < per && v < V) cnt[q] = (voff[v + 1] - voff[v] + kChunkRows - 1) / kChunkRows;
      sum += cnt[q];
    }
    int incl = sum;
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
      const int up = __shfl_up(incl, o);
      if (lane >= o) incl += up;
    }
    int start = incl - sum;
#pragma unroll
    for (int q = 0; q < FLEXMOE_MAX_VEXPERTS / kWave; ++q) {
      const int v = lane * per + q;
      if (q < per && v <= V) chunk_start[v] = start;     // entry V = total number of chunks
      start += cnt[q];
    }
    if (lane == kWave - 1 && per * kWave == V) chunk_start[V] = incl;
  }
  __syncthreads();
}

// Columns per workgroup of stage 1: 64 lanes x 16 bytes.
template <typename T> static constexpr int kSumCols = kChunkCols * Vec16<T>::n / 8;

// Stage 1: partial[chunk, c] = sum over the chunk's rows of weight(row) * in[row, c], fp32.
// WEIGHTED: weight(row p) = row_w[src[p]] (a value per assignment id); otherwise 1.
// Rows w, w + 4, ... of the chunk are summed in ascending order, the first half of them by wave w, which hands its sum to
// wave w + 4 for the second half (whose rows have come meanwhile); the four sums are added in order through
// LDS.  One workgroup sums the `chunk` it is given for the column blocks cb, cb + cb_step, ..: those of
// the first matrix s0, then those of a second one, s1.
template <typename T> struct SumInput {
  const T* in;
  int C, blocks;                                     // columns, column blocks (0: no such matrix)
  float* partial;
};
template <typename T, bool WEIGHTED>
__device__ __forceinline__ void bucket_colsum_partial(const SumInput<T>& s0, const SumInput<T>& s1, const float* __restrict__ row_w,
                                                      const int32_t* __restrict__ src, const int32_t* __restrict__ voff,
                                                      int V, int chunk, int cb, int cb_step) {
  constexpr int VN = Vec16<T>::n, U = kChunkRows / kSumWaves;
  __shared__ int chunk_start[FLEXMOE_MAX_VEXPERTS + 1];
  __shared__ float red[kSumChains][kWave][VN];
  __shared__ float weight[kChunkRows];
  chunk_starts(voff, V, chunk_start);
  if (chunk >= chunk_start[V]) return;               // uniform
  // bucket of this chunk: the last v with chunk_start[v] <= chunk (binary search, every thread)
  int lo = 0, hi = V - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (chunk_start[mid] <= chunk) lo = mid;
    else hi = mid - 1;
  }
  const int v = lo;
  // uniform: a row's address in scalar registers
  const int row0 = __builtin_amdgcn_readfirstlane(voff[v] + (chunk - chunk_start[v]) * kChunkRows);
  const int rows = __builtin_amdgcn_readfirstlane(min(kChunkRows, voff[v + 1] - row0));
  const int lane = threadIdx.x % kWave, wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave), chain = wave % kSumChains;
  const bool second = wave >= kSumChains;
  if (WEIGHTED) {
    if ((int)threadIdx.x < rows) weight[threadIdx.x] = row_w[src[row0 + threadIdx.x]];
    __syncthreads();
  }
  for (; cb < s0.blocks + s1.blocks; cb += cb_step) {
    const SumInput<T>& m = cb < s0.blocks ? s0 : s1;
    const int col = (cb < s0.blocks ? cb : cb - s0.blocks) * kSumCols<T> + lane * VN;
    const int first = chain + (second ? U * kSumChains : 0);
    uint4 raw[U];
    if (col < m.C) {
#pragma unroll
      for (int i = 0; i < U; ++i)
        raw[i] = *(const uint4*)((const char*)(m.in + (size_t)(row0 + min(first + i * kSumChains, rows - 1)) * m.C) + (uint32_t)col * sizeof(T));
    }
    auto add = [&](bool resume) {
      float acc[VN];
#pragma unroll
      for (int q = 0; q < VN; ++q) acc[q] = resume ? red[chain][lane][q] : 0.f;
      if (col < m.C) {
#pragma unroll
        for (int i = 0; i < U; ++i) {
          const int r = first + i * kSumChains;
          if (r < rows) {
            const float wt = WEIGHTED ? weight[r] : 1.f;
            float u[VN];
            Vec16<T>::unpack(raw[i], u);
#pragma unroll
            for (int q = 0; q < VN; ++q) acc[q] = fmaf(wt, u[q], acc[q]);
          }
        }
      }
#pragma unroll
      for (int q = 0; q < VN; ++q) red[chain][lane][q] = acc[q];
    };
    if (!second) add(false);
    __syncthreads();
    if (second) add(true);
    __syncthreads();
    if (wave == 0 && col < m.C) {
#pragma unroll
      for (int q = 0; q < VN; ++q) {
        float s = red[0][lane][q];
#pragma unroll
        for (int ww = 1; ww < kSumChains; ++ww) s += red[ww][lane][q];
        m.partial[(size_t)chunk * m.C + col + q] = s;
      }
    }
    __syncthreads();
  }
}
template <typename T>
__global__ __launch_bounds__(kSumThreads, 4) void bias_partial_kernel(SumInput<T> s0, SumInput<T> s1, const int32_t* __restrict__ voff, int V) {
  bucket_colsum_partial<T, false>(s0, s1, nullptr, nullptr, voff, V, blockIdx.x, blockIdx.y, gridDim.y);
}
// Second launch of the gate's backward pass: blockIdx.y < token_rows adds the gate's share of dX, the others sum dW_g's chunks.
template <typename T>
__global__ __launch_bounds__(kSumThreads, 4) void gate_bwd_apply_kernel(const float* __restrict__ dl, const int32_t* __restrict__ idx,
                                                                    const T* __restrict__ wgT, int N, int k, int d,
                                                                    T* __restrict__ dx, int token_rows, SumInput<T> xp,
                                                                    const int32_t* __restrict__ src,
                                                                    const int32_t* __restrict__ voff, int V) {
  if ((int)blockIdx.y < token_rows)
    gate_bwd_dx<T>(dl, idx, wgT, N, k, d, dx, (blockIdx.y * gridDim.x + blockIdx.x) * kSumWaves + threadIdx.x / kWave,
                   token_rows * gridDim.x * kSumWaves);
  else
    bucket_colsum_partial<T, true>(xp, SumInput<T>{nullptr, 0, 0, nullptr}, dl, src, voff, V, blockIdx.x, blockIdx.y - token_rows,
                                   gridDim.y - token_rows);
}

// Stage 2: out[e, c] = sum of the partials of e's chunks.  One workgroup per (expert, 64 columns):
// the expert's chunks, numbered through its buckets in ascending vExpert id and ascending row
// order, are dealt round-robin to the four waves; each wave adds its chunks in that order (four
// loads in flight), then the waves' sums are added in wave order.  A fixed order: reproducible.
// TRANSPOSED: out is [C, E] (the gate weights' layout).  Up to two sets of sums: the second one's column blocks follow
// the first one's.
template <typename T> struct SumOutput {
  const float* partial;
  int C, blocks;                                      // columns, blocks of 64 of them
  T* out;
};
template <typename T, bool TRANSPOSED>
__global__ __launch_bounds__(kBwdThreads) void bucket_colsum_final_kernel(const SumOutput<T> s0, const SumOutput<T> s1,
                                                                          const int32_t* __restrict__ voff,
                                                                          const int32_t* __restrict__ owner, int V, int E) {
  const bool second = (int)blockIdx.x >= s0.blocks;
  const float* partial = second ? s1.partial : s0.partial;
  const int C = second ? s1.C : s0.C;
  T* out = second ? s1.out : s0.out;
  __shared__ int chunk_start[FLEXMOE_MAX_VEXPERTS + 1];
  __shared__ int list[FLEXMOE_MAX_VEXPERTS];          // the expert's buckets, ascending
  __shared__ int nlist;
  __shared__ float red[kBwdWaves][kWave];
  chunk_starts(voff, V, chunk_start);
  const int e = blockIdx.y;
  const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
  {
    // ascending list of the expert's buckets: ballot compaction, two buckets per thread
    constexpr int kSeg = FLEXMOE_MAX_VEXPERTS / kWave;             // 64-bucket segments
    __shared__ int seg_count[kSeg];
    const unsigned long long lt = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    bool mine[kSeg / kBwdWaves];
    int pos[kSeg / kBwdWaves];
#pragma unroll
    for (int h = 0; h < kSeg / kBwdWaves; ++h) {
      const int v = (h * kBwdWaves + wave) * kWave + lane;
      mine[h] = v < V && owner[v] == e;
      const unsigned long long m = __ballot(mine[h]);
      pos[h] = __popcll(m & lt);
      if (lane == 0) seg_count[h * kBwdWaves + wave] = __popcll(m);
    }
    __syncthreads();
#pragma unroll
    for (int h = 0; h < kSeg / kBwdWaves; ++h) {
      const int seg = h * kBwdWaves + wave;
      int base = 0;
      for (int q = 0; q < seg; ++q) base += seg_count[q];
      if (mine[h]) list[base + pos[h]] = seg * kWave + lane;
    }
    if (threadIdx.x == 0) {
      int n = 0;
      for (int q = 0; q < kSeg; ++q) n += seg_count[q];
      nlist = n;
    }
    __syncthreads();
  }
  const int c = (blockIdx.x - (second ? s0.blocks : 0)) * kWave + lane;
  float s = 0.f;
  if (c < C) {
    int ord = 0;                                       // running number of the expert's chunks
    for (int i = 0; i < nlist; ++i) {
      const int v = list[i];
      const int first = chunk_start[v], cnt = chunk_start[v + 1] - first;
      // this wave's chunks of the bucket: ordinals congruent to `wave` modulo 4
      int j = (wave - ord % kBwdWaves + kBwdWaves) % kBwdWaves;
      for (; j + 3 * kBwdWaves < cnt; j += 4 * kBwdWaves) {
        const float p0 = partial[(size_t)(first + j) * C + c];
        const float p1 = partial[(size_t)(first + j + kBwdWaves) * C + c];
        const float p2 = partial[(size_t)(first + j + 2 * kBwdWaves) * C + c];
        const float p3 = partial[(size_t)(first + j + 3 * kBwdWaves) * C + c];
        s += p0;
        s += p1;
        s += p2;
        s += p3;
      }
      for (; j < cnt; j += kBwdWaves) s += partial[(size_t)(first + j) * C + c];
      ord += cnt;
    }
  }
  red[wave][lane] = s;
  __syncthreads();
  if (wave == 0 && c < C) {
    float t = red[0][lane];
    for (int ww = 1; ww < kBwdWaves; ++ww) t += red[ww][lane];
    Elem<T>::store(out + (TRANSPOSED ? (size_t)c * E + e : (size_t)e * C + c), t);
  }
}

static int max_chunks(int A, int V) { return A / kChunkRows + V; }
static size_t partial_bytes(int A, int V, int C) { return align_up((size_t)max_chunks(A, V) * C * sizeof(float), 256); }

template <typename T> static SumInput<T> sum_input(const void* in, int C, float* partial) {
  return SumInput<T>{(const T*)in, C, in ? (C + kSumCols<T> - 1) / kSumCols<T> : 0, partial};
}
template <typename T> static SumOutput<T> sum_output(const float* partial, int C, void* out) {
  return SumOutput<T>{partial, C, out ? (C + kWave - 1) / kWave : 0, (T*)out};
}
template <typename T, bool TRANSPOSED>
static hipError_t launch_final_sums(const SumOutput<T>& s0, const SumOutput<T>& s1, const int32_t* voff, const int32_t* owner,
                                    int V, int E, hipStream_t s) {
  hipLaunchKernelGGL((bucket_colsum_final_kernel<T, TRANSPOSED>), dim3(s0.blocks + s1.blocks, E), dim3(kBwdThreads), 0, s, s0, s1,
                     voff, owner, V, E);
  return hipGetLastError();
}

size_t gate_bwd_ws_bytes(int A, int d, int E, int V, int dtype) {
  const size_t s = dtype == FLEXMOE_BF16 ? 2 : 4;
  return align_up((size_t)E * d * s, 256) + partial_bytes(A, V, d);
}

template <typename T>
static hipError_t gate_bwd_t(const void* wg, const int32_t* idx, const float* w, const void* dy,
                             const void* yp, const void* xp, const int32_t* dest, const int32_t* src,
                             const int32_t* voff, const int32_t* owner, int N, int d, int E, int k, int V, float* dl,
                             void* dx, void* dwg, void* ws, hipStream_t s) {
  T* wgT = (T*)ws;
  float* partial = (float*)((char*)ws + align_up((size_t)E * d * sizeof(T), 256));
  const int A = N * k;
  const int token_blocks = min((N + kBwdWaves - 1) / kBwdWaves, 256 * 8);
  if (N > 0)
    hipLaunchKernelGGL((gate_bwd_logits_kernel<T>), dim3(token_blocks + min(256, (d * E + kBwdThreads - 1) / kBwdThreads)),
                       dim3(kBwdThreads), 0, s, (const T*)dy, (const T*)yp, dest, w, N, k, d, dl, token_blocks, (const T*)wg, E, wgT);
  // dW_g[:, e] = sum over e's bucket rows p of dl[src[p]] * Xp[p, :]
  const SumInput<T> in = sum_input<T>(xp, d, partial);
  if (N > 0) {
    const int gx = max_chunks(A, V);
    // a wave per token, in at most 1024 workgroups (four per compute unit)
    const int token_rows = max(1, min(((N + kSumWaves - 1) / kSumWaves + gx - 1) / gx, 1024 / gx));
    hipLaunchKernelGGL((gate_bwd_apply_kernel<T>), dim3(gx, token_rows + min(in.blocks, kMaxGridY - token_rows)), dim3(kSumThreads), 0,
                       s, dl, idx, (const T*)wgT, N, k, d, (T*)dx, token_rows, in, src, voff, V);
  }
  return launch_final_sums<T, true>(sum_output<T>(partial, d, dwg), sum_output<T>(nullptr, 0, nullptr), voff, owner, V, E, s);
}

hipError_t launch_gate_bwd(const void* wg, const int32_t* idx, const float* w, const void* dy,
                           const void* yp, const void* xp, const int32_t* dest, const int32_t* src,
                           const int32_t* voff, const int32_t* owner, int N, int d, int E, int k, int V, int dtype,
                           float* dl, void* dx, void* dwg, void* ws, hipStream_t s) {
  if (dtype == FLEXMOE_F32)
    return gate_bwd_t<float>(wg, idx, w, dy, yp, xp, dest, src, voff, owner, N, d, E, k, V, dl, dx, dwg, ws, s);
  return gate_bwd_t<bf16_t>(wg, idx, w, dy, yp, xp, dest, src, voff, owner, N, d, E, k, V, dl, dx, dwg, ws, s);
}

// The FFN backward leaves dHpre [A, f] at the start of its workspace; the activations behind it
// are dead once the weight gradients are done, so the partial sums go there.
size_t bias_grads_ws_bytes(int A, int d, int f, int V, int dtype) {
  const size_t s = dtype == FLEXMOE_BF16 ? 2 : 4;
  return align_up((size_t)A * f * s, 256) + partial_bytes(A, V, d) + partial_bytes(A, V, f);
}

template <typename T>
static hipError_t bias_grads_t(const void* dyp, const int32_t* voff, const int32_t* owner, int A, int d, int f, int E,
                               int V, void* db1, void* db2, void* ws, hipStream_t s) {
  const T* dhpre = (const T*)ws;
  float* partial1 = (float*)((char*)ws + align_up((size_t)A * f * sizeof(T), 256));
  float* partial2 = (float*)((char*)partial1 + partial_bytes(A, V, f));
  if (!db1 && !db2) return hipSuccess;
  const SumInput<T> s1 = sum_input<T>(db1 ? dhpre : nullptr, f, partial1), s2 = sum_input<T>(db2 ? dyp : nullptr, d, partial2);
  if (A > 0)
    hipLaunchKernelGGL((bias_partial_kernel<T>), dim3(max_chunks(A, V), min(s1.blocks + s2.blocks, kMaxGridY)), dim3(kSumThreads), 0, s,
                       s1, s2, voff, V);
  return launch_final_sums<T, false>(sum_output<T>(partial1, f, db1), sum_output<T>(partial2, d, db2), voff, owner, V, E, s);
}

hipError_t launch_bias_grads(const void* dyp, const int32_t* voff, const int32_t* owner, int A, int d, int f, int E,
                             int V, int dtype, void* db1, void* db2, void* ws, hipStream_t s) {
  if (dtype == FLEXMOE_F32) return bias_grads_t<float>(dyp, voff, owner, A, d, f, E, V, db1, db2, ws, s);
  return bias_grads_t<bf16_t>(dyp, voff, owner, A, d, f, E, V, db1, db2, ws, s);
}

}  // namespace flexmoe
