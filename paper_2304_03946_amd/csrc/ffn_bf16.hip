// bf16 expert FFN (paper Eq. 2) per vExpert bucket, forward and backward, as grouped GEMMs on
// the CDNA4 matrix cores (fp32 accumulation).
//
// Layers with enough rows for their experts share one 256x256 workgroup tile, one workgroup per compute unit: eight wavefronts with
// 128x64 accumulator blocks (32 tiles of v_mfma_f32_16x16x32_bf16) in the direct-to-LDS kernels that
// serve contractions of whole 128-wide rounds, four wavefronts with 128x128 blocks (16 tiles of
// v_mfma_f32_32x32x16_bf16) in the register-staged kernel that serves the rest.  Rows products with few rows per expert or
// little output have kernels of their own, with 32- or 64-row tiles and contraction segments (ffn_bf16_small.h; small_rows below
// draws the line).
//
//  * rows GEMMs: C[rows of bucket v, :] = In[rows of v, :] . W_owner(v)    (fwd GEMM1/GEMM2,
//    bwd dH and dXp).  The row dimension is cut per bucket: a device-side lookup maps the flat
//    row-tile index to (vExpert, tile inside it), so highly skewed bucket sizes need no host
//    synchronisation.  Rows of a ragged last tile are clamped on load and dropped on store.
//  * weight-gradient GEMMs: dW_e = sum over the vExperts v of e of L_v^T . R_v -- the contraction
//    runs over the tokens of every bucket of e in ascending vExpert id inside one accumulator,
//    which is the single-GPU image of the paper's replica gradient synchronisation.  Output tiles
//    are issued hottest expert first so the long contractions start early; when one expert's
//    contraction is much longer than the chip-wide average per compute unit it is cut into
//    segments that accumulate into fp32 partial tiles, summed in a fixed order by a second kernel
//    (the result does not depend on scheduling).
//
// Two operand pipelines:
//  * direct-to-LDS (rows_gemm_persist_bf16 where K is a multiple of 128, i.e. for every benchmark shape;
//    wgrad_gemm_persist_bf16, wgrad_gemm_dma_bf16; rows_gemm_small_bf16 has its own): global_load_lds_dwordx4 copies 32-wide K tiles
//    straight into one of four LDS stages (no register staging, no LDS store instructions); an
//    operand whose contraction index is strided in memory is copied as stored and transposed on
//    the way out of LDS by ds_read_tr16_b64.  The loads of the tile three steps ahead are
//    spread between the MFMAs of the current one, and one LDS-only barrier per K tile orders
//    stage reuse.  What bounds the K loop is the energy of bringing the operands into LDS (the stripped loop
//    without its direct loads runs 27-41 % faster on random operands, 9-18 % on constant ones: csrc/probe).
//    (Weight gradients with few rows per expert or few output tiles: 128 x 128 tiles, ffn_bf16_wgrad_small.h.)
//  * register-staged (rows_gemm_bf16; rows products with any other K that is a multiple of 8): 64-wide K
//    tiles through registers into two LDS stages, strided operands transposed 8x8 in registers.
//
// LDS tiles are XOR-swizzled at 16-byte chunk granularity so that fragment reads and tile
// writes are free of bank conflicts (measured: SQ_LDS_BANK_CONFLICT = 0).
// The MFMA is issued as (weights-fragment, activations-fragment) so that a lane ends up with 4
// consecutive output columns of one output row; the epilogue passes the accumulators through a
// wave-private LDS patch so that global stores fill whole 128-byte lines.
// GELU and its derivative act on bf16-rounded arguments, so where K is a multiple of 128 both are read from a table indexed
// by the argument's bits (constant data in the code object, computed from the fp64 formulas when the
// library is built; outside the table's range GELU equals ReLU to below bf16 resolution).
//
// The direct-to-LDS kernels are persistent: 256 workgroups, one per compute unit, each walking its share
// of the output tiles and issuing the next tile's first operand loads while the current tile's K loop
// drains (ffn_bf16_persist.h, wgrad_gemm_persist_bf16; weight gradients whose output is not a whole
// number of 256 x 256 tiles keep one workgroup per tile, wgrad_gemm_dma_bf16).
//
// Layout of the sources: ffn_bf16_tile.h (tile mapping, fragments, activation tables, epilogues, the
// register-staged kernel), ffn_bf16_dma.h (direct-to-LDS pipeline, one rows tile on it),
// ffn_bf16_persist.h (persistent rows kernels and their row-tile table), ffn_bf16_small.h (rows kernels for few rows
// and their plan), ffn_bf16_wgrad.h (weight-gradient plan and kernels), ffn_bf16_wgrad_small.h (128 x 128 weight-gradient tiles); this
// file holds the host side.
#include <algorithm>

#include "common.h"
#include "ffn_bf16_tile.h"
#include "ffn_bf16_dma.h"
#include "ffn_bf16_persist.h"
#include "ffn_bf16_small.h"
#include "ffn_bf16_wgrad.h"
#include "ffn_bf16_wgrad_small.h"

namespace flexmoe {

// =============================================================================================
// host side
// =============================================================================================
// Weight gradient: how many 32-token K tiles one workgroup contracts before the expert's sum is
// cut into a further segment: a compute unit's even share of all (output tile, K tile) pairs
// but at least 32 (shorter segments measured slower: more fp32 partial tiles), so that the hottest expert's contraction is
// no longer one serial K loop; at least 16 where the gradient of an expert is at most four output tiles and even those
// leave most of the chip idle (a share of at most 8 K tiles).  Whole training steps, f = 4 d, k 2, in us, 32 and 16: d 128,
// 4800 rows of 12 experts 150, 133; d 192, 9600 of 12 182, 169; d 256, 9600 of 12 201, 190, 16000 of 40 (share 7.8) 269, 260; past the
// line, 18400 of 40 (share 9) 274, 271, 32000 of 40 (share 15.6) 350, 365; d 512 (16 output tiles), 4000 of 40 233, 265.  0 = no cutting:
// when a segment would hold more than a quarter of all tokens (many output tiles per expert: the
// grid is busy anyway, and the fp32 partial tiles would be large).
constexpr int kComputeUnits = 256;
static int wgrad_seg_tiles(int A, int d, int f) {
  const long long out_tiles = (long long)((d + BM - 1) / BM) * ((f + BN - 1) / BN);
  const long long k_tiles = A / DK;
  const long long share = k_tiles * out_tiles / kComputeUnits;
  const long long least = share <= 8 && out_tiles <= 4 ? 16 : 32;
  const long long seg = std::max(share, least);
  return 4 * seg <= k_tiles ? (int)seg : 0;
}
// Upper bound over all load distributions: extra segments (beyond one per expert).
static int wgrad_extra_segments(int A, int V, int seg_tiles) { return seg_tiles ? (A / DK + V) / seg_tiles : 0; }

// Whether a call's weight gradients go to the 128 x 128 tiles of wgrad_gemm_small_bf16, three workgroups per compute unit, instead of
// the 256 x 256 ones (half the operand traffic per product, but one workgroup per compute unit, whose look-ups, first loads and
// stores have nothing beside them).  Whole backward passes, f = 4 d unless given, us, 256 and 128:
//  * the gradient of an expert is at most four 256 x 256 tiles, and a compute unit's even share of K tiles x output tiles at most 180, or 100
//    with four tiles: d 64, E 8, 60000 rows 139, 103; d 192, E 12, 10000 rows 115, 87, 420000 rows (share 154) 1263, 1207; d 256, E 8, 3200 rows
//    97, 66, 42000 rows (20) 216, 206, 130000 rows (63) 540, 523; past the line: d 192, E 12, 520000 rows (190) 1430, 1443; d 256, E 8,
//    230000 rows (112) 831, 843; E 64, 260000 rows (127) 863, 931; d 512, f 512, E 8, 400000 rows (195) 1167, 1244.  (In between the large tiles
//    have their moments, where they fill their last round: d 512, f 512, 60000 rows 234, 243; d 504, f 504 296, 317);
//  * the small tiles cover at most 0.8 of what the large ones do (d up to 128, 320, 384): d 128, E 8, 520000 rows 859, 760; d 384, E 12, 24000
//    rows 286, 259, 260000 rows 1887, 1791; d 640, f 1920, E 8, 60000 rows 813, 754; 0.83 (d 640, f 2560) is past the line: 60000 rows 1060, 1062;
//  * up to 112 rows per expert: d 1024, E 32, 32 rows 308, 280, 94 rows 382, 366; d 2048, E 64, 32 rows 1896, 1846, 96 rows 2426, 2410;
//    past the line: 160 rows 470, 477 and 2578, 2684;
//  * an even share of at most 20 K tiles x output tiles per compute unit: d 512, E 32 (share 16) 249, 230; d 1024, f 2048, E 8 (20) 206, 190;
//    d 512, f 1024, E 128 (20) 372, 344; past the line: d 512, E 32 (25) 291, 302; d 1024, f 2048, E 8 (31) 276, 283;
//    d 512, f 1024, E 128 (32) 428, 434.
// Not for layers of 2^26 columns and more: an operand's 32-bit offsets are bytes here (elements in the 256 x 256 kernels), of up to 31 rows.
static bool wgrad_small(int A, int d, int f, int E) {
  if (std::max(d, f) >= 1 << 26) return false;
  const long long large = (long long)((d + BM - 1) / BM) * ((f + BN - 1) / BN), small = (long long)((d + GT - 1) / GT) * ((f + GT - 1) / GT);
  return 5 * small <= 16 * large || A <= 112ll * E || A / DK * large <= (large <= 3 ? 180 : large == 4 ? 100 : 20) * kComputeUnits;
}
// A grid's dimension is fewer than 2^32 threads: of more, HIP runs what is left modulo 2^32, and reports nothing.  Both products in one
// launch are twice what either is: layers of 8 to 32 features with 2^30 columns over all experts (they fit the card's memory with few
// rows) need the launches apart.
constexpr long long kMaxGradBlocks = (1ll << 32) / kGradThreads - 1;
static bool wgrad_joint(unsigned blocks2, unsigned blocks1) { return (long long)blocks2 + blocks1 <= kMaxGradBlocks; }
static int wgrad_seg_rows_max(int A, int d, int f, int E, int V) { return E + wgrad_extra_segments(A, V, wgrad_seg_tiles(A, d, f)); }

static int max_row_tiles(int A, int V) { return A / BM + V; }

// Partial tiles of the split last round (see lookup_row_tile): none for grids that can never fill a
// round of workgroups or whose contraction is short (the fp32 round trip would cost more than the idle
// compute units).
constexpr int kSplitMinK = 1024;
static size_t rows_split_bytes(int A, int V, int K, int NC) {
  if (K % 128 || K < kSplitMinK) return 0;
  if ((long long)max_row_tiles(A, V) * ((NC + BN - 1) / BN) <= kSplitUnits) return 0;
  return (size_t)kSplitMaxSlots * BM * BN * sizeof(float);
}

// The workspace must not shrink where the number of rows grows (a caller sizes it for the largest batch and passes it to
// every smaller one), but the slots do: longer segments leave fewer.  So what is reserved for A rows is the most that any
// number of rows up to A takes, from the last number of K tiles k of each rule: segments of 16 (share <= 8, at most four
// output tiles), of 32 (share <= 32), and of a share s > 32, where (k + V) / s < (34 c + V) / 33, c = 256 / output tiles,
// because k < (s + 1) c.  More than 65 output tiles are never cut.
static int wgrad_slots_reserved(int A, int d, int f, int V) {
  const long long out_tiles = (long long)((d + BM - 1) / BM) * ((f + BN - 1) / BN);
  const int k_tiles = A / DK;
  if (out_tiles > kComputeUnits / 4 + 1) return 0;
  const int out = (int)out_tiles, k16 = (9 * kComputeUnits - 1) / out, k32 = (33 * kComputeUnits - 1) / out;
  int extra = -1;                                         // segments beyond one per expert; slots = 2 extra + 1
  if (out <= 4 && k_tiles >= 4 * 16) extra = (std::min(k_tiles, k16) + V) / 16;
  if (std::min(k_tiles, k32) >= 4 * 32) extra = std::max(extra, (std::min(k_tiles, k32) + V) / 32);
  if (k_tiles > k32) extra = std::max(extra, (34 * kComputeUnits + V * out - 1) / (33 * out));
  return 2 * extra + (extra >= 0 ? 1 : 2);
}
// fp32 partial tiles of one weight-gradient product.
static size_t wgrad_tail_bytes(int A, int d, int f, int V) {
  return align_up((size_t)wgrad_slots_reserved(A, d, f, V) * d * f * sizeof(float), 256);
}
// Work list of both.
static size_t wgrad_plan_reserved(int A, int d, int f, int E, int V) {
  return align_up(wgrad_plan_bytes(E + wgrad_slots_reserved(A, d, f, V) / 2, E, V), 256);
}

// Which rows kernels a call of these sizes takes: 32 or 64 = rows_gemm_small_bf16 with row tiles of that many rows, 0 = the
// 256 x 256 kernels.  The loads are not known here (skewed: a few experts have ten times the mean, most have less).
//
// Either pass reads an expert's weights once per row tile: the small one for about A / 64 + E / 2 tiles (half an empty one per
// expert), the other for at least one per vExpert.  How many times as many tiles the small one can afford falls with the size
// of a weight matrix, as re-reading it counts more than the matrix cores: 1.4 from 2^23 elements, 1.7 from 2^20, 2.4 below.
// Forward passes, f = 4 d unless given, in us, 256-row and 64-row tiles by mean rows per expert (loads between even and Zipf 1.5):
//   d 2048, E 64, V 64: 60 1134, 1123;             past the line: 70 1138, 1239; 100 1280, 1411
//   d 2048, E 64, V 96: 100 1511, 1425;                           130 1538, 1650
//   d 2048, E 32, V 40:                                           100 648, 656; 130 647, 786
//   d 1024, E 64, V 64: 70 355, 324;                              85 345, 338; 100 352, 375
//   d 1024, E 32, V 48: 100 237, 226; 130 243, 237;               160 247, 250; 200 280, 296
//   d 1024, E 16, V 64: 380 271, 263
//   d 1024, E 128, V 160: 100 698, 701;                           130 714, 832
//   d 512, E 128, V 160: 100 258, 244;                            130 264, 281
//   d 512, f 1024, E 128, V 128: 120 164, 156;                    140 176, 175
//   d 512, f 1024, E 128, V 160: 160 195, 181;                    220 216, 223
//   d 256, E 128, V 128: 120 114, 112;                            150 119, 123
// Training steps cross a little later (d 2048, E 64, V 96: 100 4314, 3931; 130 4402, 4449; 160 4900, 4941).
//
// And 64-row tiles for any number of rows per expert while the wider product does not fill 224 of the 256 x 256 tiles (a
// tile per compute unit: most of the chip waits for a few long tiles, and for half-empty ones); fewer where the shorter contraction is
// below 432, because a small tile's epilogue and first loads weigh more.  4 experts, f = 4 d unless given, forward and training:
//   d 2048: 1800 rows 323, 252 and 819, 647;             past the line: 2400 328, 342 and 860, 848
//   d 1024: 3600 177, 139 and 459, 379;                                 4400 183, 176 and 522, 515; 5600 187, 201 and 549, 586
//   d 512:  7200 98, 94 and 297, 286;                                   8800 113, 117 and 337, 345
//   d 256:                                                              11200 72, 69 and 206, 197; 16800 83, 87 and 253, 258
//   d 128:  11200 54, 55 and 161, 158;                                  22400 58, 61 and 177, 178; 28800 59, 66 and 187, 199
//   d 64, f 256: 24000 62, 57 and 173, 158 (94 tiles);                  44000 68, 72 and 193, 203
//
// 32-row tiles up to four rows per expert: both products, 32- and 64-row tiles, 1 row (16 tokens, d 1024, E 32, k 2) 59, 69;
// 8 rows (256 tokens, d 2048, E 64, k 2) 610, 562.
constexpr int kSmall32Rows = 4;
// The largest number of rows that takes them (every smaller one does, too):
static int small_rows_most(int d, int f, int E, int V) {
  const long long wide = std::max(d, f), few = std::min(d, f);
  if (wide >= 1 << 24) return 0;                          // 32-bit byte offsets of the weight loads: 128 rows of that many columns
  const long long matrix = (long long)d * f, tenths = matrix >= 1 << 23 ? 14 : matrix >= 1 << 20 ? 17 : 24;
  const long long by_tiles = tenths * V * 64 / 10 - 32ll * E;
  const long long by_outputs = std::min(224ll, 64 + 3 * few / 8) * BM * BN / wide;
  return (int)std::min(std::max(by_tiles, by_outputs), ((1ll << 30) - 1) / wide);      // 32-bit byte offsets of the row loads
}
static int small_rows(int A, int d, int f, int E, int V) {
  return A > small_rows_most(d, f, E, V) ? 0 : A <= kSmall32Rows * E ? 32 : 64;
}
// Whether dXp and the weight gradients share a launch: both take the small tiles, dXp's tiles fit the two workgroups per compute unit
// that the launch has, and the weight gradients are few enough that a third workgroup per compute unit, which the launch's
// larger LDS rules out, counts less than the tail of dXp and the launch saved.  Whole backward passes, us, launches of their own and one:
// d 128, f 512, E 16, 1536 rows 47, 34; d 256, f 1024, E 8, 2048 rows 62, 50, 8000 rows 85, 79; d 256, f 256, E 4, 11000 rows (352 tiles) 50, 48; d 128, f 256, E 3,
// 25400 rows (400) 67, 65; d 448, f 1216, E 18, 6000 rows (448) 84, 78; d 512, f 2048, E 32, 1024 rows 89, 82; d 768, f 3072, E 16, 1536 rows 114, 106, 4096
// rows (480) 224, 221; d 1024, f 2048, E 8, 2048 rows 100, 96; the ratio over 120 layers inside the lines 0.75 - 0.98.
// Past the lines: d 1024, f 2048, E 8, 5120 rows (704 tiles) 191, 193; d 512, f 1024, E 128 (8192
// tiles of weight gradients), 4096 rows 219, 224; d 1024, f 4096, E 32 (16384), 1024 rows 284, 294; d 2048, f 8192, E 64, 2048 rows 1835, 1951.
static bool bwd_products_merged(const FfnArgs& a) {
  if (!small_rows(a.A, a.d, a.f, a.E, a.V) || !wgrad_small(a.A, a.d, a.f, a.E)) return false;
  const long long d_tiles = (a.d + GT - 1) / GT, f_tiles = (a.f + GT - 1) / GT;
  return (a.A / 64 + a.E) * d_tiles <= kSmallSplitTarget && 2 * a.E * d_tiles * f_tiles <= 6144;
}

// Partial tiles that a product with contraction K and NC columns can leave at most (see small_segments): none for short
// contractions.
static long long small_slots(int A, int E, int bm, int K, int NC) {
  const int most = small_segments(1, (K + SK - 1) / SK);
  return most == 1 ? 0 : std::min<long long>(kSmallSlots, (long long)(A / bm + E) * ((NC + SN - 1) / SN) * most);
}
// Their workspace: row tiles (room for tiles of 32 rows, so that the size does not fall at the line to 64), row list,
// counters, partial tiles.
static size_t small_tab_bytes(int A, int E) { return align_up((size_t)(A / 32 + E + 1) * sizeof(i32x4), 256); }
static size_t small_ws_bytes(int A, int d, int f, int E, int V) {
  const int bm = small_rows(A, d, f, E, V);
  if (!bm) return 0;
  return small_tab_bytes(A, E) + align_up((size_t)A * sizeof(int32_t), 256) + align_up(kSmallSlots * sizeof(int), 256) +
         (size_t)std::max(small_slots(A, E, bm, d, f), small_slots(A, E, bm, f, d)) * bm * SN * sizeof(float);
}
// What the rows products of a call take: either the partial tiles of a split last round and the table of 256-row tiles, or the
// above.  Past the small kernels' line still what they take at the line: the size never falls where A grows.
static size_t rows_ws_bytes(int A, int d, int f, int E, int V) {
  const size_t small = small_ws_bytes(std::min(A, small_rows_most(d, f, E, V)), d, f, E, V);
  if (small_rows(A, d, f, E, V)) return small;
  return std::max(small, rows_split_bytes(A, V, f, d) + align_up(rows_tab_bytes(max_row_tiles(A, V)), 256));      // (GEMM2 and dXp are split)
}

// The workspace, in this order: dHpre (or H in a forward pass); H; the partial tiles of dW2, then of dW1; the weight
// gradients' work lists; what the rows products take.
size_t ffn_ws_bytes(int A, int d, int f, int E, int V, int dtype) {
  const size_t s = dtype == FLEXMOE_BF16 ? 2 : 4;
  size_t need = align_up((size_t)A * f * s, 256) * 2;
  if (dtype == FLEXMOE_BF16)
    need += 2 * wgrad_tail_bytes(A, d, f, V) + wgrad_plan_reserved(A, d, f, E, V) + rows_ws_bytes(A, d, f, E, V);
  return need;
}
static void* wgrad_plan_ws(const FfnArgs& a, void* ws) {
  return (char*)ws + 2 * align_up((size_t)a.A * a.f * sizeof(bf16_t), 256) + 2 * wgrad_tail_bytes(a.A, a.d, a.f, a.V);
}
static void* rows_ws(const FfnArgs& a, void* ws) { return (char*)wgrad_plan_ws(a, ws) + wgrad_plan_reserved(a.A, a.d, a.f, a.E, a.V); }
// of the 256 x 256 kernels: partial tiles of the split last round, row-tile table
static void* rows_split_ws(const FfnArgs& a, void* ws) { return rows_ws(a, ws); }
static i32x4* rows_tab_ws(const FfnArgs& a, void* ws) { return (i32x4*)((char*)rows_ws(a, ws) + rows_split_bytes(a.A, a.V, a.f, a.d)); }
// of the small ones
static int small_plan_parts(const FfnArgs& a) { return std::max(1, std::min(a.A / (a.V * 512), 2048 / a.V)); }      // waves per bucket, up to 512 workgroups
static SmallPlan small_plan_ws(const FfnArgs& a, void* ws, float** partial = nullptr) {
  SmallPlan pl;
  pl.bm = small_rows(a.A, a.d, a.f, a.E, a.V);
  pl.parts = small_plan_parts(a);
  char* at = (char*)rows_ws(a, ws);
  pl.tab = (i32x4*)at;
  at += small_tab_bytes(a.A, a.E);
  pl.rowmap = (int32_t*)at;
  at += align_up((size_t)a.A * sizeof(int32_t), 256);
  pl.counters = (int*)at;
  at += align_up(kSmallSlots * sizeof(int), 256);
  if (partial) *partial = (float*)at;
  return pl;
}
static int plan_blocks(const FfnArgs& a) {
  if (small_rows(a.A, a.d, a.f, a.E, a.V)) return 1 + (a.V * small_plan_parts(a) + 3) / 4;      // the first: row tiles; the others: the row list
  return std::max(1, std::min(64, (max_row_tiles(a.A, a.V) + kGemmThreads - 1) / kGemmThreads));
}
// What the rows kernels of one forward call look up: the row-tile table of the persistent kernels, or the small kernels'
// row list.
static void launch_rows_plan(const FfnArgs& a, void* ws, hipStream_t s) {
  const SmallPlan small = small_plan_ws(a, ws);
  if (small.bm) hipLaunchKernelGGL(small_plan_kernel, dim3(plan_blocks(a)), dim3(kGemmThreads), 0, s, a.voff, a.owner, a.E, a.V, small);
  else hipLaunchKernelGGL(rows_plan_kernel, dim3(plan_blocks(a)), dim3(kGemmThreads), 0, s, a.voff, a.owner, a.V, rows_tab_ws(a, ws));
}

template <bool WT, int EPI, bool EVAL>
static void launch_small_t(int bm, const SmallArgs& p, unsigned grid, hipStream_t s) {
  if (bm == 32) hipLaunchKernelGGL((rows_gemm_small_bf16<32, WT, EPI, EVAL>), dim3(grid), dim3(kSmallThreads), 0, s, p);
  else hipLaunchKernelGGL((rows_gemm_small_bf16<64, WT, EPI, EVAL>), dim3(grid), dim3(kSmallThreads), 0, s, p);
}
template <int EPI>
static SmallArgs small_args(const FfnArgs& a, const void* in, const void* w, const void* bias, int K, int NC, const void* hpre_in,
                            void* out0, void* out1, void* ws, const int32_t* gsrc, int gk, const int32_t* scatter_rows, int* bm,
                            unsigned* grid) {
  float* partial;
  const SmallPlan pl = small_plan_ws(a, ws, &partial);
  // The table as in the 256 x 256 kernels: where the contraction is whole 128-wide rounds.  Otherwise the activation is
  // evaluated: the table has 2^-24 for every smaller magnitude, zero included, and a negative NaN is lost in it.
  const bool gelu = EPI != EPI_PLAIN && a.act != FLEXMOE_RELU;
  const int lut = !gelu || K % 128 ? -1 : a.act == FLEXMOE_GELU_ERF ? 0 : 1;
  const SmallArgs p{(const bf16_t*)in, (const bf16_t*)w, (const bf16_t*)bias, pl.tab, pl.rowmap, K, NC, (NC + SN - 1) / SN,
                    (const bf16_t*)hpre_in, (bf16_t*)out0, (bf16_t*)out1, gsrc, gk, scatter_rows, a.act, lut, partial, pl.counters};
  // two workgroups per compute unit walk the tiles
  const long long most = (long long)(a.A / pl.bm + a.E) * p.col_tiles;
  *grid = (unsigned)std::min<long long>(kSmallSplitTarget, std::max<long long>(most * kSmallSplitMax, 1));
  *bm = pl.bm;
  return p;
}
template <bool WT, int EPI>
static hipError_t launch_small(const FfnArgs& a, const void* in, const void* w, const void* bias, int K, int NC,
                               const void* hpre_in, void* out0, void* out1, void* ws, hipStream_t s, const int32_t* gsrc,
                               int gk, const int32_t* scatter_rows) {
  int bm;
  unsigned grid;
  const SmallArgs p = small_args<EPI>(a, in, w, bias, K, NC, hpre_in, out0, out1, ws, gsrc, gk, scatter_rows, &bm, &grid);
  if constexpr (EPI != EPI_PLAIN) {
    if (a.act != FLEXMOE_RELU && p.lut < 0) {
      launch_small_t<WT, EPI, true>(bm, p, grid, s);
      return hipGetLastError();
    }
  }
  launch_small_t<WT, EPI, false>(bm, p, grid, s);
  return hipGetLastError();
}

static RowsDmaArgs rows_dma_args(const FfnArgs& a, const void* in, const void* w, const void* bias, int K, int NC,
                                 const void* hpre_in, void* out0, void* out1, const int32_t* gsrc, int gk) {
  return RowsDmaArgs{(const bf16_t*)in, (const bf16_t*)w, (const bf16_t*)bias, a.voff, a.owner, a.V, K, NC,
                     max_row_tiles(a.A, a.V), (NC + BN - 1) / BN, (const bf16_t*)hpre_in, (bf16_t*)out0,
                     (bf16_t*)out1, gsrc, gk, nullptr, 0u, nullptr};
}

template <bool WT, int EPI, int ACT>
static hipError_t launch_rows_t(const FfnArgs& a, const void* in, const void* w, const void* bias, int K, int NC,
                                const void* hpre_in, void* out0, void* out1, hipStream_t s, const int32_t* gsrc, int gk,
                                void* split_ws, const int32_t* scatter_rows, const i32x4* row_tab) {
  const int col_tiles = (NC + BN - 1) / BN;
  const int row_tiles = max_row_tiles(a.A, a.V);
  const unsigned grid = patched_grid(row_tiles, col_tiles);
  if (K % 128 == 0) {
    // K is a whole number of pipeline rounds: direct-to-LDS path, one persistent workgroup per compute unit
    RowsDmaArgs p = rows_dma_args(a, in, w, bias, K, NC, hpre_in, out0, out1, gsrc, gk);
    p.scatter_rows = scatter_rows;
    const unsigned persist = std::min(grid, (unsigned)kComputeUnits);
    if (EPI == EPI_PLAIN && split_ws && rows_split_bytes(a.A, a.V, K, NC)) {
      // the last, partly filled round of tiles is cut along K, then the partial tiles are summed
      p.split_partial = (float*)split_ws;
      p.normal_grid = grid;
      hipLaunchKernelGGL((rows_gemm_persist_bf16<WT, EPI, ACT, false>), dim3(persist), dim3(kDmaThreads), 0, s, p, row_tab);
      hipLaunchKernelGGL(rows_split_reduce_kernel, dim3(kSplitSlices, kSplitUnits / 2), dim3(kGemmThreads), 0, s, p);      // up to 128 tail tiles (two segments each)
      return hipGetLastError();
    }
    if constexpr (!WT && EPI == EPI_FWD1) {
      if (gsrc) {
        hipLaunchKernelGGL((rows_gemm_persist_bf16<WT, EPI, ACT, true>), dim3(persist), dim3(kDmaThreads), 0, s, p, row_tab);
        return hipGetLastError();
      }
    }
    hipLaunchKernelGGL((rows_gemm_persist_bf16<WT, EPI, ACT, false>), dim3(persist), dim3(kDmaThreads), 0, s, p, row_tab);
    return hipGetLastError();
  }
  if (gsrc || scatter_rows) return hipErrorInvalidValue;   // gathered / scattered rows only on the direct-to-LDS path (host check upstream)
  hipLaunchKernelGGL((rows_gemm_bf16<WT, EPI, ACT>), dim3(grid), dim3(kGemmThreads), 0, s, (const bf16_t*)in,
                     (const bf16_t*)w, (const bf16_t*)bias, a.voff, a.owner, a.V, K, NC, row_tiles, col_tiles,
                     (const bf16_t*)hpre_in, (bf16_t*)out0, (bf16_t*)out1);
  return hipGetLastError();
}

template <bool WT, int EPI>
static hipError_t launch_rows(const FfnArgs& a, const void* in, const void* w, const void* bias, int K, int NC,
                              const void* hpre_in, void* out0, void* out1, void* ws, hipStream_t s,
                              const int32_t* gsrc = nullptr, int gk = 1, void* split_ws = nullptr,
                              const int32_t* scatter_rows = nullptr) {
  if (small_rows(a.A, a.d, a.f, a.E, a.V)) return launch_small<WT, EPI>(a, in, w, bias, K, NC, hpre_in, out0, out1, ws, s, gsrc, gk, scatter_rows);
  const i32x4* tab = rows_tab_ws(a, ws);
  if (EPI == EPI_PLAIN)
    return launch_rows_t<WT, EPI, FLEXMOE_RELU>(a, in, w, bias, K, NC, hpre_in, out0, out1, s, gsrc, gk, split_ws,
                                                scatter_rows, tab);
  switch (a.act) {
    case FLEXMOE_RELU:
      return launch_rows_t<WT, EPI, FLEXMOE_RELU>(a, in, w, bias, K, NC, hpre_in, out0, out1, s, gsrc, gk, nullptr, nullptr, tab);
    case FLEXMOE_GELU_ERF:
      return launch_rows_t<WT, EPI, FLEXMOE_GELU_ERF>(a, in, w, bias, K, NC, hpre_in, out0, out1, s, gsrc, gk, nullptr, nullptr, tab);
    default:
      return launch_rows_t<WT, EPI, FLEXMOE_GELU_TANH>(a, in, w, bias, K, NC, hpre_in, out0, out1, s, gsrc, gk, nullptr, nullptr, tab);
  }
}

// One weight-gradient product's arguments and grid; `ws_tail` holds its job table and fp32 partial
// tiles when the contraction is cut into segments (wgrad_tail_bytes each).
// product: 0 = dW2 (M = f, NC = d), 1 = dW1 (M = d, NC = f): which of the plan's two work lists it reads.
static WgradDmaArgs wgrad_dma_args(const FfnArgs& a, const void* L, const void* R, int M, int NC, void* dw,
                                   void* ws_tail, void* ws, unsigned* grid, int product) {
  const int edge = wgrad_small(a.A, a.d, a.f, a.E) ? GT : BM;
  const int m_tiles = (M + edge - 1) / edge, n_tiles = (NC + edge - 1) / edge;
  const int seg_tiles = wgrad_seg_tiles(a.A, a.d, a.f);
  float* partial = seg_tiles ? (float*)ws_tail : nullptr;
  const int seg_rows_max = wgrad_seg_rows_max(a.A, a.d, a.f, a.E, a.V);
  *grid = patched_grid(seg_rows_max * m_tiles, n_tiles);
  return WgradDmaArgs{(const bf16_t*)L, (const bf16_t*)R, a.voff, a.owner, a.E, a.V, M, NC, m_tiles, n_tiles,
                      seg_tiles, seg_rows_max, partial, wgrad_plan_at(wgrad_plan_ws(a, ws), seg_rows_max, a.E, a.V, product),
                      (bf16_t*)dw};
}

// How the work lists of dW2 and dW1 are balanced (only the persistent kernels skip the holes that balancing leaves in a list).
static void wgrad_balance(const FfnArgs& a, WgradBalance* geo) {
  const int f_tiles = (a.f + BM - 1) / BM, d_tiles = (a.d + BM - 1) / BM;
  const bool whole = a.f % BM == 0 && a.d % BN == 0 && !wgrad_small(a.A, a.d, a.f, a.E);
  geo[0] = whole ? wgrad_balance_geometry(f_tiles, d_tiles) : WgradBalance{1, 1};
  geo[1] = whole ? wgrad_balance_geometry(d_tiles, f_tiles) : WgradBalance{1, 1};
}

// The work list both weight-gradient products of a backward call read and (with tokens) the row-tile table
// of its rows products: one small launch.
static void launch_bwd_plan(const FfnArgs& a, void* ws, hipStream_t s) {
  const int seg_rows_max = wgrad_seg_rows_max(a.A, a.d, a.f, a.E, a.V);
  const int row_blocks = a.A > 0 ? plan_blocks(a) : 0;
  WgradBalance geo[2];
  wgrad_balance(a, geo);
  hipLaunchKernelGGL(ffn_bwd_plan_kernel, dim3(1 + row_blocks), dim3(kGemmThreads), 0, s, a.voff, a.owner, a.E, a.V,
                     wgrad_seg_tiles(a.A, a.d, a.f), seg_rows_max,
                     wgrad_plan_at(wgrad_plan_ws(a, ws), seg_rows_max, a.E, a.V, 0),
                     geo[0], geo[1], rows_tab_ws(a, ws), small_plan_ws(a, ws));
}

// Sums of the partial tiles of `n` products (their [M, NC] have the same number of elements).
static void launch_wgrad_reduce(const FfnArgs& a, const WgradDmaArgs* g, int n, hipStream_t s) {
  if (!g->seg_tiles) return;
  const size_t elems = (size_t)g->M * g->NC;
  const int blocks = (int)std::min<size_t>((elems / 4 + kGemmThreads - 1) / kGemmThreads, 2048);
  const WgradReduceArgs r{(const int4*)g->plan.table, {{g[0].partial, g[0].dw}, {g[n - 1].partial, g[n - 1].dw}}};
  hipLaunchKernelGGL(wgrad_reduce_kernel, dim3(blocks, a.E, n), dim3(kGemmThreads), 0, s, r, elems);
}

static bool overlap(const void* p, const void* q, size_t bytes_p, size_t bytes_q) {
  return (uintptr_t)p < (uintptr_t)q + bytes_q && (uintptr_t)q < (uintptr_t)p + bytes_p;
}

// dXp = dHpre . W1^T (W1_e is [d, f], contraction index f contiguous), dW2 = H^T . dYp, dW1 = Xp^T . dHpre: the weight gradients
// each with its own partial tiles.  In this order, so that a caller who needs w1, h or dyp no longer may have a gradient written over
// them: products that share a launch only do where the later one's output is nothing that the earlier one reads.
static hipError_t launch_bwd_products(const FfnArgs& a, const void* h, const void* dyp, void* dw2, const void* xp, const void* dhpre,
                                      void* dw1, const void* w1, void* dxp, const int32_t* scatter_src, void* ws, hipStream_t s) {
  void* tail2 = (char*)ws + 2 * align_up((size_t)a.A * a.f * sizeof(bf16_t), 256);
  void* tail1 = (char*)tail2 + wgrad_tail_bytes(a.A, a.d, a.f, a.V);
  unsigned grid[2];
  const WgradDmaArgs g[2] = {wgrad_dma_args(a, h, dyp, a.f, a.d, dw2, tail2, ws, &grid[0], 0),
                             wgrad_dma_args(a, xp, dhpre, a.d, a.f, dw1, tail1, ws, &grid[1], 1)};
  const size_t w_bytes = (size_t)a.E * a.d * a.f * sizeof(bf16_t), row_bytes = (size_t)a.A * sizeof(bf16_t);
  const bool joint = wgrad_joint(grid[0], grid[1]) && !overlap(dw1, h, w_bytes, row_bytes * a.f) && !overlap(dw1, dyp, w_bytes, row_bytes * a.d);
  const WgradSmallArgs both{{g[0], g[1]}, grid[0]};
  if (a.A > 0 && joint && bwd_products_merged(a) && !overlap(dw1, w1, w_bytes, w_bytes) && !overlap(dw2, w1, w_bytes, w_bytes)) {
    int bm;
    unsigned rows_grid;
    const SmallArgs p = small_args<EPI_PLAIN>(a, dhpre, w1, nullptr, a.f, a.d, nullptr, dxp, nullptr, ws, nullptr, 1, scatter_src, &bm, &rows_grid);
    rows_grid = (rows_grid + kXcds - 1) / kXcds * kXcds;
    const dim3 blocks(rows_grid + grid[0] + grid[1]);
    if (bm == 32) hipLaunchKernelGGL(bwd_products_small_bf16<32>, blocks, dim3(kGradThreads), 0, s, p, both, rows_grid);
    else hipLaunchKernelGGL(bwd_products_small_bf16<64>, blocks, dim3(kGradThreads), 0, s, p, both, rows_grid);
    launch_wgrad_reduce(a, g, 2, s);
    return hipGetLastError();
  }
  if (a.A > 0) {
    const hipError_t err = launch_rows<true, EPI_PLAIN>(a, dhpre, w1, nullptr, a.f, a.d, nullptr, dxp, nullptr, ws, s, nullptr, 1,
                                                        rows_split_ws(a, ws), scatter_src);
    if (err != hipSuccess) return err;
  }
  if (wgrad_small(a.A, a.d, a.f, a.E)) {
    if (joint) {
      hipLaunchKernelGGL(wgrad_gemm_small_bf16, dim3(grid[0] + grid[1]), dim3(kGradThreads), 0, s, both);
    } else {
      for (int i = 0; i < 2; ++i)
        hipLaunchKernelGGL(wgrad_gemm_small_bf16, dim3(grid[i]), dim3(kGradThreads), 0, s, WgradSmallArgs{{g[i], g[i]}, grid[i]});
    }
    launch_wgrad_reduce(a, g, 2, s);
    return hipGetLastError();
  }
  // (One launch for dXp, dW2 and dW1, which filled the partly empty last rounds of the three grids of 256 x 256 tiles, was measured
  // against three persistent launches: the latter are 2 % faster on the GPT-medium-like backward pass and 4.5 % on the Swin-like one.)
  for (int i = 0; i < 2; ++i) {
    if (a.f % BM == 0 && a.d % BN == 0)      // whole output tiles: one persistent workgroup per compute unit
      hipLaunchKernelGGL(wgrad_gemm_persist_bf16, dim3(std::min(grid[i], (unsigned)kComputeUnits)), dim3(kDmaThreads), 0, s, g[i]);
    else
      hipLaunchKernelGGL(wgrad_gemm_dma_bf16, dim3(grid[i]), dim3(kDmaThreads), 0, s, g[i]);
    launch_wgrad_reduce(a, &g[i], 1, s);
  }
  return hipGetLastError();
}

// h_keep (all forward variants): where act(Hpre) goes -- the caller's buffer, kept for the backward pass -- or
// null: the workspace.
hipError_t launch_ffn_fwd_bf16(const FfnArgs& a, const void* xp, const void* w1, const void* b1, const void* w2,
                               const void* b2, void* hpre, void* h_keep, void* yp, void* ws, hipStream_t s) {
  if (a.A == 0) return hipSuccess;
  launch_rows_plan(a, ws, s);
  void* h = h_keep ? h_keep : ws;
  hipError_t err = launch_rows<false, EPI_FWD1>(a, xp, w1, b1, a.d, a.f, nullptr, hpre, h, ws, s);
  if (err != hipSuccess) return err;
  return launch_rows<false, EPI_PLAIN>(a, h, w2, b2, a.f, a.d, nullptr, yp, nullptr, ws, s, nullptr, 1, rows_split_ws(a, ws));
}

// Forward with the expert-wise layout transformation folded into GEMM1's row loads: bucket row p
// is row src[p] / k of x.  d must be a multiple of 128 (direct-to-LDS path).
hipError_t launch_ffn_fwd_gather_bf16(const FfnArgs& a, const void* x, const int32_t* src, int k, const void* w1,
                                      const void* b1, const void* w2, const void* b2, void* hpre, void* h_keep, void* yp,
                                      void* ws, hipStream_t s) {
  if (a.A == 0) return hipSuccess;
  launch_rows_plan(a, ws, s);
  void* h = h_keep ? h_keep : ws;
  hipError_t err = launch_rows<false, EPI_FWD1>(a, x, w1, b1, a.d, a.f, nullptr, hpre, h, ws, s, src, k);
  if (err != hipSuccess) return err;
  return launch_rows<false, EPI_PLAIN>(a, h, w2, b2, a.f, a.d, nullptr, yp, nullptr, ws, s, nullptr, 1, rows_split_ws(a, ws));
}

// The expert path of a top-1 layer without Xp and Yp: rows gathered through src on load (as above)
// and the second product's rows stored straight to y[src[p], :] -- with one expert per token the gate
// weight is exactly 1, so this is flexmoe_combine folded into the epilogue.  d and f multiples of 128.
hipError_t launch_ffn_fwd_top1_bf16(const FfnArgs& a, const void* x, const int32_t* src, const void* w1, const void* b1,
                                    const void* w2, const void* b2, void* hpre, void* h_keep, void* y, void* ws,
                                    hipStream_t s) {
  if (a.A == 0) return hipSuccess;
  launch_rows_plan(a, ws, s);
  void* h = h_keep ? h_keep : ws;
  hipError_t err = launch_rows<false, EPI_FWD1>(a, x, w1, b1, a.d, a.f, nullptr, hpre, h, ws, s, src, 1);
  if (err != hipSuccess) return err;
  return launch_rows<false, EPI_PLAIN>(a, h, w2, b2, a.f, a.d, nullptr, y, nullptr, ws, s, nullptr, 1, rows_split_ws(a, ws), src);
}

// scatter_src (top-1 layers, needs f % 128 == 0): bucket row p of dXp is stored as row scatter_src[p] of
// `dxp`, which is then dX [N, d] itself -- the backward reverse routing folded into the epilogue.
// h_kept: act(Hpre) as the forward pass left it in the caller's buffer, or null: it is computed again from
// hpre by the dH kernel (into the workspace), which then stores two [A, f] tensors instead of one.
hipError_t launch_ffn_bwd_bf16(const FfnArgs& a, const void* dyp, const void* xp, const void* hpre, const void* h_kept,
                               const void* w1, const void* w2, void* dxp, void* dw1, void* dw2, void* ws, hipStream_t s,
                               const int32_t* scatter_src) {
  bf16_t* dhpre = (bf16_t*)ws;
  bf16_t* h_ws = (bf16_t*)((char*)ws + align_up((size_t)a.A * a.f * sizeof(bf16_t), 256));
  const bf16_t* h = h_kept ? (const bf16_t*)h_kept : h_ws;
  hipError_t err;
  launch_bwd_plan(a, ws, s);
  if (a.A > 0) {
    // dH = dYp . W2^T fused with act'(Hpre); W2_e is [f, d], contraction index d contiguous
    err = h_kept ? launch_rows<true, EPI_DHQ>(a, dyp, w2, nullptr, a.d, a.f, hpre, dhpre, nullptr, ws, s)
                 : launch_rows<true, EPI_DH>(a, dyp, w2, nullptr, a.d, a.f, hpre, dhpre, h_ws, ws, s);
    if (err != hipSuccess) return err;
  }
  return launch_bwd_products(a, h, dyp, dw2, xp, dhpre, dw1, w1, dxp, scatter_src, ws, s);
}

}  // namespace flexmoe

// For tests: which kernels a bf16 call of these sizes takes (operands that do not overlap).  out[0] row tiles of the few-rows kernels
// (0: the 256 x 256 ones); [1] weight gradients on 128 x 128 tiles; [2] both in one launch; [3] dXp in that launch, too; [4] K tiles of a
// segment (0: no cutting); [5], [6] bins over which dW2's and dW1's work lists are dealt out (1: not balanced); [7] most threads of
// one weight-gradient launch.
extern "C" void flexmoe_debug_bf16_paths(int A, int d, int f, int E, int V, long long* out) {
  using namespace flexmoe;
  const FfnArgs a{A, d, f, E, V, FLEXMOE_RELU, nullptr, nullptr};
  const bool small = wgrad_small(A, d, f, E);
  unsigned grid[2];
  wgrad_dma_args(a, nullptr, nullptr, f, d, nullptr, nullptr, nullptr, &grid[0], 0);
  wgrad_dma_args(a, nullptr, nullptr, d, f, nullptr, nullptr, nullptr, &grid[1], 1);
  const bool joint = small && wgrad_joint(grid[0], grid[1]);
  WgradBalance geo[2];
  wgrad_balance(a, geo);
  out[0] = small_rows(A, d, f, E, V);
  out[1] = small;
  out[2] = joint;
  out[3] = A > 0 && joint && bwd_products_merged(a);
  out[4] = wgrad_seg_tiles(A, d, f);
  for (int i = 0; i < 2; ++i) out[5 + i] = geo[i].groups * geo[i].per_slot;
  out[7] = (joint ? (long long)grid[0] + grid[1] : std::max(grid[0], grid[1])) * (small ? kGradThreads : kDmaThreads);
}

#ifdef FLEXMOE_TILE_PHASES
// Profiling build only: copies the per-workgroup phase counters of the persistent GEMM kernels (5 x 256 x 4 uint64,
// see TilePhases) to host memory.
extern "C" int flexmoe_debug_tile_phases(unsigned long long* host_out) {
  return (int)hipMemcpyFromSymbol(host_out, HIP_SYMBOL(flexmoe::g_tile_phases), sizeof(flexmoe::g_tile_phases));
}
#endif
