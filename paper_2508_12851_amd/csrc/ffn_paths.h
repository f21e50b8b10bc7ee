// Which tile path serves a bf16 expert FFN, by the sizes the host knows (no HIP in here: the rules run
// and are tested on the CPU).
#ifndef PRISM_FFN_PATHS_H_
#define PRISM_FFN_PATHS_H_

#include <stddef.h>

#include "prism.h"

namespace prism {

constexpr int kDecodeMaxTokens = 64;    // batches up to this size take the decode tiles
constexpr int kStreamMaxTokens = 512;   // wide bf16 layers: batches up to this size split the down projection as those do,
constexpr int kMidMaxTokens = 256;      // up to this one in 128 x 128 tiles with non-temporal weight loads,
constexpr int kSquareMaxTokens = 448;   // up to this one in 128 x 128 tiles if the hidden size is 1025 to 2560 (ffn_path)

static inline size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }
static inline int ceil_div(int a, int b) { return (a + b - 1) / b; }

// Partial tiles of a down projection whose last round of work items is cut along the contraction:
// one tile per workgroup.  Prefill batches of layers whose contraction is long enough for the cut
// to pay: an item of K / 32 k-tiles takes about 0.74 us per k-tile, the cut saves at least half of
// one item per launch and costs two short launches plus up to 64 MB of fp32 tiles written and read
// (about 40 us); with fewer than 128 k-tiles (the gate/up GEMM of the same layers included, whose
// contraction is H) it was measured to lose.
constexpr int kSliceMinFfn = 4096;
// Smaller batches of such layers are not cut.  (Up to kStreamMaxTokens most of these layers split the
// whole down projection instead; those with too many row tiles for that, 16 experts of 4096 columns at
// 400 tokens for instance, run in prefill tiles and are cut from here on.)
constexpr int kSliceMinTokens = 353;
static inline bool slicing_shape(const prism_layer_desc& d) {
  return d.dtype == PRISM_BF16 && d.ffn >= kSliceMinFfn && d.hidden >= 128;
}
static inline bool down_slicing_applies(const prism_layer_desc& d, int T) {
  return slicing_shape(d) && T >= kSliceMinTokens;
}

// Work items of the down projection in prefill tiles: column tiles x row tiles, the latter estimated
// from what the host knows (half of the experts hosted, rows spread evenly).
static inline int prefill_down_items(const prism_layer_desc& d, int T) {
  const int row_tiles = ceil_div(T * d.top_k, 256) + d.n_experts / 2 + d.n_shared * ceil_div(T, 256);
  return row_tiles * ceil_div(d.hidden, 256);
}

// Batches between the decode and the prefill sizes whose down projection in prefill tiles would
// have too few items for the machine.  Layers of many small experts have enough at any batch size.
static inline bool stream_tiles_apply(const prism_layer_desc& d, int T) {
  if (T <= kDecodeMaxTokens || T > kStreamMaxTokens || d.hidden < 256 || d.ffn < 1024) return false;
  return prefill_down_items(d, T) <= 128;
}

// Rows per expert: what an even spread of the picks over all experts would give, all the host knows.
// Layers whose down projection may cut its last round keep the prefill tiles, which the cut fills better.
constexpr int kFewRows = 112;            // most rows per expert of the 128-row tiles ...
constexpr int kFewRowsFewItems = 144;    // ... if prefill tiles would leave compute units without an item
constexpr int kFewRowsOnePick = 2560;    // most rows of a batch of one pick per token in them
constexpr int kVeryFewRows = 16;         // most rows per expert of the 64-row tiles
constexpr int kVeryFewTokens = 1024;     // most tokens in them: an expert has at most that many rows
static inline bool few_rows_per_expert(const prism_layer_desc& d, int T) {
  if (T <= kDecodeMaxTokens || d.hidden < 192 || d.ffn < 192 || slicing_shape(d)) return false;
  if (d.top_k == 1 && T > kFewRowsOnePick) return false;
  const int most = prefill_down_items(d, T) <= 256 ? kFewRowsFewItems : kFewRows;
  return (long long)T * d.top_k <= (long long)most * d.n_experts;
}

enum class FfnPath {
  kDecodeTiled,    // 64 x 128 tiles, 32-wide k-tiles; contraction of the down projection split
  kDecode,         // 64 x 128, 64-wide k-tiles; split
  kDecodeShort,    // the same with a short ring, for short contractions
  kStream,         // 128 x 128, weights non-temporal, items dealt to the XCDs one by one, or 128 x 256 in lists (the device chooses); split
  kSplitSquare,    // 128 x 128; split
  kSplitWide,      // 128 x 256; split
  kFewRows64,      // 64 x 128, weights non-temporal
  kFewRows128,     // gate/up 128 x 256, down 128 x 128
  kPrefill,        // 256 x 256
  kPrefillShort    // the same with a short ring
};

// The path of a batch of T > 0 tokens of layer d (bf16).
static inline FfnPath ffn_path(const prism_layer_desc& d, int T) {
  if (T <= kDecodeMaxTokens) {
    // Decode batch: every expert has at most 64 rows, the layer is bound by streaming
    // the weights once.  Small tiles make ~1000 work items; the down projection also
    // splits its contraction (the slices are summed by a last kernel or by the combine).
    // No weight tile is shared between workgroups here, so every item starts its
    // contraction at a different k-tile: at any moment the workgroups then read
    // different column ranges of the weight rows, whose power-of-two pitch would
    // otherwise send them all to the same few memory channels.
    // Tiled weights: 32-wide k-tiles, so that one load instruction takes one whole 1 KiB
    // tile (with 64-wide k-tiles it would take halves of two), and twice the stages.
    // An expert has one row tile here, so every weight element is read by exactly one
    // workgroup, once: the weight loads are marked non-temporal (grouped_gemm.h, STREAM_B).
    if (d.weight_layout == PRISM_WEIGHTS_TILED && d.hidden >= 256 && d.ffn >= 1024)
      return FfnPath::kDecodeTiled;
    if (d.hidden >= 192 && d.ffn >= 192)
      return FfnPath::kDecode;
    return FfnPath::kDecodeShort;
  }
  // Batches of a few hundred tokens of a wide layer are still bound by streaming the weights
  // once, but an expert now has up to a few hundred rows; the down projection splits its
  // contraction as for decode batches.  64-wide k-tiles take whole 128-byte lines of the
  // activations (and of row-major weights), which 32-wide ones ask the L2 for twice.
  // Up to 256 tokens an expert has one or two row tiles: 128 x 128, dealt item by item and
  // non-temporal, unless some expert has two and 128 x 256 tiles make items enough, which only the
  // device knows (schedule.h, "Two widths"): with one or two of 8 hosted, a layer has fewer wide tiles
  // than the machine has workgroups.  Layer, weights from HBM, 128 x 128 against 128 x 256: 4096 x 14336, 66 tokens, 1 hosted
  // 94 / 128 us; 200 tokens, 1 hosted, evenly spread picks 104 / 143 (the other way with 5 hosted, 412 /
  // 376); 3072 x 8192, 96 tokens, 2 hosted 83 / 101; 2048 x 8192, 66 tokens, 5 hosted 116 / 132, and 131 if
  // dealt in rectangles with temporal loads.  16 shapes, 1 to 8 hosted, against the better of those two for
  // the shape: up to 160 tokens ahead by 6 % on average and up to 27 %, from there to 256 even on average.
  if (stream_tiles_apply(d, T) && T <= kMidMaxTokens) return FfnPath::kStream;
  // Beyond, the row tiles of an expert stand next to each other in an XCD's list, so that the later
  // ones find the weight tile in the L2, and tiles of 128 activation rows x 256 weight rows bring twice
  // the HBM bytes per k-tile for the same waits and barriers as 128 x 128.  4096 x 14336 layer, 5 of 8 experts
  // hosted, tiled weights, against 128 x 256 x 32 tiles up to 352 tokens and prefill tiles from there: 502 -> 419 us
  // at 352, 529 -> 445 at 400, 554 -> 502 at 512.  A padded row tile of 256 costs its loads and MFMAs like
  // a full one: prefill tiles with the cut last round are even at 1024 tokens (between 512 and there: not
  // split here, see kStreamMaxTokens).
  // With few output columns (H up to 2560) the wide tiles make too few items for the machine, in the
  // down projection above all: 128 x 128 there (5 of 8 experts, layer: 1024 x 14336, 300 tokens 143 against 157
  // us; at H = 3072 the wide ones lead, 14336 x 3072, 300 tokens, 194 / 223).  Near 512 tokens popular
  // experts have three and four row tiles, which make items enough: 4 hosted, evenly spread picks,
  // 512 tokens, wide against 128 x 128: 2560 x 7168 179 / 203 us, 1536 x 8192 125 / 144, 2048 x 14336 217 / 247; at
  // 420 tokens the 128 x 128 ones still lead (mean over 1 to 6 hosted 1536 x 8192 -9 %, 2560 x 7168 -5 %), and
  // with H = 1024 at all sizes (4096 wide, 512 tokens: -9 %).
  if (stream_tiles_apply(d, T)) {
    const bool square = d.hidden <= 1024 || (d.hidden <= 2560 && T <= kSquareMaxTokens);
    return square ? FfnPath::kSplitSquare : FfnPath::kSplitWide;
  }
  // Many narrow experts with few rows each.  256-row tiles are mostly padding there, and the narrow
  // layers have items enough without a split.  Time of both GEMMs against the 256 x 256 tiles:
  //   gate/up 128 x 256, down 128 x 128, 64-wide k-tiles: 60 experts, 4 picks, 4 shared, 333 tokens
  //   (22 rows) 172 -> 148 us, 600 tokens 221 -> 179; 256 experts, 8 picks, 800 tokens 173 -> 158; whole
  //   layer, 160 of 256 hosted, 3500 tokens (109 rows) 327 -> 314.  From 120 rows on the two are even or
  //   the full tiles ahead (evenly spread picks, layer: 60 experts, 2150 tokens, 143 rows, 454 against
  //   478 us; 64 experts, 8 hosted, 1300 tokens, 122 rows, 122 against 134) where those make items enough.
  //   In smaller layers the lower tiles win up to 144 rows by their number (314 random layers of 113 to 144
  //   rows, mean time against the full tiles: up to 128 items of the down projection in full tiles -22 %,
  //   129 to 192 -16 %, 193 to 256 -11 %, 257 to 384 -5 % and up to +8 %, beyond 800 -1 % and up to +9 %).
  //   One pick per token is what a peer asks for: all rows are for the hosted experts, however few
  //   they are, and one with hundreds of rows pays for every row tile (8 of 256 experts of 2048 x 1408
  //   hosted, FFN: 2200 rows 94 -> 77 us, 3000 rows 92 -> 100, 4096 rows 100 -> 117).
  //   64 x 128, weights non-temporal, up to 16 rows (an expert has one tile, its weights are read
  //   once): 64 experts, 80 tokens 138 -> 107 us; 256 experts, 100 tokens 108 -> 81, 400 tokens
  //   147 -> 116 (126 in the tiles above).  Shared experts take all tokens and read their weights
  //   once per 64 rows: with 4 of them at 200 tokens the larger tiles are ahead, 128 against 140.  So
  //   do the experts of that peer: 1000 rows 65 us in either, 1500 rows 79 against 62.
  if (few_rows_per_expert(d, T)) {
    if ((long long)T * d.top_k <= (long long)kVeryFewRows * d.n_experts && (long long)T * d.n_shared <= 512 &&
        T <= kVeryFewTokens)
      return FfnPath::kFewRows64;
    return FfnPath::kFewRows128;
  }
  // Prefill batch: 256 x 256 tiles (GEMM1: 128 gate + 128 up weight rows).  Very short
  // contractions (H or F of 64) get the shallowest ring.
  if (d.hidden >= 128 && d.ffn >= 128)
    return FfnPath::kPrefill;
  return FfnPath::kPrefillShort;
}

// Whether the gate/up GEMM of a kPrefill batch reads its tokens from a copy in row order
// (expert_ffn.hip, pack_tokens_kernel).  The copy costs 4 H bytes of traffic per row and a launch; what
// it saves grows with the 4 H F operations of the row's gate/up products.  Layers whose down projection
// may cut its last round, tiled weights: from 2.2e10 elements of rows x H x F on (layer with the copy
// against without: 600 tokens, 2 picks, of 3072 x 6144, 2.3e10, 216 against 231 us; of 1024 x 14336, 1.8e10,
// 184 / 178; of 2048 x 8192, 2.0e10, 192 / 190).  Row-major weights arrive as half lines too, and the GEMM
// waits for those first: from 1.1e11 on (4096 x 14336, all hosted, 560 tokens, 6.6e10, 859 / 799 us, 800 tokens,
// 9.4e10, 934 / 904, 1400 tokens, 1.6e11, 1126 / 1153; 4096 x 4096, 5 hosted, 800 tokens, 2.7e10, 231 / 218).
constexpr size_t kPackTiled = 22000000000, kPackRowMajor = 110000000000;
static inline bool pack_rows_pays(const prism_layer_desc& d, int T) {
  const size_t rows = (size_t)T * (d.top_k + d.n_shared);
  const size_t from = d.weight_layout == PRISM_WEIGHTS_TILED ? kPackTiled : kPackRowMajor;
  // (the places lie behind the rows, in the partial sums' region: four fp32 rows per token and more)
  return slicing_shape(d) && T > kStreamMaxTokens && T <= 512 * d.hidden && rows * d.hidden * d.ffn >= from &&
         align_up(rows, 16) * d.hidden * 2 < 0xFFFF0000ull;
}

}  // namespace prism
#endif  // PRISM_FFN_PATHS_H_
