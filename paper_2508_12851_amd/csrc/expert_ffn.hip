// Grouped SwiGLU expert FFN over the locally hosted and the shared experts
// (paper Sec. III-A: the local expert execution of a server).
//
//   GEMM1  h[r, f] = silu( x[tok(r)] . W_gate^e[f] ) * ( x[tok(r)] . W_up^e[f] )
//   GEMM2  y[r, n] = h[r] . W_down^e[n]
//
// Both are "NT" contractions (activation rows and weight rows are contiguous
// along the contraction index), grouped by expert: device-built work schedules
// list the (row tile, column tile) items of every hosted expert, so the host
// never needs the routing-dependent segment sizes.
//
// bf16 path: the persistent grouped GEMM of grouped_gemm.h
// (v_mfma_f32_32x32x16_bf16, 4 wavefronts per workgroup, operand k-tiles in an
// LDS ring filled by direct-to-LDS loads), in the tile shapes chosen at the end
// of this file.  GEMM1 loads the gate rows and the up rows of the same f range
// into one tile, so silu(gate)*up is a register epilogue and only h is written.
// Activation rows of GEMM1 are gathered through local_src; large batches of wide
// layers first copy them in row order (pack_tokens_kernel).  Which tiles a batch
// takes: ffn_paths.h.  fp32 layers: expert_ffn_f32.hip.
#include "grouped_gemm.h"
#include "prism_internal.h"

namespace prism {
namespace {

// ---------------------------------------------------------------------------
// bf16 path: two grouped GEMMs on the matrix cores
// ---------------------------------------------------------------------------
template <int BM_, int BN_, int BK_, int STAGES_> struct TileCfg {
  static constexpr int BM = BM_, BN = BN_, BK = BK_, STAGES = STAGES_;
};

// Fixed cost of one round of items of a split down projection, as weight bytes a workgroup
// could have streamed meanwhile (first loads of the ring, epilogue, partial-tile stores): fitted
// to the times of a 32-token batch of the 4096 x 14336 layer run with 2 to 8 splits.
constexpr float kSplitRoundBytes = 14 * 8192.f;

// Wide tiles of a path with two widths (schedule.h, "Two widths"): ring of their own, fewest items.
constexpr int kWideStages = 3;
constexpr int kWideItemsUp = 150, kWideItemsDown = 48;

// What the schedule builders need to know about a path's two GEMMs (C1: gate/up, C2: down).
template <typename C1, typename C2, bool SPLIT_DOWN, bool ROTATE, bool WIDTHS>
FfnShapes shapes_of(const prism_layer_desc& d, int T) {
  FfnShapes f{};
  f.bm1 = C1::BM;
  f.nt1 = ceil_div(d.ffn, C1::BN / 2);     // GEMM1 tile: BN/2 gate rows + BN/2 up rows
  f.bm2 = C2::BM;
  f.nt2 = ceil_div(d.hidden, C2::BN);
  f.interleave = ROTATE;
  // prefill tiles: the down projection's last round may be cut along its contraction
  f.slice_kt2 = !SPLIT_DOWN && C2::BM == 256 && down_slicing_applies(d, T) ? d.ffn / C2::BK : 0;
  if (SPLIT_DOWN) {
    f.split_kt2 = d.ffn / C2::BK;
    f.split_min_kt2 = C2::STAGES - 1;      // a slice must be at least as long as the k-tile ring
    f.split_wgs2 = gg::gemm_wgs_per_xcd<C2::BM, C2::BN, 2, C2::BK, C2::STAGES, false, true>();
    const float kt_bytes = (float)(C2::BN * C2::BK * 2);   // weight bytes of one k-tile
    f.split_round_kt2 = kSplitRoundBytes / kt_bytes;
    // one more split: every row written once more as fp32 and read once more, shared by all workgroups
    f.split_row_kt2 = (float)d.hidden * 8.f / (float)(gg::kXcds * f.split_wgs2) / kt_bytes;
  }
  if (WIDTHS) {
    static_assert(!WIDTHS || (SPLIT_DOWN && ROTATE && kWideStages <= C1::STAGES && kWideStages <= C2::STAGES),
                  "the wide tiles' ring is no longer than the slices that the narrow ones allow");
    f.wide_nt1 = ceil_div(d.ffn, C1::BN);
    f.wide_nt2 = ceil_div(d.hidden, 2 * C2::BN);
    f.wide_items1 = kWideItemsUp;
    f.wide_items2 = kWideItemsDown;
  }
  return f;
}

// Sums the contraction slices of the split down projection: y = bf16(sum_s part[s]).
__global__ __launch_bounds__(256) void reduce_splits_kernel(const float* __restrict__ part,
                                                            const int32_t* __restrict__ local_offsets,
                                                            int E, int A, int rows, int H,
                                                            const int32_t* __restrict__ n_splits_ptr,
                                                            uint16_t* __restrict__ y) {
  const int n_splits = min(*n_splits_ptr, kDecodeSplits);   // what the schedule builder chose
  const int vec_per_row = H / 4;
  const long long gid = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (gid >= (long long)rows * vec_per_row) return;
  const int row = (int)(gid / vec_per_row);
  if (row >= local_offsets[E] && row < A) return;   // rows that hold no assignment
  const int col = (int)(gid - (long long)row * vec_per_row) * 4;
  f32x4 v[kDecodeSplits];   // all slices asked for before the first is added
#pragma unroll
  for (int s = 0; s < kDecodeSplits; ++s)
    if (s < n_splits) v[s] = *reinterpret_cast<const f32x4*>(part + ((size_t)s * rows + row) * H + col);
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int s = 0; s < kDecodeSplits; ++s)
    if (s < n_splits) acc += v[s];
  bf16x4 o;
#pragma unroll
  for (int e = 0; e < 4; ++e) o[e] = (bf16_t)acc[e];
  *reinterpret_cast<bf16x4*>(y + (size_t)row * H + col) = o;
}

// Adds up the slices of the down-projection tiles whose contraction the schedule cut (its last
// round of work items): y tile = bf16(sum of the tile's fp32 partial tiles, in slice order).
// One workgroup per (line of the schedule's list of sliced items, 16 rows of the tile) -- few
// lines are in use at a time, so the rows of a tile are spread over many workgroups; lines that
// are not in use end at once.
constexpr int kSliceTile = 256;    // the partial tiles are 256 x 256 (the prefill tile)
constexpr int kSumRows = 16;       // rows of a tile per workgroup of sum_slices_kernel
constexpr int kSumChunks = kSliceTile / kSumRows;
__global__ __launch_bounds__(256) void sum_slices_kernel(const int32_t* __restrict__ sched, int capacity,
                                                         const float* __restrict__ part, int N,
                                                         uint16_t* __restrict__ y) {
  const int line = blockIdx.x / kSumChunks, chunk = blockIdx.x % kSumChunks;
  const int4* red = reinterpret_cast<const int4*>(sched + gg::sched_reduce_offset(capacity)) +
                    (size_t)line * (gg::kReduceInts / 4);
  const int n_slices = red[1].x;
  if (n_slices <= 0) return;
  const int4 a = red[0];
  const int row_start = a.x, row_count = a.y, first = a.w;
  const int row_end = min(row_count, chunk * kSumRows + kSumRows);
  const int col0 = a.z * kSliceTile;
  const int col = (threadIdx.x & 63) * 4;
  if (col0 + col >= N) return;
  // Two rows per wavefront and pass; all slices of both rows are asked for before the first is
  // added (the partial tiles are read once: non-temporal); the sums themselves run in slice order.
  for (int r0 = chunk * kSumRows + (threadIdx.x >> 6); r0 < row_end; r0 += 8) {
    f32x4 v[2][gg::kMaxSlices];
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int c = 0; c < gg::kMaxSlices; ++c)
        if (c < n_slices && r0 + 4 * u < row_end)
          v[u][c] = __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(
              part + ((size_t)(first + c) * kSliceTile + r0 + 4 * u) * kSliceTile + col));
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      if (r0 + 4 * u >= row_end) break;
      f32x4 sum = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int c = 0; c < gg::kMaxSlices; ++c)
        if (c < n_slices) sum += v[u][c];
      bf16x4 o;
#pragma unroll
      for (int e = 0; e < 4; ++e) o[e] = (bf16_t)sum[e];
      *reinterpret_cast<bf16x4*>(y + (size_t)(row_start + r0 + 4 * u) * N + col0 + col) = o;
    }
  }
}

// Prefill batches of wide layers: the token of every row the gate/up GEMM multiplies, copied into
// 16 x 32 tiles in row order, so that the GEMM fetches its 32-wide activation k-tiles as whole cache
// lines instead of half a line of each gathered row (grouped_gemm.h, "Intermediate").
// Bound: HBM, 4 H bytes per row.  4096 tokens of the 4096 x 14336 layer: gate/up with the copy 1341
// us against 1411 gathered (row-major weights 1386 against 1457), 1000 tokens 395 against 410, 600
// tokens 380 against 382.  A wavefront takes 16 rows x 256 columns.
__global__ __launch_bounds__(256) void pack_tokens_kernel(const uint4* __restrict__ x,
                                                          const int32_t* __restrict__ local_src,
                                                          const int32_t* __restrict__ local_offsets, int E, int A,
                                                          int rows, int T, int top_k, int H, uint4* __restrict__ out,
                                                          int32_t* __restrict__ row_places) {
  const int lane = threadIdx.x & 63;
  const int r = blockIdx.x * 16 + (lane >> 2);
  if (r >= rows || (r >= local_offsets[E] && r < A)) return;   // rows that hold no assignment
  const int tok = r < A ? local_src[r] / top_k : (r - A) % T;
  if (blockIdx.y == 0 && threadIdx.x < 64 && (lane & 3) == 0) row_places[r] = blockIdx.x * (H / 32) * 16 + (lane >> 2);
  const int tiles = H / 32, tile0 = (blockIdx.y * 4 + (threadIdx.x >> 6)) * 8;
  const uint4* src = x + (size_t)tok * (H / 8) + (lane & 3);
  uint4* dst = out + (size_t)blockIdx.x * tiles * 64 + lane;
  uint4 v[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) v[j] = src[min(tile0 + j, tiles - 1) * 4];
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int j = 0; j < 8; ++j)
    if (tile0 + j < tiles) dst[(tile0 + j) * 64] = v[j];
}
template <typename C1, typename C2, bool SPLIT_DOWN, bool STREAM_B, bool ROTATE, bool WIDTHS>
prism_status run_bf16_ffn(const prism_layer_desc& d, const void* x, const prism_expert_weights& w,
                          const int32_t* local_src, const int32_t* local_offsets, int T, void* y,
                          void* h, bool h_tiled, void* x_rows, int32_t* tiles, float* part, float* slice_part, hipStream_t st,
                          void* const* stage_events, const int32_t** deferred_splits,
                          bool schedules_built) {
  using gg::GemmArgs;
  const int A = T * d.top_k;
  const int rows = A + d.n_shared * T;
  // the k-tile ring of a workgroup must not be longer than its contraction slice
  if (d.hidden / C1::BK < C1::STAGES - 1 || d.ffn / C2::BK < C2::STAGES - 1) return PRISM_ERR_UNSUPPORTED;
  int32_t* sched1 = tiles;
  int32_t* sched2 = tiles + tile_table_ints(d, T);
  // The schedules (built here, or by the caller's dispatch) follow ffn_schedule_shapes(), which
  // must describe the kernels this instantiation launches.
  const FfnShapes f = shapes_of<C1, C2, SPLIT_DOWN, ROTATE, WIDTHS>(d, T);
  const FfnShapes told = ffn_schedule_shapes(d, T);
  if (f.bm1 != told.bm1 || f.nt1 != told.nt1 || f.bm2 != told.bm2 || f.nt2 != told.nt2 ||
      f.interleave != told.interleave || f.slice_kt2 != told.slice_kt2 || f.split_kt2 != told.split_kt2 ||
      f.split_wgs2 != told.split_wgs2 || f.wide_nt1 != told.wide_nt1 || f.wide_nt2 != told.wide_nt2)
    return PRISM_ERR_LAUNCH;
  const int nt1 = f.nt1, nt2 = f.nt2;
  // the down projection's last round of items may be cut along the contraction (prefill only)
  const int slice_kt = slice_part != nullptr ? f.slice_kt2 : 0;
  if (slice_kt != f.slice_kt2) return PRISM_ERR_INVALID_ARG;   // the schedule would hold slice entries
  constexpr bool kCanSlice = !SPLIT_DOWN && C2::BM == kSliceTile;   // as shapes_of
  static_assert(!kCanSlice || (C2::BN == kSliceTile && C2::BK == 32), "sum_slices_kernel assumes the prefill tile");
  static_assert(!kCanSlice || C1::BK == 32, "a gate/up k-tile reads one 64-byte row of the tiles of the token copy");
  if (!schedules_built) PRISM_TRY(gg::launch_build_schedules(d, local_offsets, T, tiles, st));

  GemmArgs g1{};
  g1.A = (const uint16_t*)x;
  g1.B0 = w.w_gate; g1.B1 = w.w_up; g1.SB0 = w.shared_w_gate; g1.SB1 = w.shared_w_up;
  g1.C = (uint16_t*)h;
  g1.sched = sched1; g1.local_src = local_src;
  g1.src_bytes = (uint32_t)A * 4;
  g1.a_bytes = (uint32_t)((size_t)T * d.hidden * 2);
  g1.b_bytes = (uint32_t)((size_t)d.ffn * d.hidden * 2);
  g1.K = d.hidden; g1.N = d.ffn; g1.top_k = d.top_k; g1.E = d.n_experts;
  g1.b_tiled = d.weight_layout == PRISM_WEIGHTS_TILED;
  g1.c_tiled = h_tiled;
  g1.a_pitch = (uint32_t)d.hidden * 2;
  g1.a_kstep = 64;
  if (kCanSlice && pack_rows_pays(d, T)) {
    int32_t* row_places = (int32_t*)((uint8_t*)x_rows + align_up(rows, 16) * d.hidden * 2);
    hipLaunchKernelGGL(pack_tokens_kernel, dim3((unsigned)ceil_div(rows, 16), (unsigned)ceil_div(d.hidden, 1024)),
                       dim3(256), 0, st, (const uint4*)x, local_src, local_offsets, d.n_experts, A, rows, T, d.top_k,
                       d.hidden, (uint4*)x_rows, row_places);
    PRISM_CHECK_LAUNCH();
    trace(stage_events, PRISM_STAGE_DISPATCH, 1, st);   // the copy counts as dispatch: its end is recorded anew
    g1.A = (const uint16_t*)x_rows;
    g1.a_bytes = (uint32_t)(align_up(rows, 16) * d.hidden * 2);
    g1.a_tiled = 1;
    g1.local_src = row_places;
    g1.src_bytes = (uint32_t)rows * 4;
    g1.top_k = 1;
    g1.a_pitch = 64;
    g1.a_kstep = 1024;
  }
  trace(stage_events, PRISM_STAGE_FFN_UP, 0, st);
  if constexpr (WIDTHS) {
    static_assert(STREAM_B && ROTATE, "as the kernel's narrow tiles");
    PRISM_TRY((gg::launch_gemm_widths<C1::BM, C1::BN, C1::BK, C1::STAGES, kWideStages, true, false>(g1, st)));
  } else {
    PRISM_TRY((gg::launch_gemm<C1::BM, C1::BN, 2, 2, C1::BK, C1::STAGES, true, false, ROTATE, STREAM_B>(
        g1, gg::sched_capacity(d, T, C1::BM, nt1), st)));
  }
  trace(stage_events, PRISM_STAGE_FFN_UP, 1, st);

  GemmArgs g2{};
  g2.A = (const uint16_t*)h;
  g2.B0 = w.w_down; g2.B1 = nullptr; g2.SB0 = w.shared_w_down; g2.SB1 = nullptr;
  g2.C = (uint16_t*)y;
  g2.Cpart = SPLIT_DOWN ? part : slice_part; g2.c_rows = rows;
  g2.sched = sched2; g2.local_src = local_src;
  g2.a_bytes = (uint32_t)((h_tiled ? align_up(rows, 16) : (size_t)rows) * d.ffn * 2);
  g2.b_bytes = (uint32_t)((size_t)d.ffn * d.hidden * 2);
  g2.K = d.ffn; g2.N = d.hidden; g2.top_k = d.top_k; g2.E = d.n_experts;
  g2.b_tiled = d.weight_layout == PRISM_WEIGHTS_TILED;
  g2.a_tiled = h_tiled;
  g2.a_pitch = (uint32_t)d.ffn * 2;
  g2.a_kstep = h_tiled ? 1024 : 64;
  // SPLIT_DOWN: the number of contraction slices is in the schedule's header (schedule.h, "Splits")
  const int32_t* n_splits = sched2 + 2;
  trace(stage_events, PRISM_STAGE_FFN_DOWN, 0, st);
  if constexpr (WIDTHS) {
    PRISM_TRY((gg::launch_gemm_widths<C2::BM, C2::BN, C2::BK, C2::STAGES, kWideStages, false, SPLIT_DOWN>(g2, st)));
  } else {
    PRISM_TRY((gg::launch_gemm<C2::BM, C2::BN, 2, 2, C2::BK, C2::STAGES, false, SPLIT_DOWN, ROTATE, STREAM_B>(
        g2, gg::sched_capacity(d, T, C2::BM, nt2), st)));
  }
  if constexpr (kCanSlice) {
    if (slice_kt > 0)   // the cut last round: one slice entry per workgroup, fp32 partial tiles
      PRISM_TRY((gg::launch_gemm<C2::BM, C2::BN, 2, 2, C2::BK, C2::STAGES, false, false, false, false, true>(
          g2, gg::sched_capacity(d, T, C2::BM, nt2), st)));
  }
  if (slice_kt > 0) {
    hipLaunchKernelGGL(sum_slices_kernel, dim3(gg::kXcds * (gg::kSliceSlots / 2) * kSumChunks), dim3(256), 0, st, sched2,
                       gg::sched_capacity(d, T, C2::BM, nt2), slice_part, d.hidden, (uint16_t*)y);
    PRISM_CHECK_LAUNCH();
  }
  if (SPLIT_DOWN && deferred_splits != nullptr) {
    *deferred_splits = n_splits;   // the caller's combine sums the slices itself
  } else if (SPLIT_DOWN) {
    const long long threads = (long long)rows * (d.hidden / 4);
    hipLaunchKernelGGL(reduce_splits_kernel, dim3((unsigned)((threads + 255) / 256)), dim3(256), 0, st,
                       part, local_offsets, d.n_experts, A, rows, d.hidden, n_splits, (uint16_t*)y);
    PRISM_CHECK_LAUNCH();
  }
  trace(stage_events, PRISM_STAGE_FFN_DOWN, 1, st);
  return PRISM_OK;
}

// One tile path of the bf16 FFN: tile shapes of the two GEMMs, whether the down projection is
// split along its contraction, whether the weight loads are marked non-temporal, whether the items
// are dealt to the XCDs one by one with rotated contractions (grouped_gemm.h, ROTATE), whether the
// schedule may choose tiles twice as wide instead.
template <typename C1_, typename C2_, bool SPLIT_DOWN_, bool STREAM_B_, bool ROTATE_, bool WIDTHS_ = false> struct Path {
  using C1 = C1_;
  using C2 = C2_;
  static constexpr bool kSplitDown = SPLIT_DOWN_, kStreamB = STREAM_B_, kRotate = ROTATE_, kWidths = WIDTHS_;
};

// Calls fn(Path<...>{}) with the path that serves a bf16 batch of T tokens of layer d (ffn_paths.h).
template <typename Fn>
auto select_path(const prism_layer_desc& d, int T, Fn&& fn) {
  using Decode = TileCfg<64, 128, 64, 4>;
  using Square = TileCfg<128, 128, 64, 4>;
  using Wide = TileCfg<128, 256, 64, 3>;
  switch (ffn_path(d, T)) {
    case FfnPath::kDecodeTiled: return fn(Path<TileCfg<64, 128, 32, 8>, TileCfg<64, 128, 32, 8>, true, true, true>{});
    case FfnPath::kDecode: return fn(Path<Decode, Decode, true, true, true>{});
    case FfnPath::kDecodeShort: return fn(Path<TileCfg<64, 128, 32, 3>, TileCfg<64, 128, 32, 3>, true, true, true>{});
    case FfnPath::kStream: return fn(Path<Square, Square, true, true, true, true>{});
    case FfnPath::kSplitSquare: return fn(Path<Square, Square, true, false, false>{});
    case FfnPath::kSplitWide: return fn(Path<Wide, Wide, true, false, false>{});
    case FfnPath::kFewRows64: return fn(Path<Decode, Decode, false, true, false>{});
    case FfnPath::kFewRows128: return fn(Path<Wide, Square, false, false, false>{});
    case FfnPath::kPrefill: return fn(Path<TileCfg<256, 256, 32, 4>, TileCfg<256, 256, 32, 4>, false, false, false>{});
    default: return fn(Path<TileCfg<256, 256, 32, 3>, TileCfg<256, 256, 32, 3>, false, false, false>{});
  }
}

}  // namespace

prism_status launch_expert_ffn(const prism_layer_desc& d, const void* x,
                               const prism_expert_weights& w, const int32_t* local_src,
                               const int32_t* local_offsets, int T, void* y, void* h,
                               bool h_tiled, void* x_rows, int32_t* tiles, float* part, float* slice_part, hipStream_t st,
                               void* const* stage_events, const int32_t** deferred_splits,
                               bool schedules_built) {
  if (deferred_splits != nullptr) *deferred_splits = nullptr;
  if (T == 0) return PRISM_OK;
  if (d.dtype == PRISM_F32)
    return launch_expert_ffn_f32(d, x, w, local_src, local_offsets, T, y, h, st, stage_events);

  const int rows = T * (d.top_k + d.n_shared);
  // bf16: schedules for the two GEMMs, then the GEMMs.  Buffer addressing uses
  // 32-bit byte offsets, so every operand matrix must stay below 4 GiB.
  constexpr size_t kMaxOperandBytes = 0xFFFF0000ull;
  if ((size_t)T * d.hidden * 2 >= kMaxOperandBytes || (size_t)rows * d.ffn * 2 >= kMaxOperandBytes ||
      (size_t)d.ffn * d.hidden * 2 >= kMaxOperandBytes)
    return PRISM_ERR_UNSUPPORTED;
  if (align_up(rows, 16) * d.ffn * 2 >= kMaxOperandBytes) h_tiled = false;   // (the buffer holds the plain rows too)
  return select_path(d, T, [&](auto path) {
    using P = decltype(path);
    return run_bf16_ffn<typename P::C1, typename P::C2, P::kSplitDown, P::kStreamB, P::kRotate, P::kWidths>(
        d, x, w, local_src, local_offsets, T, y, h, h_tiled, x_rows, tiles, part, slice_part, st, stage_events, deferred_splits,
        schedules_built);
  });
}

FfnShapes ffn_schedule_shapes(const prism_layer_desc& d, int T) {
  return select_path(d, T, [&](auto path) {
    using P = decltype(path);
    return shapes_of<typename P::C1, typename P::C2, P::kSplitDown, P::kRotate, P::kWidths>(d, T);
  });
}

}  // namespace prism
