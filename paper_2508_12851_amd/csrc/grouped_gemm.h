// Grouped "NT" GEMM on the bf16 matrix cores of gfx950, used for both halves of
// the SwiGLU expert FFN (paper Sec. III-A, local expert execution):
//
//   GATED   h[r, f] = silu( x[tok(r)] . W_gate^g[f] ) * ( x[tok(r)] . W_up^g[f] )
//   plain   y[r, n] = h[r] . W_down^g[n]
//
// Rows are grouped by expert g; a device-built schedule gives every workgroup its
// (row tile, column tile) items, so the host never needs the routing-dependent
// segment sizes.
//
// Kernel shape: BM x BN output tile per workgroup of 4 wavefronts (WGM x WGN),
// v_mfma_f32_32x32x16_bf16, operand tiles of BK contraction elements staged in
// LDS in a ring of STAGES stages.  An LDS row holds BK contraction elements
// (128 or 64 bytes) as 16-byte chunks; chunk c of row r sits in slot
// c ^ key(r) (key = (r >> 1) & 7 for 128-byte rows, (r >> 2) & 3 for 64-byte
// rows), so the 16-byte operand reads of 16 consecutive rows hit 16 different
// slots of the 256-byte bank window.  Stages are filled by buffer_load_dwordx4
// ... lds (no VGPR staging): one instruction fills 1 KiB, and because each
// lane's LDS slot is fixed (lane * 16 bytes), the swizzle is applied to the
// global chunk a lane fetches instead.  A stage is awaited with s_waitcnt
// vmcnt(n), n = the loads of the younger stages, then one s_barrier per stage
// orders the ring.
//
// The kernel is persistent: a workgroup walks its list of items, and the ring
// keeps running across items -- while the last k-tiles of one item are being
// multiplied, the first k-tiles of the next are already being fetched, and they
// land while the epilogue of the first stores its results.
//
// Work order: the hardware hands consecutive workgroup ids to the 8 XCDs in
// turn, each with a private L2.  The schedule (schedule.h) gives every XCD one
// list of items in which consecutive items form small rectangles of row tiles x
// column tiles of one expert, so the workgroups resident on an XCD share a few
// activation tiles and a few weight tiles in that XCD's L2.
#ifndef PRISM_GROUPED_GEMM_H_
#define PRISM_GROUPED_GEMM_H_

#include <type_traits>

#include "prism_internal.h"
#include "schedule.h"

namespace prism {
namespace gg {

// Workgroup b builds the schedule p[b] (one launch serves both GEMMs of the FFN).
template <bool WIDTHS>
__global__ __launch_bounds__(512) void build_schedule_kernel(
    const int32_t* __restrict__ local_offsets, int E, int S, int T, int A_total,
    const sched_params_t<WIDTHS> p0, const sched_params_t<WIDTHS> p1) {
  const sched_params_t<WIDTHS> p[1] = {blockIdx.x == 0 ? p0 : p1};
  build_schedules_block<1, WIDTHS>(local_offsets, E, S, T, A_total, p);
}

struct GemmArgs {
  const uint16_t* A;        // GATED: x [T, K]; else h [rows, K]
  const void* const* B0;    // routed: W_gate (GATED) or W_down tables
  const void* const* B1;    // routed: W_up table (GATED only)
  const void* const* SB0;   // shared experts, same roles
  const void* const* SB1;
  uint16_t* C;              // GATED: h [rows, N]; else y [rows, N]
  float* Cpart;             // SPLITK: [n_splits][c_rows][N] fp32 partial sums
  int c_rows;               // rows of one partial-sum slice
  const int32_t* sched;
  const int32_t* local_src;
  uint32_t src_bytes;       // size of local_src in bytes (T * k * 4)
  uint32_t a_bytes;         // size of A in bytes (buffer range check), < 2^32
  uint32_t b_bytes;         // size of one weight matrix in bytes, < 2^32
  int K;                    // contraction length (H for GEMM1, F for GEMM2)
  int N;                    // output columns (F for GEMM1, H for GEMM2)
  int top_k;
  int E;
  int b_tiled;              // weights in 16 x 32 tiles (prism.h) instead of row-major
  int a_tiled;              // A in the same tiles.  GATED: A is the packed copy of x, and local_src holds, for every
                            // output row, the place of its first 32 elements in 64-byte units (top_k is 1)
  uint32_t a_pitch;         // bytes from one source row of A to the next (GATED and a_tiled: 64)
  int a_kstep;              // bytes from 32 contraction elements of a row of A to the next 32
  int c_tiled;              // GATED: h is written in the same tiles ("Intermediate" below)
};

// Intermediate.  h is written by one of the two GEMMs and read by the other, so it lies in the order
// that serves both: 16 x 32 tiles of 1 KiB over the absolute row number, like packed weights.  The
// down projection then fetches its activation k-tiles as whole cache lines (a row-major row gives
// 64 bytes per 32-wide k-tile, half a line, and the L2 is asked for the other half again in the next
// one), and a store instruction of the gate/up epilogue covers 32 pieces of 16 bytes that the next
// three complete to a contiguous 2 KiB instead of lines whole rows apart.  Down projection, row-major
// before: 4096 tokens of the 4096 x 14336 layer 716 -> 643 us, 8192 of the 60-expert layer 306 -> 293,
// 2500 of the 64-expert one 122 -> 117; 64-wide k-tiles took whole lines already and gain 0 to 2 %.
constexpr int kGemmThreads = 256;

// Epilogue strips: 32 rows x 64 bf16 columns per wavefront at a row pitch of 144 bytes
// (16-byte aligned rows whose starts fall into different banks).  Used by the plain GEMM when a
// wavefront's output is at least 64 bf16 columns wide (the gated GEMM, whose epilogue is
// dominated by the SiLU arithmetic, ran 5-10 % slower with it).
constexpr int kStripPitch = 144;
constexpr int kStripBytes = 32 * kStripPitch;
template <int WN, bool GATED, bool SPLITK> constexpr bool staged_store() {
  return !SPLITK && !GATED && (WN / 32) % 2 == 0;
}
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// Schedule entries and pointer tables are written before the kernel starts and
// never during it; reading them through the constant address space lets the
// compiler use scalar loads, which the vector-memory counter does not see.
typedef const __attribute__((address_space(4))) int4* const_int4_ptr;
typedef const __attribute__((address_space(4))) int32_t* const_int_ptr;
typedef const void* const __attribute__((address_space(4)))* const_ptr_table;

// silu(z) = z / (1 + e^-z) with the hardware exp2 and reciprocal (each within 1 ulp;
// the result is rounded to bf16 right after).
__device__ __forceinline__ float silu(float z) {
  return z * __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(-1.44269504088896341f * z));
}

// LDS slot swizzle.  The LDS serves a 16-byte-per-lane read 16 lanes (256 bytes,
// 64 banks) per cycle, so 16 consecutive rows read at the same logical chunk
// must land in 16 different 16-byte slots of the 256-byte bank window: rows
// that share (row * row_bytes) mod 256 get different keys.
template <int BK> __device__ __forceinline__ int swizzle_key(int row) {
  return BK == 64 ? ((row >> 1) & 7) : ((row >> 2) & 3);
}

// BM x BN output tile per workgroup; BN counts weight rows in the tile (for
// GATED: BN/2 gate rows and BN/2 up rows).  Wavefronts form a WGM x WGN grid.
// BK contraction elements per LDS stage (32 or 64), STAGES stages in flight.
// SPLITK: n workgroups share every item, each over its own slice of the contraction, n being
// what the schedule builder chose (schedule.h, "Splits"); the tile is written as fp32 partial
// sums to p.Cpart[slice][row][col] (plain GEMM only).
// ROTATE: every item walks its k-tiles cyclically from an item-dependent start, so
// concurrent workgroups read different column ranges of their weight rows (for
// schedules in which workgroups share no weight tiles, i.e. one row tile per group).
// These are the schedules that deal their items to the XCDs one by one; the kernel works out
// its items from the schedule's table of row tiles (schedule.h) instead of reading lists.
// STREAM_B: the weight loads carry the non-temporal hint.  For batches in which every weight
// tile is read by one workgroup only (one row tile per expert) the weights cross the memory
// system once, and reads marked that way stream from HBM about 15 % faster than plain ones
// (7.0-7.2 against 6.2-6.4 TB/s for direct-to-LDS loads on this machine).
// SLICES: the launch takes the schedule's slice entries -- the items of a partly filled last
// round, cut along the contraction (schedule.h, "Last round") -- instead of its item lists: an
// entry covers its own range of k-tiles and leaves its accumulators as an fp32 tile in slot
// `part` of p.Cpart (plain GEMM only).  A launch of its own, so that the kernel that does the
// bulk of the work carries none of this.
template <int BM, int BN, int WGM, int WGN, int BK, int STAGES, bool GATED, bool SPLITK = false,
          bool ROTATE = false, bool STREAM_B = false, bool SLICES = false>
__global__ __launch_bounds__(kGemmThreads) void grouped_gemm_kernel(const GemmArgs p) {
#include "grouped_gemm_body.h"
}

// The tiles the schedule chose (schedule.h, "Two widths"): BM x BN streamed, or BM x 2 BN in lists.  One launch
// for both: a second one that ends at once would cost about 4 us.
template <int BM, int NARROW, int BK, int NARROW_STAGES, int WIDE_STAGES, bool GATED, bool SPLITK>
__global__ __launch_bounds__(kGemmThreads) void grouped_gemm_widths_kernel(const GemmArgs p) {
  constexpr int WGM = 2, WGN = 2;
  constexpr bool SLICES = false;
  if (((const_int_ptr)p.sched)[3] != 0) {
    constexpr int BN = 2 * NARROW, STAGES = WIDE_STAGES;
    constexpr bool ROTATE = false, STREAM_B = false;
#include "grouped_gemm_body.h"
  } else {
    constexpr int BN = NARROW, STAGES = NARROW_STAGES;
    constexpr bool ROTATE = true, STREAM_B = true;
#include "grouped_gemm_body.h"
  }
}

// Launches the schedule builder for the two GEMMs of the FFN of a batch of T tokens.
static inline prism_status launch_build_schedules(const prism_layer_desc& d,
                                                  const int32_t* local_offsets, int T,
                                                  int32_t* tiles, hipStream_t st) {
  WidthParams p0, p1;
  ffn_sched_params(d, T, tiles, &p0, &p1);
  auto launch = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3(2), dim3(512), 0, st, local_offsets, d.n_experts, d.n_shared, T, T * d.top_k, p0, p1);
  };
  if (p0.wide_ntiles > 0) launch(build_schedule_kernel<true>);
  else launch(build_schedule_kernel<false>);
  PRISM_CHECK_LAUNCH();
  return PRISM_OK;
}

// LDS of one workgroup of a tile shape, and how many of them a CU holds.
template <int BM, int BN, int WGN, int BK, int STAGES, bool GATED, bool SPLITK>
constexpr int gemm_lds_bytes() {
  return STAGES * (BM + BN) * BK * 2 + (GATED ? 4096 : 0) +           // ring + source-row slots
         (staged_store<BN / WGN, GATED, SPLITK>() ? 4 * kStripBytes : 0);   // + strips
}
constexpr int kCusPerXcd = 32;
template <int BM, int BN, int WGN, int BK, int STAGES, bool GATED, bool SPLITK>
constexpr int gemm_wgs_per_xcd() {
  return kCusPerXcd * ((160 * 1024) / gemm_lds_bytes<BM, BN, WGN, BK, STAGES, GATED, SPLITK>());
}

// capacity: items per XCD list (sched_capacity).  The grid holds as many workgroups
// as fit on the machine at once (each then walks several items), or one per item.
template <int BM, int BN, int WGM, int WGN, int BK, int STAGES, bool GATED, bool SPLITK = false,
          bool ROTATE = false, bool STREAM_B = false, bool SLICES = false>
prism_status launch_gemm(const GemmArgs& args, int capacity, hipStream_t st, int max_slots = 0) {
  constexpr int smem = gemm_lds_bytes<BM, BN, WGN, BK, STAGES, GATED, SPLITK>();
  static_assert(smem <= 160 * 1024, "LDS per workgroup");
  auto kernel = grouped_gemm_kernel<BM, BN, WGM, WGN, BK, STAGES, GATED, SPLITK, ROTATE, STREAM_B, SLICES>;
  static LdsLimitOnce lds_limit;   // one per instantiation
  if (!raise_lds_limit(lds_limit, (const void*)kernel, smem)) return PRISM_ERR_LAUNCH;
  if (capacity <= 0) return PRISM_OK;
  // persistent workgroups per XCD: as many as are resident at once (SPLITK: the schedule says
  // how they pair up, so the launch is never cut down to the list length)
  int slots = gemm_wgs_per_xcd<BM, BN, WGN, BK, STAGES, GATED, SPLITK>();
  if (max_slots > 0) slots = max_slots;
  if (!SPLITK && slots > capacity) slots = capacity;
  hipLaunchKernelGGL(kernel, dim3((unsigned)(slots * kXcds)), dim3(kGemmThreads), smem, st, args);
  PRISM_CHECK_LAUNCH();
  return PRISM_OK;
}

// The same for grouped_gemm_widths_kernel.
template <int BM, int BN, int BK, int STAGES, int WIDE_STAGES, bool GATED, bool SPLITK>
prism_status launch_gemm_widths(const GemmArgs& args, hipStream_t st) {
  constexpr int narrow = gemm_lds_bytes<BM, BN, 2, BK, STAGES, GATED, SPLITK>();
  constexpr int wide = gemm_lds_bytes<BM, 2 * BN, 2, BK, WIDE_STAGES, GATED, SPLITK>();
  constexpr int smem = narrow > wide ? narrow : wide;
  static_assert(smem <= 160 * 1024 && smem > 80 * 1024, "one workgroup per CU");
  auto kernel = grouped_gemm_widths_kernel<BM, BN, BK, STAGES, WIDE_STAGES, GATED, SPLITK>;
  static LdsLimitOnce lds_limit;   // one per instantiation
  if (!raise_lds_limit(lds_limit, (const void*)kernel, smem)) return PRISM_ERR_LAUNCH;
  hipLaunchKernelGGL(kernel, dim3(kCusPerXcd * kXcds), dim3(kGemmThreads), smem, st, args);
  PRISM_CHECK_LAUNCH();
  return PRISM_OK;
}

}  // namespace gg
}  // namespace prism
#endif  // PRISM_GROUPED_GEMM_H_
