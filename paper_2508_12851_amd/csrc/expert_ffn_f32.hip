// Grouped SwiGLU expert FFN of fp32 layers (paper Sec. III-A) on the fp32 matrix cores.
//
//   GATED   h[r, f] = silu( x[tok(r)] . W_gate^e[f] ) * ( x[tok(r)] . W_up^e[f] )
//   plain   y[r, n] = h[r] . W_down^e[n]
//
// Bound: the matrix cores' fp32 rate (v_mfma_f32_32x32x2_f32: 157 TFLOP/s nominal on 256 CUs) once an expert
// has a few dozen rows, the weight stream below that.
//
// Split: a workgroup owns 64 rows of one expert x 64 weight rows (GATED: 32 gate rows and the 32 up
// rows of the same f), and its 8 wavefronts split the contraction: each multiplies its own eighth in
// 16-wide k-tiles that it stages through 8 KiB of LDS of its own, so the k-loop has no workgroup
// barrier, and a tile of even the smallest layer is spread over all four SIMDs (242 registers: one
// workgroup, two wavefronts per SIMD).  The next k-tile travels from memory to registers during the MFMAs of this
// one (32 MFMAs of 64 clocks per wavefront and k-tile).
//
// Sums: fp32 results must not get worse than those of the kernel that this one replaced (64 lane sums
// of K / 64 terms, then a tree).  Four products are added in the matrix core, the four partial sums of
// a k-tile pairwise, the k-tile sums of a wavefront one after the other (K / 128 terms, the only chain
// that grows with the contraction), the eighths as a tree.  Relative 2-norm of the error against 64 bits,
// random operands, 256 / 1024 / 2048 terms: 7.8e-8 / 9.2e-8 / 1.06e-7, before 7.9e-8 / 1.0e-7 / 1.23e-7.
//
// One wavefront per output element with the products on the vector ALU (the kernel before) read
// every weight row once per activation row: at 500 tokens of a 1024 x 2048 layer, 5 of 8 experts
// hosted, gate/up + down took 1173 + 1105 us.
#include "prism_internal.h"

namespace prism {
namespace {

struct F32Args {
  const float* x;
  const void* const* wg; const void* const* wu; const void* const* wd;
  const void* const* swg; const void* const* swu; const void* const* swd;
  const int32_t* local_src; const int32_t* local_offsets;
  float* h; float* y;
  int T, H, F, E, S, top_k;
};

constexpr int kBM = 64;                  // rows of a tile
constexpr int kBN = 64;                  // weight rows of a tile
constexpr int kBK = 16;                  // contraction elements per k-tile
constexpr int kWaves = 8;
constexpr int kThreads = kWaves * kWave;
constexpr int kXcds = 8;
constexpr int kMaxGridX = 1 << 22;       // workgroups in one row of the grid
static_assert((long long)kMaxGridX * kThreads < (1LL << 32) && kMaxGridX % kXcds == 0, "a row the hardware takes, whole XCD turns");
constexpr int kRowBytes = kBK * 4;
constexpr int kStageBytes = (kBM + kBN) * kRowBytes;         // one wavefront's k-tile
constexpr int kRedPitch = kBN + 4;                           // floats; rows start in different banks
constexpr int kRedFloats = kBM * kRedPitch;                  // one wavefront's partial tile
constexpr int kLdsBytes = kWaves / 2 * kRedFloats * 4;
static_assert(kLdsBytes >= kWaves * kStageBytes, "the partial tiles replace the k-tiles");

// Rows of fp32 matrices start at any multiple of 4 bytes (F need not be a multiple of 4).
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));
// Pointers that come out of a table in memory: said to be global memory, which the compiler cannot know.
typedef const __attribute__((address_space(1))) float* global_ptr;
typedef const __attribute__((address_space(1))) f32x4u* global_ptr4;

struct RowTile {
  int g;           // expert (g < E), shared expert E + s, or -1: nothing here
  int row_start;   // first row in h / y
  int row_count;
  int tok_base;    // shared experts: token of the first row; routed ones: -1
};

// Row tile number b: the tiles of the routed experts in expert order, then those of the shared
// ones.  Every wavefront finds it for itself (4 experts per lane, one scan).
__device__ __forceinline__ RowTile find_row_tile(const F32Args& p, int b) {
  const int lane = threadIdx.x & 63;
  int off[5];
#pragma unroll
  for (int j = 0; j < 5; ++j) off[j] = p.local_offsets[min(4 * lane + j, p.E)];
  int tiles = 0;
#pragma unroll
  for (int j = 0; j < 4; ++j) tiles += (off[j + 1] - off[j] + kBM - 1) / kBM;
  const int incl = wave_inclusive_scan(tiles);
  const int total = __builtin_amdgcn_readlane(incl, 63);
  if (b < total) {
    int rel = b - (incl - tiles), e = 0, start = 0, count = 0;
    const unsigned long long mine = __ballot(rel >= 0 && rel < tiles);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int t = (off[j + 1] - off[j] + kBM - 1) / kBM;
      if (rel >= 0 && rel < t) {
        e = 4 * lane + j;
        start = off[j] + rel * kBM;
        count = min(kBM, off[j + 1] - start);
      }
      rel -= t;
    }
    const int owner = __ffsll(mine) - 1;
    return RowTile{__builtin_amdgcn_readlane(e, owner), __builtin_amdgcn_readlane(start, owner),
                   __builtin_amdgcn_readlane(count, owner), -1};
  }
  const int per_shared = (p.T + kBM - 1) / kBM;
  const int s = (b - total) / per_shared, tok = (b - total - s * per_shared) * kBM;
  if (s >= p.S) return RowTile{-1, 0, 0, -1};
  return RowTile{p.E + s, p.T * (p.top_k + s) + tok, min(kBM, p.T - tok), tok};
}

template <bool GATED>
__global__ __launch_bounds__(kThreads) void ffn_f32_kernel(const F32Args p, int n_row_tiles, int n_items) {
  extern __shared__ __align__(16) float smem[];
  // Consecutive workgroups go to the 8 XCDs in turn; every XCD takes a contiguous eighth of the
  // items, row tiles running fastest, so that the row tiles of an expert read its weight rows
  // through one L2.
  const unsigned wg = blockIdx.y * gridDim.x + blockIdx.x, wgs = gridDim.x * gridDim.y;   // (gridDim.x % 8 == 0)
  const int item = (int)(wg % kXcds * (wgs / kXcds) + wg / kXcds);
  if (item >= n_items) return;
  const int ct = item / n_row_tiles;
  const RowTile rt = find_row_tile(p, item - ct * n_row_tiles);
  if (rt.g < 0) return;

  const int K = GATED ? p.H : p.F, N = GATED ? p.F : p.H;
  constexpr int kCols = GATED ? kBN / 2 : kBN;      // output columns of the tile
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int r32 = lane & 31, q = lane >> 5;

  // ---- global -> LDS assignment: lane l brings chunk l % 4 (4 elements) of rows l / 4 + 16 i ----
  const int lrow = lane >> 2, chunk = lane & 3;
  const bool routed = rt.g < p.E;
  const int gi = routed ? rt.g : rt.g - p.E;
  const float* a_ptr[4];
  uint32_t b_off[4];      // elements (H and F are at most 16384)
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int br = lrow + 16 * i;
    const int rr = min(br, rt.row_count - 1);   // rows past the end repeat the last one
    if (GATED) {
      const int tok = routed ? p.local_src[rt.row_start + rr] / p.top_k : rt.tok_base + rr;
      a_ptr[i] = p.x + (size_t)tok * K;
    } else {
      a_ptr[i] = p.h + (size_t)(rt.row_start + rr) * K;
    }
    b_off[i] = (uint32_t)min(ct * kCols + br % kCols, N - 1) * (uint32_t)K;
  }
  const global_ptr b_lo = (global_ptr)(GATED ? (routed ? p.wg[gi] : p.swg[gi]) : (routed ? p.wd[gi] : p.swd[gi]));
  const global_ptr b_hi = GATED ? (global_ptr)(routed ? p.wu[gi] : p.swu[gi]) : b_lo;   // rows 32 .. 63

  // this wavefront's k-tiles
  const int n_kt = (K + kBK - 1) / kBK;
  const int kt0 = (int)((long long)n_kt * wave / kWaves), kt1 = (int)((long long)n_kt * (wave + 1) / kWaves);
  f32x4 fa[4], fb[4];
  // Element k = kt kBK + 4 chunk and the three after it, of every row this lane brings.  At the end
  // of the rows the last 4 elements come instead (cut_tail puts them right).
  auto fetch = [&](int kt) {
    const uint32_t k = (uint32_t)min(kt * kBK + chunk * 4, K - 4);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      fa[i] = *reinterpret_cast<const f32x4u*>(a_ptr[i] + k);
      fb[i] = *(global_ptr4)((i < 2 ? b_lo : b_hi) + (b_off[i] + k));
    }
  };
  // Last k-tile, if the rows end inside it: what was fetched sits d elements further on; zeros past K.
  auto cut_tail = [&](int kt) {
    const int k = kt * kBK + chunk * 4, d = k - max(min(k, K - 4), 0);
    auto cut = [&](f32x4& v) {
      const f32x4 w = v;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        float x = w[e];
        if (e < 3 && d == 1) x = w[(e + 1) & 3];
        if (e < 2 && d == 2) x = w[(e + 2) & 3];
        if (e < 1 && d == 3) x = w[3];
        v[e] = k + e < K ? x : 0.f;
      }
    };
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      cut(fa[i]);
      cut(fb[i]);
    }
  };

  // 64-byte LDS rows; chunk c of row r sits in slot c ^ ((r >> 2) & 3), so that the 16-byte reads
  // of 16 consecutive rows fall into 16 different slots of the 256-byte bank window.
  uint8_t* const stage = reinterpret_cast<uint8_t*>(smem) + wave * kStageBytes;
  const int wr = lrow * kRowBytes + (chunk ^ ((lrow >> 2) & 3)) * 16;
  const int key = (r32 >> 2) & 3;

  f32x16 acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;
  const bool two = rt.row_count > 32;   // tiles of at most 32 rows leave out the second half
  const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};

  if (kt0 < kt1) {
    if (K >= 4) {
      fetch(kt0);
    } else {   // rows of 1 to 3 elements
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          fa[i][e] = a_ptr[i][min(e, K - 1)];
          fb[i][e] = ((i < 2 ? b_lo : b_hi) + b_off[i])[min(e, K - 1)];
        }
    }
  }
  for (int kt = kt0; kt < kt1; ++kt) {
    if (kt * kBK + kBK > K) cut_tail(kt);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      *reinterpret_cast<f32x4*>(stage + wr + i * 16 * kRowBytes) = fa[i];
      *reinterpret_cast<f32x4*>(stage + wr + (kBM + i * 16) * kRowBytes) = fb[i];
    }
    // the LDS of a wavefront executes in program order; the fence keeps the compiler to it
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    if (kt + 1 < kt1) fetch(kt + 1);
    // Lane (r32, q) holds chunk 2 c + q of its row: MFMA j of pair c consumes element j, i.e. the
    // elements 8 c + j and 8 c + 4 + j of the k-tile, the same ones on both sides.
    f32x4 a[2][2], b[2][2];
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      const int slot = ((2 * c + q) ^ key) * 16;
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        a[s][c] = *reinterpret_cast<const f32x4*>(stage + (s * 32 + r32) * kRowBytes + slot);
        b[s][c] = *reinterpret_cast<const f32x4*>(stage + (kBM + s * 32 + r32) * kRowBytes + slot);
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    auto multiply = [&](int i) {
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        f32x16 part[4];
#pragma unroll
        for (int u = 0; u < 4; ++u)
          part[u] = __builtin_amdgcn_mfma_f32_32x32x2f32(b[j][u >> 1][2 * (u & 1)], a[i][u >> 1][2 * (u & 1)], zero, 0, 0, 0);
#pragma unroll
        for (int u = 0; u < 4; ++u)
          part[u] = __builtin_amdgcn_mfma_f32_32x32x2f32(b[j][u >> 1][2 * (u & 1) + 1], a[i][u >> 1][2 * (u & 1) + 1],
                                                         part[u], 0, 0, 0);
        acc[i][j] += (part[0] + part[1]) + (part[2] + part[3]);
        // one accumulator at a time: its partial sums take 64 registers until they are added
        asm volatile("" : "+v"(acc[i][j]));
      }
    };
    multiply(0);
    if (two) multiply(1);
  }

  // ---- the eighths as a tree: 4..7 into 0..3 through LDS, then the four tiles by all threads ----
  // Register v of lane (r32, q): row r32 of the row half, column 8 (v / 4) + 4 q + v % 4.
  float* const slot = smem + (wave & 3) * kRedFloats + r32 * kRedPitch + q * 4;
  auto each_quad = [&](auto&& fn) {
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int vg = 0; vg < 4; ++vg)
          fn(reinterpret_cast<f32x4*>(slot + i * 32 * kRedPitch + j * 32 + vg * 8), acc[i][j], vg);
  };
  auto put = [](f32x4* d, f32x16& s, int vg) { *d = f32x4{s[vg * 4], s[vg * 4 + 1], s[vg * 4 + 2], s[vg * 4 + 3]}; };
  __syncthreads();
  if (wave >= 4) each_quad(put);
  __syncthreads();
  if (wave < 4)
    each_quad([](f32x4* d, f32x16& s, int vg) {
      const f32x4 o = *d;
#pragma unroll
      for (int e = 0; e < 4; ++e) s[vg * 4 + e] += o[e];
    });
  __syncthreads();
  if (wave < 4) each_quad(put);
  __syncthreads();

  const int row = threadIdx.x >> 3, c4 = (threadIdx.x & 7) * 4;
  if (row >= rt.row_count) return;
  auto total = [&](int col) {
    f32x4 t[4];
#pragma unroll
    for (int w = 0; w < 4; ++w) t[w] = *reinterpret_cast<const f32x4*>(smem + w * kRedFloats + row * kRedPitch + col);
    return (t[0] + t[2]) + (t[1] + t[3]);
  };
  float* const out = (GATED ? p.h : p.y) + (size_t)(rt.row_start + row) * N;
  auto store = [&](int n, const f32x4& v) {
    if (n + 4 <= N) {
      *reinterpret_cast<f32x4u*>(out + n) = v;
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (n + e < N) out[n + e] = v[e];
    }
  };
  if (GATED) {
    const f32x4 ag = total(c4), au = total(c4 + kBN / 2);
    f32x4 o;
#pragma unroll
    for (int e = 0; e < 4; ++e) o[e] = (ag[e] / (1.0f + expf(-ag[e]))) * au[e];
    store(ct * kCols + c4, o);
  } else {
    store(ct * kCols + c4, total(c4));
    store(ct * kCols + c4 + kBN / 2, total(c4 + kBN / 2));
  }
}

template <bool GATED>
prism_status launch_f32_gemm(const F32Args& a, hipStream_t st) {
  const int A = a.T * a.top_k;
  // row tiles there can be: a full one per 64 assignments, and one that is not per expert with rows
  const long long row_tiles = (long long)A / kBM + std::min(a.E, A) + (long long)a.S * ceil_div(a.T, kBM);
  const long long items = row_tiles * ceil_div(GATED ? a.F : a.H, GATED ? kBN / 2 : kBN);
  // One dimension of a grid may hold fewer than 2^32 threads: beyond kMaxGridX workgroups they stand in
  // several rows of equal length.  (2^31 items, each for up to 64 x 32 elements of h, are beyond any memory.)
  if (items >= 0x7FFF0000LL) return PRISM_ERR_UNSUPPORTED;
  const unsigned down = (unsigned)((items + kMaxGridX - 1) / kMaxGridX);
  const unsigned across = (unsigned)align_up((size_t)((items + down - 1) / down), kXcds);
  static LdsLimitOnce lds_limit;   // one per instantiation
  if (!raise_lds_limit(lds_limit, (const void*)ffn_f32_kernel<GATED>, kLdsBytes)) return PRISM_ERR_LAUNCH;
  hipLaunchKernelGGL(ffn_f32_kernel<GATED>, dim3(across, down), dim3(kThreads), kLdsBytes, st, a,
                     (int)row_tiles, (int)items);
  PRISM_CHECK_LAUNCH();
  return PRISM_OK;
}

}  // namespace

prism_status launch_expert_ffn_f32(const prism_layer_desc& d, const void* x, const prism_expert_weights& w,
                                   const int32_t* local_src, const int32_t* local_offsets, int T, void* y,
                                   void* h, hipStream_t st, void* const* stage_events) {
  if (d.weight_layout != PRISM_WEIGHTS_ROW_MAJOR) return PRISM_ERR_UNSUPPORTED;
  if ((size_t)d.hidden * 4 > 64 * 1024 || (size_t)d.ffn * 4 > 64 * 1024) return PRISM_ERR_UNSUPPORTED;
  const F32Args a{(const float*)x, w.w_gate, w.w_up, w.w_down, w.shared_w_gate, w.shared_w_up,
                  w.shared_w_down, local_src, local_offsets, (float*)h, (float*)y,
                  T, d.hidden, d.ffn, d.n_experts, d.n_shared, d.top_k};
  trace(stage_events, PRISM_STAGE_FFN_UP, 0, st);
  PRISM_TRY(launch_f32_gemm<true>(a, st));
  trace(stage_events, PRISM_STAGE_FFN_UP, 1, st);
  trace(stage_events, PRISM_STAGE_FFN_DOWN, 0, st);
  PRISM_TRY(launch_f32_gemm<false>(a, st));
  trace(stage_events, PRISM_STAGE_FFN_DOWN, 1, st);
  return PRISM_OK;
}

}  // namespace prism
