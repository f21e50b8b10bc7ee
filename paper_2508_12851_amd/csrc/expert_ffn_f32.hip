// Grouped SwiGLU expert FFN of fp32 layers (paper Sec. III-A) on the fp32 matrix cores.
//
//   GATED   h[r, f] = silu( x[tok(r)] . W_gate^e[f] ) * ( x[tok(r)] . W_up^e[f] )
//   plain   y[r, n] = h[r] . W_down^e[n]
//
// Bound: the matrix cores.  In fp32 (v_mfma_f32_32x32x2_f32) they do 157 TFLOP/s nominal, in bf16 sixteen
// times that, so every fp32 operand is taken as the sum of three bf16 parts of 8 bits and a product as the six
// products of parts that reach 2^-24 of it (three of the nine are left out, 2^-26 and below).
//
// Split: a workgroup owns 64 rows of one expert x 64 weight rows (GATED: 32 gate rows and the 32 up
// rows of the same f), and its 8 wavefronts split the contraction: each multiplies its own eighth in
// 16-wide k-tiles that it stages through 8 KiB of LDS of its own, so the k-loop has no workgroup
// barrier, and a tile of even the smallest layer is spread over all four SIMDs (one workgroup, two
// wavefronts per SIMD).  The next k-tile travels from memory to registers during the products of this one (24
// MFMAs of 32 clocks and about as much conversion, which the SIMD's other wavefront overlaps).  The workgroups are
// persistent: the first operands of the next item are asked for before the sums of this one.
//
// Sums: fp32 results must not get worse than those of fp32 products.  The leading parts' products
// have accumulators of their own (16 terms per rounding, chains of K / 128), the other five products, 2^-8 and
// below, share a second set, and the eighths are added as a tree.  Relative 2-norm of the FFN's error against
// 64 bits, N(0, 1) tokens, H x F: 256 x 512 1.27e-7 (in fp32 1.50e-7), 1024 x 2048 1.72e-7 (1.78e-7), 2048 x 1024
// 1.79e-7 (1.86e-7), 4096 x 512 2.18e-7 (2.10e-7): contractions beyond 2048 stay in fp32, and so does a
// wavefront's eighth whose sums are not finite, because an infinity has no parts.
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

constexpr int kBM = 64;                  // most rows of a tile
constexpr float kHalfTile = 0.85f;       // time of a tile of 32 rows, in tiles of 64
constexpr int kBN = 64;                  // weight rows of a tile
constexpr int kBK = 16;                  // contraction elements per k-tile
constexpr int kWaves = 8;
constexpr int kThreads = kWaves * kWave;
constexpr int kXcds = 8;
constexpr int kWorkgroups = 256;         // persistent: one per CU
constexpr int kSplitMaxK = 2048;         // longest contraction multiplied in bf16 parts
constexpr int kRowBytes = kBK * 4;
constexpr int kStageBytes = (kBM + kBN) * kRowBytes;         // one wavefront's k-tile
constexpr int kRedPitch = kBN + 4;                           // floats; rows start in different banks
constexpr int kRedFloats = kBM * kRedPitch;                  // one wavefront's partial tile
constexpr int kLdsBytes = kWaves * kStageBytes + kWaves / 2 * kRedFloats * 4;   // k-tiles, partial tiles
static_assert(kLdsBytes <= 160 * 1024, "LDS per workgroup");

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

// The row tiles: those of the routed experts in expert order, then those of the shared ones.  Every
// wavefront holds the offsets of four experts per lane and finds a tile by its number with a ballot.
// All are 64 or all are 32 rows high, whichever takes less time by the rounds of items it makes of the launch's
// workgroups: 887 rows of 5 experts x 16 column tiles are 272 items of 64 rows, two rounds on 256 workgroups, and
// 496 of 32, also two (down projection of 2048 x 1024, 62 -> 52 us); 64 tokens make one round of either, and lower tiles
// spread the work further (layer of 256 x 512: 36.9 -> 34.6 us).
struct RowTiles {
  int off[5];      // offsets of experts 4 lane .. 4 lane + 4
  int before;      // row tiles of the experts before lane's
  int routed;      // row tiles of all routed experts
  int shift;       // 2^shift rows per tile
};
__device__ __forceinline__ int tiles_of(int rows, int shift) { return (rows + (1 << shift) - 1) >> shift; }
__device__ __forceinline__ RowTiles load_row_tiles(const F32Args& p, int n_col_tiles) {
  const int lane = threadIdx.x & 63;
  RowTiles r;
#pragma unroll
  for (int j = 0; j < 5; ++j) r.off[j] = p.local_offsets[min(4 * lane + j, p.E)];
  float best = INFINITY;
#pragma unroll
  for (int shift = 6; shift >= 5; --shift) {
    int tiles = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) tiles += tiles_of(r.off[j + 1] - r.off[j], shift);
    const int incl = wave_inclusive_scan(tiles);
    const int routed = __builtin_amdgcn_readlane(incl, 63);
    const float items = (float)(routed + p.S * tiles_of(p.T, shift)) * (float)n_col_tiles;
    const float time = ceilf(items / (float)gridDim.x) * (shift == 6 ? 1.f : kHalfTile);
    if (time < best) {
      best = time;
      r.before = incl - tiles;
      r.routed = routed;
      r.shift = shift;
    }
  }
  return r;
}
__device__ __forceinline__ RowTile row_tile(const F32Args& p, const RowTiles& r, int b) {
  if (b < r.routed) {
    int rel = b - r.before, e = 0, start = 0, count = 0;
    bool mine = false;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int t = tiles_of(r.off[j + 1] - r.off[j], r.shift);
      if (rel >= 0 && rel < t) {
        mine = true;
        e = 4 * (threadIdx.x & 63) + j;
        start = r.off[j] + (rel << r.shift);
        count = min(1 << r.shift, r.off[j + 1] - start);
      }
      rel -= t;
    }
    const int owner = __ffsll((unsigned long long)__ballot(mine)) - 1;
    return RowTile{__builtin_amdgcn_readlane(e, owner), __builtin_amdgcn_readlane(start, owner),
                   __builtin_amdgcn_readlane(count, owner), -1};
  }
  const int per_shared = tiles_of(p.T, r.shift), s = (b - r.routed) / per_shared, tok = (b - r.routed - s * per_shared) << r.shift;
  return RowTile{p.E + s, p.T * (p.top_k + s) + tok, min(1 << r.shift, p.T - tok), tok};
}

// An fp32 value is the sum of three bf16 values: the nearest one, the nearest one to what is left, and
// the rest, whose 24 - 8 - 8 bits fit (exact unless the value is below 2^-110 or overflows when rounded).  The
// differences come from a dot product with (-1, 0) or (0, -1), one instruction instead of unpacking
// a half and subtracting it.  (From registers: the compiler's inline constant for (0, -1) is not that pair.)
struct Parts {
  bf16x8 v[3];
};
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ void split_pair(float a, float b, uint32_t minus_lo, uint32_t minus_hi, uint32_t (&o)[3]) {
  float r[2] = {a, b};
#pragma unroll
  for (int u = 0; u < 3; ++u) {
    const bf16x2 h = {(bf16_t)r[0], (bf16_t)r[1]};
    o[u] = __builtin_bit_cast(uint32_t, h);
    if (u < 2) {
      r[0] = __builtin_amdgcn_fdot2_f32_bf16(h, __builtin_bit_cast(bf16x2, minus_lo), r[0], false);
      r[1] = __builtin_amdgcn_fdot2_f32_bf16(h, __builtin_bit_cast(bf16x2, minus_hi), r[1], false);
    }
  }
}

template <bool GATED>
__global__ __launch_bounds__(kThreads) void ffn_f32_kernel(const F32Args p) {
#if defined(__HIP_DEVICE_COMPILE__)   // the bf16 dot product exists in device code only
  extern __shared__ __align__(16) float smem[];
  const int K = GATED ? p.H : p.F, N = GATED ? p.F : p.H;
  constexpr int kCols = GATED ? kBN / 2 : kBN;      // output columns of the tile
  // Consecutive workgroups go to the 8 XCDs in turn; every XCD takes a contiguous eighth of the
  // items, row tiles running fastest, so that the row tiles of an expert read its weight rows
  // through one L2.
  const int n_col_tiles = (N + kCols - 1) / kCols;
  const RowTiles tiles = load_row_tiles(p, n_col_tiles);
  const int n_row_tiles = tiles.routed + p.S * tiles_of(p.T, tiles.shift);
  const int n_items = n_row_tiles * n_col_tiles;
  const int xcd = blockIdx.x % kXcds, slots = gridDim.x / kXcds;
  const int item_end = (int)((long long)n_items * (xcd + 1) / kXcds);
  int item = (int)((long long)n_items * xcd / kXcds) + blockIdx.x / kXcds;
  if (item >= item_end) return;

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int r32 = lane & 31, q = lane >> 5;

  // ---- global -> LDS assignment: lane l brings chunk l % 4 (4 elements) of rows l / 4 + 16 i ----
  const int lrow = lane >> 2, chunk = lane & 3;
  const float* a_ptr[4];
  uint32_t b_off[4];      // elements (H and F are at most 16384)
  global_ptr b_lo, b_hi;  // weight rows 0 .. 31 and 32 .. 63
  // What an item needs from memory before its first operand can be fetched.
  struct Item {
    RowTile rt;
    int ct;
    int src[4];                  // GATED, routed: entries of local_src of this lane's rows
    const void* lo;
    const void* hi;
  };
  auto find_item = [&](int it) {
    Item n;
    n.ct = it / n_row_tiles;
    n.rt = row_tile(p, tiles, it - n.ct * n_row_tiles);
    const bool routed = n.rt.g < p.E;
    const int gi = routed ? n.rt.g : n.rt.g - p.E;
    n.lo = GATED ? (routed ? p.wg[gi] : p.swg[gi]) : (routed ? p.wd[gi] : p.swd[gi]);
    n.hi = GATED ? (routed ? p.wu[gi] : p.swu[gi]) : n.lo;
#pragma unroll
    for (int i = 0; i < 4; ++i)
      n.src[i] = GATED && routed ? p.local_src[n.rt.row_start + min(lrow + 16 * i, n.rt.row_count - 1)] : 0;
    return n;
  };
  auto set_addresses = [&](const Item& n) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int br = lrow + 16 * i;
      const int rr = min(br, n.rt.row_count - 1);   // rows past the end repeat the last one
      if (GATED)
        a_ptr[i] = p.x + (size_t)(n.rt.g < p.E ? n.src[i] / p.top_k : n.rt.tok_base + rr) * K;
      else
        a_ptr[i] = p.h + (size_t)(n.rt.row_start + rr) * K;
      b_off[i] = (uint32_t)min(n.ct * kCols + br % kCols, N - 1) * (uint32_t)K;
    }
    b_lo = (global_ptr)n.lo;
    b_hi = (global_ptr)n.hi;
  };

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
  auto fetch_first = [&] {
    if (kt0 >= kt1) return;
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
  // puts the k-tile that was fetched into LDS and asks for the next one
  auto next_k_tile = [&](int kt) {
    if (kt * kBK + kBK > K) cut_tail(kt);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      *reinterpret_cast<f32x4*>(stage + wr + i * 16 * kRowBytes) = fa[i];
      *reinterpret_cast<f32x4*>(stage + wr + (kBM + i * 16) * kRowBytes) = fb[i];
    }
    // the LDS of a wavefront executes in program order; the fence keeps the compiler to it
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    if (kt + 1 < kt1) fetch(kt + 1);
  };
  // Lane (r32, q) holds chunks q and 2 + q of its row, the same elements on both sides.
  auto read_chunk = [&](int row, int c) {
    return *reinterpret_cast<const f32x4*>(stage + row * kRowBytes + ((2 * c + q) ^ key) * 16);
  };
  uint32_t minus_lo = 0x0000BF80u, minus_hi = 0xBF800000u;   // (-1, 0) and (0, -1)
  asm volatile("" : "+s"(minus_lo), "+s"(minus_hi));
  auto read_parts = [&](int row) {
    u32x4 w[3];
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      const f32x4 v = read_chunk(row, c);
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        uint32_t o[3];
        split_pair(v[2 * e], v[2 * e + 1], minus_lo, minus_hi, o);
#pragma unroll
        for (int u = 0; u < 3; ++u) w[u][2 * c + e] = o[u];
      }
    }
    return Parts{{__builtin_bit_cast(bf16x8, w[0]), __builtin_bit_cast(bf16x8, w[1]), __builtin_bit_cast(bf16x8, w[2])}};
  };

  f32x16 acc[2][2];
  const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  // The products as six bf16 ones, the leading part's in sums of their own.  Tiles of at most 32 rows (two: false)
  // leave out the second half.
  auto multiply_parts = [&](bool two) {
    f32x16 low[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j) acc[i][j] = low[i][j] = zero;
    for (int kt = kt0; kt < kt1; ++kt) {
      next_k_tile(kt);
      const Parts b[2] = {read_parts(kBM + r32), read_parts(kBM + 32 + r32)};
      auto half = [&](int i) {
        const Parts a = read_parts(i * 32 + r32);
        auto mul = [&](f32x16 (&d)[2], int u, int w) {
#pragma unroll
          for (int j = 0; j < 2; ++j) d[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(b[j].v[w], a.v[u], d[j], 0, 0, 0);
        };
        mul(low[i], 2, 0);
        mul(acc[i], 0, 0);
        mul(low[i], 1, 1);
        mul(low[i], 0, 2);
        mul(low[i], 1, 0);
        mul(low[i], 0, 1);
      };
      half(0);
      if (two) half(1);
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    }
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j) acc[i][j] += low[i][j];
  };
  // The products on the fp32 matrix cores: pairs, the pairs of a k-tile as a tree.  MFMA j of chunk pair c
  // consumes element j, i.e. the elements 8 c + j and 8 c + 4 + j of the k-tile.
  auto multiply_f32 = [&](bool two) {
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j) acc[i][j] = zero;
    fetch_first();
    for (int kt = kt0; kt < kt1; ++kt) {
      next_k_tile(kt);
      f32x4 a[2][2], b[2][2];
#pragma unroll
      for (int c = 0; c < 2; ++c)
#pragma unroll
        for (int s = 0; s < 2; ++s) {
          a[s][c] = read_chunk(s * 32 + r32, c);
          b[s][c] = read_chunk(kBM + s * 32 + r32, c);
        }
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      auto half = [&](int i) {
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
      half(0);
      if (two) half(1);
    }
  };
  auto all_finite = [&] {
    float z = 0.f;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int v = 0; v < 16; ++v) z = fmaf(acc[i][j][v], 0.f, z);
    return __ballot(z != 0.f) == 0;   // (a NaN is not equal to zero)
  };

  // Register v of lane (r32, q): row r32 of the row half, column 8 (v / 4) + 4 q + v % 4.
  float* const red = smem + kWaves * kStageBytes / 4;
  float* const slot = red + (wave & 3) * kRedFloats + r32 * kRedPitch + q * 4;
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

  Item cur = find_item(item);
  set_addresses(cur);
  fetch_first();
  while (true) {
    const bool has_next = item + slots < item_end;
    item += slots;
    const Item next = find_item(has_next ? item : item - slots);   // asked for before the products
    const RowTile rt = cur.rt;
    const int ct = cur.ct;
    const bool two = rt.row_count > 32;
    bool in_f32 = K > kSplitMaxK;
    if (!in_f32) {
      multiply_parts(two);
      // an infinity or NaN is no sum of three parts, nor is a value that rounds up to infinity: once more in fp32
      in_f32 = !all_finite();
    }
    if (in_f32) multiply_f32(two);
    if (has_next) {   // the next item's first k-tile travels during the sums of this one
      set_addresses(next);
      fetch_first();
    }

    // ---- the eighths as a tree: 4..7 into 0..3 through LDS, then the four tiles by all threads ----
    lds_barrier();   // the item before has been read
    if (wave >= 4) each_quad(put);
    lds_barrier();
    if (wave < 4)
      each_quad([](f32x4* d, f32x16& s, int vg) {
        const f32x4 o = *d;
#pragma unroll
        for (int e = 0; e < 4; ++e) s[vg * 4 + e] += o[e];
        *d = f32x4{s[vg * 4], s[vg * 4 + 1], s[vg * 4 + 2], s[vg * 4 + 3]};
      });
    lds_barrier();

    const int row = threadIdx.x >> 3, c4 = (threadIdx.x & 7) * 4;
    if (row < rt.row_count) {
      auto total = [&](int col) {
        f32x4 t[4];
#pragma unroll
        for (int w = 0; w < 4; ++w) t[w] = *reinterpret_cast<const f32x4*>(red + w * kRedFloats + row * kRedPitch + col);
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
    if (!has_next) break;
    cur = next;
  }
#endif
}

template <bool GATED>
prism_status launch_f32_gemm(const F32Args& a, hipStream_t st) {
  const int A = a.T * a.top_k;
  // items there can be, in tiles of 2^shift rows: a full row tile per 2^shift assignments, and one that is not per
  // expert with rows
  auto items = [&](int shift) {
    const long long row_tiles = ((long long)A >> shift) + std::min(a.E, A) + (long long)a.S * ceil_div(a.T, 1 << shift);
    return row_tiles * ceil_div(GATED ? a.F : a.H, GATED ? kBN / 2 : kBN);
  };
  // (2^31 items of 64 rows, each for up to 64 x 32 elements of h, are beyond any memory)
  if (items(6) >= 0x7FFF0000LL) return PRISM_ERR_UNSUPPORTED;
  static LdsLimitOnce lds_limit;   // one per instantiation
  if (!raise_lds_limit(lds_limit, (const void*)ffn_f32_kernel<GATED>, kLdsBytes)) return PRISM_ERR_LAUNCH;
  // one workgroup fits a CU
  hipLaunchKernelGGL(ffn_f32_kernel<GATED>, dim3((unsigned)std::min<long long>(kWorkgroups, align_up((size_t)items(5), kXcds))),
                     dim3(kThreads), kLdsBytes, st, a);
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
