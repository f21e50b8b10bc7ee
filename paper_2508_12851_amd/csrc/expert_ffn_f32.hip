// Grouped SwiGLU expert FFN of fp32 layers (paper Sec. III-A) on the fp32 matrix cores.
//
//   GATED   h[r, f] = silu( x[tok(r)] . W_gate^e[f] ) * ( x[tok(r)] . W_up^e[f] )
//   plain   y[r, n] = h[r] . W_down^e[n]
//
// Bound: the matrix cores.  In fp32 (v_mfma_f32_32x32x2_f32) they do 157 TFLOP/s nominal, in bf16 sixteen
// times that, so every fp32 operand is taken as the sum of three bf16 parts of 8 bits and a product as the eight
// products of parts that reach 2^-25 of it.  (The parts are at most 1, 2^-8 and 2^-17 of the value; the ninth product, of the two
// smallest ones, is at most 2^-34.)
//
// Split: a workgroup owns 64 rows of one expert x 64 weight rows (GATED: 32 gate rows and the 32 up
// rows of the same f), and its 8 wavefronts split the contraction: each multiplies its own eighth in
// 16-wide k-tiles that it stages through 8 KiB of LDS of its own, so the k-loop has no workgroup
// barrier, and a tile of even the smallest layer is spread over all four SIMDs (one workgroup, two
// wavefronts per SIMD).  The next k-tile travels from memory to registers during the products of this one (32
// MFMAs of 32 clocks and about as much conversion, which the SIMD's other wavefront overlaps).  The workgroups are
// persistent: the first operands of the next item are asked for before the sums of this one.
//
// Sums: fp32 results must not get worse than those of fp32 products.  A v_mfma_f32_32x32x16_bf16 adds its first 8 products
// to the accumulator, rounds, adds the other 8, rounds, and of an accumulator smaller than its products it drops
// bits.  So the leading parts' products of a k-tile start from zero and are added to the sum of the wavefront by the
// vector ALU (K / 128 roundings of that sum, as with fp32 products), the other seven products, 2^-8 and below, stay in
// sums of their own to the end, and of the eighths only pairs are added in fp32, the rest in fp64.  Relative 2-norm of the
// FFN's error against 64 bits, with fp32 products (tree of eighths in fp32) -> here, H x F:
//   N(0, 1)                   256 x 512 1.50e-7 -> 1.15e-7, 1024 x 2048 1.77e-7 -> 1.48e-7, 2048 x 1024 1.86e-7 -> 1.56e-7
//   uniform in [0, 1)         256 x 512 4.70e-8 -> 4.01e-8, 1024 x 2048 5.11e-8 -> 4.53e-8, 2048 x 1024 4.94e-8 -> 4.26e-8
//   8 nonzeros per row        256 x 512 1.16e-7 -> 0.96e-7, 1024 x 2048 1.11e-7 -> 0.90e-7, 2048 x 1024 1.11e-7 -> 0.90e-7
//   one nonzero per row       256 x 512 6.74e-8 -> 6.74e-8, 1024 x 2048 6.69e-8 -> 6.68e-8, 2048 x 1024 6.84e-8 -> 6.85e-8
//   N(0, 1) exp(N(0, 1))      256 x 512 1.51e-7 -> 1.31e-7, 1024 x 2048 1.75e-7 -> 1.62e-7, 2048 x 1024 1.85e-7 -> 1.72e-7
//   N(0, 1) exp(2 N(0, 1))    256 x 512 1.49e-7 -> 1.49e-7, 1024 x 2048 1.75e-7 -> 1.77e-7, 2048 x 1024 1.83e-7 -> 1.87e-7
// Longer contractions would add up more low products and stay in fp32 (LONG).  What has no parts, infinities and very small
// values, is looked at again (see "Small values").
//
// FFN of fp32 products as one launch of a workgroup per item -> here, us: 500 tokens, 1024 x 2048, 5 of 8 experts hosted 160 -> 124
// (six products, and leading sums kept in the matrix cores: 102), every tenth token zero 160 -> 138; 256 x 512, 64 tokens
// 18.2 -> 18.4; LONG, 2056 x 2056, 200
// tokens 154 -> 137, 4096 x 4096, 4 / 500 tokens 169 / 784 -> 173 / 715.
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
// Time of a tile of 32 rows, in tiles of 64.  In parts, whose conversions of weights stay: 0.6 / 0.85 FFN of 500 tokens, 1024 x
// 2048, 127 / 118 us.  In fp32, where half the MFMAs go: 2056 x 2056, 200 tokens 137 / 151, 500 tokens 232 / 243.
constexpr float kHalfTile = 0.85f, kHalfTileF32 = 0.6f;
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
constexpr int kTileBytes = kWaves * kRedFloats * 4;
// Marks: two bits per item of a workgroup (from the start again after 512): its sums need a closer look, or do if some
// operand is very small.  Two words more: any mark, and whether the second walk has seen such an operand.
constexpr int kMarkWords = 32;
constexpr uint32_t kLook = 1, kLookIfSmall = 2;
constexpr int kControlWords = kMarkWords + 2;
constexpr int kLdsBytes = kTileBytes + kControlWords * 4 + (PRISM_MAX_EXPERTS + 1) * 4;
static_assert(kRedFloats * 4 >= kStageBytes && kLdsBytes <= 160 * 1024, "a partial tile replaces its wavefront's k-tile");
// Which sums of products of parts are good (see "Small values"): of operands up to kPlainMax those from kPlainMin on, otherwise those
// beyond kLossPerOperand (A + B) + kLossFloor.
constexpr float kPlainMax = 0x1p30f, kPlainMin = 0x1p-60f;
constexpr float kLossPerOperand = 0x1p-99f, kLossFloor = 0x1p-116f;
constexpr float kExactFrom = 0x1p-110f;  // elements that are the sum of their parts, zeros aside

// Rows of fp32 matrices start at any multiple of 4 bytes (F need not be a multiple of 4).
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));
// Pointers that come out of a table in memory: said to be global memory, which the compiler cannot know.
typedef const __attribute__((address_space(1))) float* global_ptr;
typedef const __attribute__((address_space(1))) f32x4u* global_ptr4;

// Entry i, the same in all lanes, of a table of weight pointers, which no kernel writes: a scalar load.
__device__ __forceinline__ global_ptr table_entry(const void* const* table, int i) {
  typedef const __attribute__((address_space(4))) uint64_t* const_table;
  return (global_ptr)((const_table)(uint64_t)table)[__builtin_amdgcn_readfirstlane(i)];
}

struct RowTile {
  int g;           // expert (g < E), shared expert E + s, or -1: nothing here
  int row_start;   // first row in h / y
  int row_count;
  int tok_base;    // shared experts: token of the first row; routed ones: -1
};

// The row tiles: those of the routed experts in expert order, then those of the shared ones.  A lane
// stands for four experts, and a wavefront finds a tile by its number with a ballot.
// All are 64 or all are 32 rows high, whichever takes less time by the rounds of items it makes of the launch's
// workgroups (half_tile: time of a lower one): 887 rows of 5 experts x 16 column tiles are 272 items of 64 rows, two rounds on 256 workgroups, and
// 496 of 32, also two (down projection of 2048 x 1024, 62 -> 52 us); 64 tokens make one round of either, and lower tiles
// spread the work further (layer of 256 x 512: 36.9 -> 34.6 us).
struct RowTiles {
  const int* off;  // LDS: offsets of experts 4 lane .. 4 lane + 4
  int before;      // row tiles of the experts before lane's
  int routed;      // row tiles of all routed experts
  int shift;       // 2^shift rows per tile
};
__device__ __forceinline__ int tiles_of(int rows, int shift) { return (rows + (1 << shift) - 1) >> shift; }
__device__ __forceinline__ RowTiles load_row_tiles(const F32Args& p, int n_col_tiles, float half_tile, int tid, const int* s_off) {
  RowTiles r;
  r.off = s_off + 4 * (tid & 63);
  float best = INFINITY;
#pragma unroll
  for (int shift = 6; shift >= 5; --shift) {
    int tiles = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) tiles += tiles_of(r.off[j + 1] - r.off[j], shift);
    const int incl = wave_inclusive_scan(tiles);
    const int routed = __builtin_amdgcn_readlane(incl, 63);
    const float items = (float)(routed + p.S * tiles_of(p.T, shift)) * (float)n_col_tiles;
    const float time = ceilf(items / (float)gridDim.x) * (shift == 6 ? 1.f : half_tile);
    if (time < best) {
      best = time;
      r.before = incl - tiles;
      r.routed = routed;
      r.shift = shift;
    }
  }
  return r;
}
__device__ __forceinline__ RowTile row_tile(const F32Args& p, const RowTiles& r, int tid, int b) {
  if (b < r.routed) {
    int rel = b - r.before, e = 0, start = 0, count = 0;
    bool mine = false;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int t = tiles_of(r.off[j + 1] - r.off[j], r.shift);
      if (rel >= 0 && rel < t) {
        mine = true;
        e = 4 * (tid & 63) + j;
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

#if defined(__HIP_DEVICE_COMPILE__)   // the bf16 dot product exists in device code only
// A workgroup's walk over its items.  LONG: products in fp32.  AGAIN: only the marked items, with a closer look at their
// sums (see "Small values").  That is a walk of its own, with registers of its own: inside the first one its code made the
// smallest FFN 20.1 us instead of 18.2, and 4 us of the larger ones.
template <bool GATED, bool LONG, bool AGAIN>
__device__ __forceinline__ void walk_items(const F32Args& p, float* const smem, const int tid) {
  uint32_t* const marks = reinterpret_cast<uint32_t*>(smem) + kTileBytes / 4;
  const int K = GATED ? p.H : p.F, N = GATED ? p.F : p.H;
  constexpr int kCols = GATED ? kBN / 2 : kBN;      // output columns of the tile
  // Consecutive workgroups go to the 8 XCDs in turn; every XCD takes a contiguous eighth of the
  // items, row tiles running fastest, so that the row tiles of an expert read its weight rows
  // through one L2.
  const int n_col_tiles = (N + kCols - 1) / kCols;
  const RowTiles tiles = load_row_tiles(p, n_col_tiles, LONG ? kHalfTileF32 : kHalfTile, tid, reinterpret_cast<int*>(marks) + kControlWords);
  const int n_row_tiles = tiles.routed + p.S * tiles_of(p.T, tiles.shift);
  const int n_items = n_row_tiles * n_col_tiles;
  const int xcd = blockIdx.x % kXcds, slots = gridDim.x / kXcds;
  const int item_end = (int)((long long)n_items * (xcd + 1) / kXcds);
  int item = (int)((long long)n_items * xcd / kXcds) + blockIdx.x / kXcds;
  if (item >= item_end) return;

  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r32 = lane & 31, q = lane >> 5;

  // ---- global -> LDS assignment: lane l brings chunk l % 4 (4 elements) of rows l / 4 + 16 i ----
  const int lrow = lane >> 2, chunk = lane & 3;
  uint32_t a_row[4];      // rows of x or h
  uint32_t b_off[4];      // elements (H and F are at most 16384)
  global_ptr b_lo, b_hi;  // weight rows 0 .. 31 and 32 .. 63
  // What an item needs from memory before its first operand can be fetched.
  struct Item {
    RowTile rt;
    int ct;
    int src[4];                  // GATED, routed: entries of local_src of this lane's rows
    global_ptr lo, hi;           // weight rows 0 .. 31 and 32 .. 63
  };
  auto find_item = [&](int it) {
    Item n;
    n.ct = it / n_row_tiles;
    n.rt = row_tile(p, tiles, tid, it - n.ct * n_row_tiles);
    const bool routed = n.rt.g < p.E;
    const int gi = routed ? n.rt.g : n.rt.g - p.E;
    n.lo = table_entry(GATED ? (routed ? p.wg : p.swg) : (routed ? p.wd : p.swd), gi);
    n.hi = GATED ? table_entry(routed ? p.wu : p.swu, gi) : n.lo;
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
        a_row[i] = n.rt.g < p.E ? n.src[i] / p.top_k : n.rt.tok_base + rr;
      else
        a_row[i] = n.rt.row_start + rr;
      b_off[i] = (uint32_t)min(n.ct * kCols + br % kCols, N - 1) * (uint32_t)K;
    }
    b_lo = n.lo;
    b_hi = n.hi;
  };

  // this wavefront's k-tiles
  const int n_kt = (K + kBK - 1) / kBK;
  const int kt0 = (int)((long long)n_kt * wave / kWaves), kt1 = (int)((long long)n_kt * (wave + 1) / kWaves);
  f32x4 fa[4], fb[4];
  float largest;          // !LONG: magnitude of the elements this lane brought
  const float* const a_base = GATED ? p.x : p.h;
  // Element k = kt kBK + 4 chunk and the three after it, of every row this lane brings.  At the end
  // of the rows the last 4 elements come instead (cut_tail puts them right).
  auto fetch = [&](int kt) {
    const uint32_t k = (uint32_t)min(kt * kBK + chunk * 4, K - 4);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      fa[i] = *reinterpret_cast<const f32x4u*>(a_base + ((uint64_t)a_row[i] * (uint32_t)K + k));
      fb[i] = *(global_ptr4)((i < 2 ? b_lo : b_hi) + (b_off[i] + k));
    }
  };
  auto fetch_first = [&] {
    if (kt0 >= kt1) return;
    if (!LONG || K >= 4) {
      fetch(kt0);
    } else {   // rows of 1 to 3 elements
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          fa[i][e] = a_base[(uint64_t)a_row[i] * (uint32_t)K + min(e, K - 1)];
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
  uint8_t* const stage = reinterpret_cast<uint8_t*>(smem + wave * kRedFloats);   // (its partial tile replaces its k-tile)
  const int wr = lrow * kRowBytes + (chunk ^ ((lrow >> 2) & 3)) * 16;
  const int key = (r32 >> 2) & 3;
  // m: the largest magnitude so far
  auto grow = [](float& m, const f32x4& v) {
    asm("v_max3_f32 %0, %0, |%1|, |%2|\n\tv_max3_f32 %0, %0, |%3|, |%4|" : "+&v"(m) : "v"(v[0]), "v"(v[1]), "v"(v[2]), "v"(v[3]));
  };
  // puts the k-tile that was fetched into LDS and asks for the next one
  auto next_k_tile = [&](int kt, bool with_max) {
    if (kt * kBK + kBK > K) cut_tail(kt);
    if (with_max)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        grow(largest, fa[i]);
        grow(largest, fb[i]);
      }
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
  // The products as eight bf16 ones (see "Sums" above).  Tiles of at most 32 rows (two: false) leave out the second half.
  auto multiply_parts = [&](bool two) {
    f32x16 low[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j) acc[i][j] = low[i][j] = zero;
    largest = 0.f;
    for (int kt = kt0; kt < kt1; ++kt) {
      next_k_tile(kt, true);
      const Parts b[2] = {read_parts(kBM + r32), read_parts(kBM + 32 + r32)};
      auto half = [&](int i) {
        const Parts a = read_parts(i * 32 + r32);
        __builtin_amdgcn_sched_barrier(0);   // one block's products at a time: two leading sums at once would spill
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          auto mul = [&](const f32x16& c, int u, int w) { return __builtin_amdgcn_mfma_f32_32x32x16_bf16(b[j].v[w], a.v[u], c, 0, 0, 0); };
          f32x16 lead = mul(zero, 0, 0);
          f32x16& d = low[i][j];
          d = mul(d, 2, 1);
          d = mul(d, 1, 2);
          d = mul(d, 2, 0);
          d = mul(d, 1, 1);
          d = mul(d, 0, 2);
          d = mul(d, 1, 0);
          d = mul(d, 0, 1);
          acc[i][j] += lead;
          asm volatile("" : "+v"(acc[i][j]));
          __builtin_amdgcn_sched_barrier(0);
        }
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
  // acc += the products of a k-tile on the fp32 matrix cores: pairs, the pairs of a k-tile as a tree.  MFMA j of chunk
  // pair c consumes element j, i.e. the elements 8 c + j and 8 c + 4 + j of the k-tile.
  auto add_products = [&](const f32x4 (&a)[2], const f32x4 (&b)[2], f32x16& sum) {
    f32x16 part[4];
#pragma unroll
    for (int u = 0; u < 4; ++u)
      part[u] = __builtin_amdgcn_mfma_f32_32x32x2f32(b[u >> 1][2 * (u & 1)], a[u >> 1][2 * (u & 1)], zero, 0, 0, 0);
#pragma unroll
    for (int u = 0; u < 4; ++u)
      part[u] = __builtin_amdgcn_mfma_f32_32x32x2f32(b[u >> 1][2 * (u & 1) + 1], a[u >> 1][2 * (u & 1) + 1], part[u], 0, 0, 0);
    sum += (part[0] + part[1]) + (part[2] + part[3]);
    // one accumulator at a time: its partial sums take 64 registers until they are added
    asm volatile("" : "+v"(sum));
  };
  auto read_row = [&](int row, f32x4 (&v)[2]) {
#pragma unroll
    for (int c = 0; c < 2; ++c) v[c] = read_chunk(row, c);
  };
  auto multiply_f32 = [&](bool two) {
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j) acc[i][j] = zero;
    for (int kt = kt0; kt < kt1; ++kt) {
      next_k_tile(kt, false);
      f32x4 a[2][2], b[2][2];
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        read_row(s * 32 + r32, a[s]);
        read_row(kBM + s * 32 + r32, b[s]);
      }
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      auto half = [&](int i) {
#pragma unroll
        for (int j = 0; j < 2; ++j) add_products(a[i], b[j], acc[i][j]);
      };
      half(0);
      if (two) half(1);
    }
  };
  // Small values: the three parts of an element miss at most 2^-134 (the smallest bf16 value is 2^-133), nothing of one from
  // 2^-110 on.  A wavefront's sum of at most 2^9 products of a row whose largest element is A with a weight row whose largest is B
  // is off by at most 2^-125 (A + B) for that, and by 2^-142 for products below the smallest fp32 value.  A sum of more
  // than 2^26 times as much keeps what fp32 products would; the others, and those that are not finite, are taken from fp32
  // products.  Each sum is judged by its own value and operands, so that a result depends on nothing else in the tile.
  auto redo_sums = [&](bool two) {
    float a_max[4] = {0.f, 0.f, 0.f, 0.f}, b_max[4] = {0.f, 0.f, 0.f, 0.f};   // rows lrow + 16 i
    fetch_first();
    for (int kt = kt0; kt < kt1; ++kt) {
      if (kt * kBK + kBK > K) cut_tail(kt);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        grow(a_max[i], fa[i]);
        grow(b_max[i], fb[i]);
      }
      if (kt + 1 < kt1) fetch(kt + 1);
    }
    float ra[2], rb[2];   // rows s 32 + r32
    auto of_rows = [&](float (&m)[4], float (&o)[2]) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {   // a row is brought by four lanes
        m[i] = fmaxf(m[i], __shfl_xor(m[i], 1));
        m[i] = fmaxf(m[i], __shfl_xor(m[i], 2));
      }
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        const float lo = __shfl(m[2 * s], (r32 & 15) * 4), hi = __shfl(m[2 * s + 1], (r32 & 15) * 4);
        o[s] = r32 < 16 ? lo : hi;
      }
    };
    of_rows(a_max, ra);
    of_rows(b_max, rb);
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        uint32_t bad = 0;
        if (i == 0 || two)
#pragma unroll
          for (int v = 0; v < 16; ++v) {
            const float x = fabsf(acc[i][j][v]), c = __shfl(rb[j], 8 * (v / 4) + 4 * q + v % 4);
            // (a zero row gives zeros either way)
            const bool lost = x <= kLossPerOperand * (ra[i] + c) + kLossFloor && ra[i] > 0.f && c > 0.f;
            bad |= (uint32_t)(lost || !(x < INFINITY)) << v;
          }
        if (__ballot(bad != 0) == 0) continue;
        f32x16 sum = zero;
        fetch_first();
        for (int kt = kt0; kt < kt1; ++kt) {
          next_k_tile(kt, false);
          f32x4 a[2], b[2];
          read_row(i * 32 + r32, a);
          read_row(kBM + j * 32 + r32, b);
          __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
          add_products(a, b, sum);
        }
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[i][j][v] = (bad >> v) & 1 ? sum[v] : acc[i][j][v];
      }
  };
  // The smallest magnitude but zero, as twice its bits less one (a zero gives the largest number).
  auto shrink_nonzero = [](uint32_t& m, const float (&v)[2]) {
    m = min(m, min(2 * __builtin_bit_cast(uint32_t, v[0]) - 1, 2 * __builtin_bit_cast(uint32_t, v[1]) - 1));
  };
  auto below = [](uint32_t m, float limit) { return m < 2 * __builtin_bit_cast(uint32_t, limit) - 1; };
  // Whether some sum of this wavefront needs a closer look.  Mostly one comparison for all says no (a NaN stays one either
  // way); zeros are left to add_and_store.
  auto look = [&](bool two) {
    float small = INFINITY;
    auto each = [&](auto&& fn) {
#pragma unroll
      for (int j = 0; j < 2; ++j) {
#pragma unroll
        for (int v = 0; v < 16; v += 2) fn(acc[0][j][v], acc[0][j][v + 1]);
        if (two)
#pragma unroll
          for (int v = 0; v < 16; v += 2) fn(acc[1][j][v], acc[1][j][v + 1]);
      }
    };
    each([&](float x, float y) { asm("v_min3_f32 %0, %0, |%1|, |%2|" : "+v"(small) : "v"(x), "v"(y)); });
    if (__builtin_expect(__ballot(!(largest <= kPlainMax && small >= kPlainMin)) == 0, 1)) return false;
    uint32_t nonzero = ~0u;
    each([&](float x, float y) { shrink_nonzero(nonzero, {x, y}); });
    return __ballot(!(largest <= kPlainMax) || below(nonzero, kPlainMin)) != 0;
  };
  // Whether an element of this wavefront's k-tiles is below kExactFrom and not zero.
  auto any_small_element = [&] {
    uint32_t nonzero = ~0u;
    for (int kt = kt0; kt < kt1; ++kt) {   // (the first one has been fetched)
      if (kt * kBK + kBK > K) cut_tail(kt);
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int e = 0; e < 4; e += 2) {
          shrink_nonzero(nonzero, {fa[i][e], fa[i][e + 1]});
          shrink_nonzero(nonzero, {fb[i][e], fb[i][e + 1]});
        }
      if (kt + 1 < kt1) fetch(kt + 1);
    }
    return __ballot(below(nonzero, kExactFrom)) != 0;
  };

  int number = 0;   // of the item in this workgroup
  auto mark_word = [&] { return &marks[number / 16 % kMarkWords]; };
  auto mark = [&](uint32_t what) {
    atomicOr(mark_word(), what << (number % 16 * 2));
    marks[kMarkWords] = 1;
  };
  // Whether row `row` (the same in all lanes) of an item's activations has an element that is not zero.
  auto nonzero_row = [&](const RowTile& rt, int row) {
    const int r = rt.row_start + row;
    const int a = !GATED ? r : rt.g < p.E ? p.local_src[r] / p.top_k : rt.tok_base + row;
    const float* const x = a_base + (uint64_t)(uint32_t)a * (uint32_t)K;
    bool nonzero = false;
    for (int k0 = 0; k0 < K && !nonzero; k0 += 1024)
#pragma unroll
      for (int k = k0; k < k0 + 1024; k += 256) {   // (what is past the end comes again)
        const f32x4 v = *reinterpret_cast<const f32x4u*>(x + min(k + lane * 4, K - 4));
        nonzero |= __ballot(v[0] != 0.f || v[1] != 0.f || v[2] != 0.f || v[3] != 0.f) != 0;
      }
    return nonzero;
  };
  // ---- the eighths: through LDS, where they take the k-tiles' place, and added by all threads ----
  // Register v of lane (r32, q): row r32 of the row half, column 8 (v / 4) + 4 q + v % 4.
  auto add_and_store = [&](const RowTile& rt, int ct) {
    // !LONG: what depends on the lane is worked out anew, in registers across the products it would push others out
    int t = tid;
    if (!LONG) asm volatile("" : "+v"(t));
    float* const slot = smem + wave * kRedFloats + (t & 31) * kRedPitch + ((t >> 5) & 1) * 4;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int vg = 0; vg < 4; ++vg)
          *reinterpret_cast<f32x4*>(slot + i * 32 * kRedPitch + j * 32 + vg * 8) =
              f32x4{acc[i][j][vg * 4], acc[i][j][vg * 4 + 1], acc[i][j][vg * 4 + 2], acc[i][j][vg * 4 + 3]};
    lds_barrier();
    const int row = t >> 3, c4 = (t & 7) * 4;
    float small = INFINITY;   // smallest magnitude of this lane's totals
    if (row < rt.row_count) {
      auto total = [&](int col) {
        f32x4 s[kWaves], o;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) s[w] = *reinterpret_cast<const f32x4*>(smem + w * kRedFloats + row * kRedPitch + col);
#pragma unroll
        for (int e = 0; e < 4; ++e)
          o[e] = (float)(((double)(s[0][e] + s[4][e]) + (double)(s[2][e] + s[6][e])) +
                         ((double)(s[1][e] + s[5][e]) + (double)(s[3][e] + s[7][e])));
        return o;
      };
      const f32x4 t0 = total(c4), t1 = total(c4 + kBN / 2);
#pragma unroll
      for (int e = 0; e < 4; e += 2) {
        asm("v_min3_f32 %0, %0, |%1|, |%2|" : "+v"(small) : "v"(t0[e]), "v"(t0[e + 1]));
        asm("v_min3_f32 %0, %0, |%1|, |%2|" : "+v"(small) : "v"(t1[e]), "v"(t1[e + 1]));
      }
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
        f32x4 o;
#pragma unroll
        for (int e = 0; e < 4; ++e) o[e] = (t0[e] / (1.0f + expf(-t0[e]))) * t1[e];
        store(ct * kCols + c4, o);
      } else {
        store(ct * kCols + c4, t0);
        store(ct * kCols + c4 + kBN / 2, t1);
      }
    }
    // A total of zero: of a zero row (padding), or to be looked at if it can be the sum of terms that all vanished.  (A
    // wavefront's zero in a total that is not does no harm: with the operands that look() lets pass it is off by 2^-94.)
    if (!LONG && !AGAIN) {
      unsigned long long zeros = __ballot(small == 0.f);
      if (__builtin_expect(zeros != 0, 0))
        do {
          const int first = __ffsll(zeros) - 1 & ~7;   // of the 8 lanes of a row
          if (nonzero_row(rt, wave * 8 + first / 8)) mark(kLookIfSmall);
          zeros &= ~(255ull << first);
        } while (zeros != 0);
    }
    lds_barrier();   // before the next k-tiles
  };

  if (AGAIN) {
    uint32_t* const small_seen = &marks[kMarkWords + 1];
    for (; item < item_end; item += slots, ++number) {
      const uint32_t what = *mark_word() >> (number % 16 * 2) & 3;
      if (what == 0) continue;
      const Item it = find_item(item);
      set_addresses(it);
      fetch_first();
      if (!(what & kLook)) {
        if (any_small_element()) *small_seen = 1;
        lds_barrier();
        const bool seen = *small_seen != 0;
        lds_barrier();
        if (!seen) continue;
        *small_seen = 0;
        fetch_first();
      }
      const bool two = it.rt.row_count > 32;
      multiply_parts(two);
      if (kt0 < kt1) redo_sums(two);
      add_and_store(it.rt, it.ct);
    }
    return;
  }
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
    if (LONG) {
      multiply_f32(two);
    } else {
      multiply_parts(two);
      if (__builtin_expect(kt0 < kt1 && look(two), 0)) mark(kLook);
    }
    if (has_next) {   // the next item's first k-tile travels during the sums of this one
      set_addresses(next);
      fetch_first();
    }
    add_and_store(rt, ct);
    if (!has_next) break;
    cur = next;
    ++number;
  }
}
#endif

template <bool GATED, bool LONG>
__global__ __launch_bounds__(kThreads) void ffn_f32_kernel(const F32Args p) {
#if defined(__HIP_DEVICE_COMPILE__)
  extern __shared__ __align__(16) float smem[];
  int* const marks = reinterpret_cast<int*>(smem) + kTileBytes / 4;
  for (int i = threadIdx.x; i <= kControlWords + PRISM_MAX_EXPERTS; i += kThreads)
    marks[i] = i < kControlWords ? 0 : p.local_offsets[min(i - kControlWords, p.E)];
  __syncthreads();
  walk_items<GATED, LONG, false>(p, smem, threadIdx.x);
  if (!LONG && marks[kMarkWords] != 0) {   // (written before the last barrier)
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    walk_items<GATED, LONG, true>(p, smem, tid);
  }
#endif
}

template <bool GATED, bool LONG>
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
  if (!raise_lds_limit(lds_limit, (const void*)ffn_f32_kernel<GATED, LONG>, kLdsBytes)) return PRISM_ERR_LAUNCH;
  // one workgroup fits a CU
  hipLaunchKernelGGL((ffn_f32_kernel<GATED, LONG>), dim3((unsigned)std::min<long long>(kWorkgroups, align_up((size_t)items(5), kXcds))),
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
  auto in_parts = [](int K) { return K >= 4 && K <= kSplitMaxK; };   // (LONG has the code for rows shorter than a load)
  trace(stage_events, PRISM_STAGE_FFN_UP, 0, st);
  PRISM_TRY((in_parts(d.hidden) ? launch_f32_gemm<true, false> : launch_f32_gemm<true, true>)(a, st));
  trace(stage_events, PRISM_STAGE_FFN_UP, 1, st);
  trace(stage_events, PRISM_STAGE_FFN_DOWN, 0, st);
  PRISM_TRY((in_parts(d.ffn) ? launch_f32_gemm<false, false> : launch_f32_gemm<false, true>)(a, st));
  trace(stage_events, PRISM_STAGE_FFN_DOWN, 1, st);
  return PRISM_OK;
}

}  // namespace prism
