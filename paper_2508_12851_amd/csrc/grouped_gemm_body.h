// The body of the grouped GEMM kernels (grouped_gemm.h), for the tile BM x BN x BK, the ring of STAGES, the wavefront grid
// WGM x WGN and the options GATED, SPLITK, ROTATE, STREAM_B, SLICES of the scope that includes it; p: its GemmArgs.  Text and
// not a function: as an inlined function of the arguments it compiles to other code in every kernel, 0.3 to 0.6 %
// slower for decode batches.
#if defined(__HIP_DEVICE_COMPILE__)   // buffer resources exist in device code only
  static_assert(WGM * WGN == 4, "four wavefronts per workgroup");
  static_assert(BK == 32 || BK == 64, "LDS rows are 64 or 128 bytes");
  constexpr int WM = BM / WGM, WN = BN / WGN;
  constexpr int MI = WM / 32, NJ = WN / 32;
  static_assert(MI >= 1 && NJ >= 1 && (!GATED || NJ % 2 == 0), "tile shape");
  static_assert(!(GATED && SPLITK), "the gated epilogue needs complete sums");
  static_assert(!SLICES || (!GATED && !SPLITK && !ROTATE), "slices are entries of the plain prefill GEMM");
  constexpr int kRowBytes = BK * 2;
  constexpr int CPR = BK / 8;                 // 16-byte chunks per LDS row
  constexpr int RPG = 1024 / kRowBytes;       // rows filled by one wavefront-wide 16-byte load
  static_assert(BM % (4 * RPG) == 0 && BN % (4 * RPG) == 0, "tile rows split over 4 wavefronts");
  constexpr int A_CH = BM / (4 * RPG);        // load instructions per wavefront per stage
  constexpr int B_CH = BN / (4 * RPG);
  constexpr int LPS = A_CH + B_CH;
  constexpr int kStageBytes = (BM + BN) * kRowBytes;
  constexpr int KK = BK / 16;                 // MFMA k-steps per stage
  static_assert(STAGES >= 3, "ring needs a free stage to refill during an iteration");
  static_assert((STAGES - 1) * LPS <= 63, "vmcnt is a 6-bit counter");

  // wide bf16 output tiles are stored through LDS strips (see the epilogue)
  constexpr bool kStagedStore = staged_store<WN, GATED, SPLITK>();
  constexpr int kStripBase = STAGES * kStageBytes + (GATED ? 4096 : 0);

  extern __shared__ __align__(16) uint8_t smem[];

  // ---- this workgroup's items: slot, slot + slots, ... of its XCD's list -----------
  const int xcd = blockIdx.x % kXcds;
  int slot = blockIdx.x / kXcds;
  const const_int_ptr sched_c = (const_int_ptr)p.sched;
  const int count = sched_c[(SLICES ? 20 : 4) + xcd];
  int launched = gridDim.x / kXcds;
  // SPLITK: the schedule says how many workgroups share an item; neighbouring workgroups of an
  // XCD take the splits of one item slot, and those left over when the count does not divide the
  // launch end here.
  const int n_splits = SPLITK ? max(sched_c[2], 1) : 1;
  const int split = SPLITK ? slot % n_splits : 0;
  if (SPLITK) {
    slot /= n_splits;
    launched /= n_splits;
    if (slot >= launched) return;
  }
  if (slot >= count) return;
  // The list takes ceil(count / launched slots) rounds; the fewest workgroups that still
  // finish in that many rounds share it evenly (a workgroup that would sit out the last
  // round only takes memory bandwidth from the others in the rounds before).
  const int rounds = (count + launched - 1) / launched;
  const int slots = (count + rounds - 1) / rounds;
  if (slot >= slots) return;
  // slice entries sit in the last kSliceSlots places of every list
  const const_int4_ptr items =
      (const_int4_ptr)(p.sched + kSchedHeader) +
      ((size_t)xcd * sched_c[1] + (SLICES ? sched_c[1] - kSliceSlots : 0)) * (kItemInts / 4);

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // kept in a scalar register
  const int wm = wave / WGN, wn = wave % WGN;
  const int r32 = lane & 31, q = lane >> 5;

  // this workgroup's slice of the contraction, in k-tiles
  const int KT_all = p.K / BK;
  const int kt_first = SPLITK ? (int)((long long)KT_all * split / n_splits) : 0;
  const int kt_last = SPLITK ? (int)((long long)KT_all * (split + 1) / n_splits) : KT_all;
  const int KT = kt_last - kt_first;
  if (KT <= 0) return;

  // ---- global -> LDS assignment ------------------------------------------------
  // Wavefront w fills row groups w, w + 4, ...; a lane owns LDS slot lane % CPR of
  // row lane / CPR of the group and fetches the chunk that belongs in that slot.
  // Loads are buffer_load_dwordx4 ... lds with a per-lane 32-bit byte offset that
  // never changes within an item and the k offset in a scalar register, so a load
  // costs no vector ALU work; the buffer size makes an out-of-range row read zeros.
  // Row lrow = wave RPG + lane / CPR + 4 RPG i (>= 32 rows: does not change the key), chunk (lane % CPR) ^ key(lrow).
  const __amdgpu_buffer_rsrc_t a_rsrc =
      __builtin_amdgcn_make_buffer_rsrc((void*)p.A, 0, (int)p.a_bytes, kBufferFlags);

  // Item header as stored in the schedule.
  struct Item {
    int g, row_start, row_count, tok_base, nt;
    int kt0, kt_n, part;     // SLICES: the entry's k-tiles [kt0, kt0 + kt_n) and its partial-tile slot
  };
  // What the loads and the epilogue of an item need.
  struct Ctx {
    int row_start, row_count, nt;
    int kt0, kt_n, part;     // as in Item
    int rot;                 // ROTATE: k-tile this item starts its contraction with
    const void* b0;
    const void* b1;
    uint32_t a_voff[A_CH];
    uint32_t b_voff[B_CH];
  };
  // ROTATE schedules hold one line per row tile instead of item lists (schedule.h)
  const int n_ntiles = (p.N + (GATED ? BN / 2 : BN) - 1) / (GATED ? BN / 2 : BN);
  auto fetch_item = [&](int idx) {   // idx is clamped: the result is only used when idx < count
    const int i = min(idx, count - 1);
    if (ROTATE) {
      const unsigned seq = (unsigned)i * kXcds + (unsigned)xcd;
      const unsigned tile = seq / (unsigned)n_ntiles;
      const int4 h0 = ((const_int4_ptr)(p.sched + kSchedHeader))[tile];
      return Item{h0.x, h0.y, h0.z, h0.w, (int)(seq - tile * (unsigned)n_ntiles), 0, KT, -1};
    }
    const int4 h0 = items[2 * i];
    const int4 h1 = items[2 * i + 1];
    if (SLICES) return Item{h0.x, h0.y, h0.z, h0.w, h1.x, h1.y, h1.z, h1.w};
    return Item{h0.x, h0.y, h0.z, h0.w, h1.x, 0, KT, -1};
  };
  // Second hop: expert pointers (scalar loads) and, for the gathered GEMM, the
  // source rows of the row tile: each wavefront pulls the tile's BM entries of
  // local_src into its own 1 KiB of LDS with one buffer_load ... lds (so the load is
  // counted like the ring's loads and no VGPR waits on it), and reads its lanes'
  // entries from there once the load has surely landed.
  struct Raw {
    const void* b0;
    const void* b1;
  };
  static_assert(!GATED || BM <= 256, "one 1 KiB load brings the source rows of a row tile");
  uint8_t* const src_lds = smem + STAGES * kStageBytes + wave * 1024;
  const __amdgpu_buffer_rsrc_t src_rsrc =
      __builtin_amdgcn_make_buffer_rsrc((void*)p.local_src, 0, (int)p.src_bytes, kBufferFlags);
  auto fetch_raw = [&](const Item& it) {
    Raw r;
    const const_ptr_table t0 = (const_ptr_table)(it.g < p.E ? p.B0 : p.SB0);
    const const_ptr_table t1 = (const_ptr_table)(GATED ? (it.g < p.E ? p.B1 : p.SB1) : (it.g < p.E ? p.B0 : p.SB0));
    const int gi = it.g < p.E ? it.g : it.g - p.E;
    r.b0 = t0[gi];
    r.b1 = t1[gi];
    // Entry j of the LDS slot = local_src[row_start + j].  The whole byte offset sits in the
    // per-lane operand, which the hardware checks against the buffer size (a scalar offset
    // would escape that check), so entries past the end of local_src arrive as zeros instead
    // of being read.  Shared-expert tiles take their tokens from tok_base: their load is
    // issued out of range on purpose, which keeps the count of loads in flight uniform.
    if (GATED)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(
          src_rsrc, (lds_ptr_t)src_lds, 16,
          it.tok_base >= 0 && !p.a_tiled ? kOutOfRange : (uint32_t)it.row_start * 4u + (uint32_t)lane * 16u, 0, 0, 0);
    return r;
  };
  // Byte offset of row n of a matrix of K columns, tiles (16 rows x 32 columns, 1 KiB, row-tile major) or
  // row-major alike: (n / 16) blocks of 32 K bytes, n % 16 rows of the pitch inside.  A lane adds its 16-byte chunk c
  // of k-tile 0 (a 64-wide one spans two neighbouring tiles); the k-tile is added per load.  No branch per row: a
  // workgroup has one wavefront per SIMD, and nothing else runs there while it prepares an item.
  const uint32_t block_bytes = (uint32_t)p.K * 32u;
  auto chunk_offset = [&](int c, int tiled) {
    return tiled ? (uint32_t)(c >> 2) * 1024u + (uint32_t)(c & 3) * 16u : (uint32_t)c * 16u;
  };
  const uint32_t b_pitch = p.b_tiled ? 64u : (uint32_t)p.K * 2u;
  const uint32_t h_pitch = p.a_tiled ? 64u : p.a_pitch;   // plain GEMM: rows of h
  // a / top_k for a < 2^30, top_k <= 8: the excess of a * ceil(2^32 / top_k) / 2^32 stays below 1 / top_k
  const uint32_t k_magic = p.top_k > 1 ? 0xFFFFFFFFu / (uint32_t)p.top_k + 1u : 0u;
  auto make_ctx = [&](const Item& it, const Raw& raw) {
    Ctx cx;
    cx.row_start = it.row_start; cx.row_count = it.row_count; cx.nt = it.nt;
    cx.kt0 = it.kt0; cx.kt_n = it.kt_n; cx.part = it.part;
    cx.rot = ROTATE ? (int)((unsigned)(it.nt * 13 + it.g * 29) % (unsigned)KT) : 0;
    cx.b0 = raw.b0; cx.b1 = raw.b1;
    // what depends on the lane is worked out anew per item: in registers across the k-loop it would push others out
    int l = lane;
    asm volatile("" : "+v"(l));
    const int sub = l / CPR, lrow = wave * RPG + sub;
    const int c = (l % CPR) ^ swizzle_key<BK>(lrow);
#pragma unroll
    for (int i = 0; i < A_CH; ++i) {
      const int rr = min(lrow + 4 * RPG * i, it.row_count - 1);
      uint32_t off;
      if (GATED) {
        const uint32_t a = reinterpret_cast<const uint32_t*>(src_lds)[rr];
        const uint32_t tok = k_magic != 0 ? __umulhi(a, k_magic) : a;
        off = (it.tok_base >= 0 && !p.a_tiled ? (uint32_t)(it.tok_base + rr) : tok) * p.a_pitch + (uint32_t)c * 16u;
      } else {
        const uint32_t row = (uint32_t)(it.row_start + rr);
        off = (row >> 4) * block_bytes + (row & 15u) * h_pitch + chunk_offset(c, p.a_tiled);
      }
      // Rows past the end of a partly filled tile get an offset beyond the buffer: the
      // hardware then returns zeros, and all-zero operands cost the matrix cores far
      // less power than real data (the chip is power-limited in this kernel).
      cx.a_voff[i] = lrow + 4 * RPG * i < it.row_count ? off : kOutOfRange;
    }
    const uint32_t b_lane = (uint32_t)sub * b_pitch + chunk_offset(c, p.b_tiled);
#pragma unroll
    for (int i = 0; i < B_CH; ++i) {
      const int g0 = wave * RPG + 4 * RPG * i;      // first tile row of the group (scalar)
      // GATED: tile rows [w WN, w WN + WN/2) are gate rows, the next WN/2 the up rows of the same f.  (N is a
      // multiple of 64: a group's rows all exist, or the last group stands in for it.)
      const int n = GATED ? it.nt * (BN / 2) + g0 / WN * (WN / 2) + g0 % WN % (WN / 2) : it.nt * BN + g0;
      const uint32_t n0 = (uint32_t)min(n, p.N - RPG);
      cx.b_voff[i] = (n0 >> 4) * block_bytes + (n0 & 15u) * b_pitch + b_lane;
    }
    return cx;
  };

  // Issues loads [first, last) of the LPS loads that fill one stage with k-tile kt
  // of item cx (A row groups first, then B row groups).
  auto issue_loads = [&](const Ctx& cx, int kt, int stage, int first, int last) {
    // wave-uniform LDS base of this wavefront's first row group; lane * 16 is implicit
    uint8_t* base = smem + stage * kStageBytes + wave * RPG * kRowBytes;
    int kt_mem = kt;
    if (ROTATE) {
      kt_mem += cx.rot;
      if (kt_mem >= KT) kt_mem -= KT;
    }
    const int kel = (kt_first + (SLICES ? cx.kt0 : 0) + kt_mem) * BK;   // first contraction element
    const int koff = kel * 2;
    const int koff_tiled = (kel >> 5) * 1024;   // kel is a multiple of 32
    const int koff_b = p.b_tiled ? koff_tiled : koff;
    const int koff_a = (kel >> 5) * p.a_kstep;
    const __amdgpu_buffer_rsrc_t b0_rsrc =
        __builtin_amdgcn_make_buffer_rsrc((void*)cx.b0, 0, (int)p.b_bytes, kBufferFlags);
    const __amdgpu_buffer_rsrc_t b1_rsrc =
        __builtin_amdgcn_make_buffer_rsrc((void*)cx.b1, 0, (int)p.b_bytes, kBufferFlags);
#pragma unroll
    for (int i = 0; i < A_CH; ++i)
      if (i >= first && i < last)
        __builtin_amdgcn_raw_ptr_buffer_load_lds(a_rsrc, (lds_ptr_t)(base + i * 4 * RPG * kRowBytes),
                                                 16, cx.a_voff[i], koff_a, 0, 0);
#pragma unroll
    for (int i = 0; i < B_CH; ++i)
      if (A_CH + i >= first && A_CH + i < last) {
        const int g0 = wave * RPG + 4 * RPG * i;
        const bool up = GATED && (g0 % WN) >= WN / 2;
        __builtin_amdgcn_raw_ptr_buffer_load_lds(up ? b1_rsrc : b0_rsrc,
                                                 (lds_ptr_t)(base + (BM + i * 4 * RPG) * kRowBytes),
                                                 16, cx.b_voff[i], koff_b, 0, STREAM_B ? kNonTemporal : 0);
      }
  };

  // operand rows of this lane inside the LDS tile
  // Row subtile i of this wavefront is tile rows 32 (i WGM + wm) .. (the subtiles of
  // the WGM wavefront rows interleave).
  const int a_off = (wm * 32 + r32) * kRowBytes;          // + 32 WGM i rows
  const int b_off = (BM + wn * WN + r32) * kRowBytes;     // + 32 j rows
  const int key_r = swizzle_key<BK>(r32);

  bf16x8 af[2][MI], bfr[2][NJ];
  auto read_frags = [&](int stage, int kk, int buf) {
    const uint8_t* base = smem + stage * kStageBytes;
    const int slot_b = ((kk * 2 + q) ^ key_r) * 16;
    // in the order the MFMAs below consume them
    af[buf][0] = *reinterpret_cast<const bf16x8*>(base + a_off + slot_b);
#pragma unroll
    for (int j = 0; j < NJ; ++j)
      bfr[buf][j] = *reinterpret_cast<const bf16x8*>(base + b_off + j * 32 * kRowBytes + slot_b);
#pragma unroll
    for (int i = 1; i < MI; ++i)
      af[buf][i] = *reinterpret_cast<const bf16x8*>(base + a_off + i * WGM * 32 * kRowBytes + slot_b);
  };

  f32x16 acc[MI][NJ];

  // Ring protocol.  The k-tiles of this workgroup's items form one stream; stream
  // position g is computed from stage g % STAGES.  The prologue fills stages
  // 0..STAGES-2.  Iteration g, spread evenly over its MFMA steps, refills stage
  // (g - 1) % STAGES -- free since the barrier that ended iteration g - 1 -- with
  // stream position g + STAGES - 1 (which may belong to the next item).  In its last
  // step the wavefront waits until position g + 1 has landed (vmcnt counts only the
  // younger loads), drains its own LDS reads, meets the others at the barrier and
  // reads the first operands of position g + 1.  The last part of the refill is
  // issued after the barrier so that it, too, sits among MFMAs.
  constexpr int kPart = (LPS + KK - 1) / KK;     // most loads one step issues
  int stage = 0;                       // g % STAGES
  int fill_stage = STAGES - 1;         // (g + STAGES - 1) % STAGES
  // first: the first k-tile of an item, whose products start the sums (clearing the accumulators would take
  // as long as a k-tile's products, with nothing else to issue).
  const f32x16 kZero = {};
  auto k_iteration = [&](const Ctx& fill_cx, int fill_kt, auto first) __attribute__((always_inline)) {
    const int next_stage = stage + 1 == STAGES ? 0 : stage + 1;
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) {
      constexpr int kReads = MI + NJ;
      constexpr int kMfma = MI * NJ;
      if (kk + 1 < KK) {
        read_frags(stage, kk + 1, (kk + 1) & 1);
      } else {
        wait_vmcnt<(STAGES - 3) * LPS + (KK - 1) * LPS / KK>();
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        read_frags(next_stage, 0, (kk + 1) & 1);
      }
      issue_loads(fill_cx, fill_kt, fill_stage, kk * LPS / KK, (kk + 1) * LPS / KK);
#pragma unroll
      for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j0 = 0; j0 < NJ; ++j0) {
          // snake order over the grid of accumulators: every MFMA shares an operand with the one
          // before it (0.5 % on the power-limited prefill GEMMs)
          const int j = (i & 1) ? NJ - 1 - j0 : j0;
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bfr[kk & 1][j], af[kk & 1][i],
                                                              first && kk == 0 ? kZero : acc[i][j], 0, 0, 0);
        }
      // Issue order inside the step: one MFMA first (so the wait for this step's
      // operands precedes any new LDS read), then the next step's operand reads one
      // per MFMA, then this step's share of the refill one per MFMA.
      // (Tiles with too little matrix work per step are left to the compiler.)
      if constexpr (kMfma >= kReads + kPart + 1) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
#pragma unroll
        for (int r = 0; r < kReads; ++r) {
          __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
          __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        }
#pragma unroll
        for (int r = 0; r < kPart; ++r) {
          __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
          __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        }
        __builtin_amdgcn_sched_group_barrier(0x008, kMfma - 1 - kReads - kPart, 0);
      } else if constexpr (kMfma >= (kReads > kPart ? kReads : kPart) + 1) {
        // fewer MFMAs per step: an operand read and a refill load share the gap after an MFMA
        constexpr int kGaps = kReads > kPart ? kReads : kPart;
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
#pragma unroll
        for (int r = 0; r < kGaps; ++r) {
          if (r < kReads) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
          if (r < kPart) __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
          __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        }
        __builtin_amdgcn_sched_group_barrier(0x008, kMfma - 1 - kGaps, 0);
      }
    }
    stage = next_stage;
    fill_stage = fill_stage + 1 == STAGES ? 0 : fill_stage + 1;
  };

  // The weight rows are the MFMA's first operand, so accumulator register v of
  // lane (r32, q) is output row (activation row) r32 of subtile i and output
  // column 8 (v / 4) + 4 q + v % 4 of subtile j: four consecutive columns per
  // register quad, i.e. one 8-byte (bf16) or 16-byte (fp32 partial) piece.
  //
  // Stored straight from there, an instruction writes 16 bytes to each of 32 rows, and the
  // write path then takes a fifth of a short-contraction item (12.6k clocks against 54k of
  // k-loop for the 1408-long down projection).  Wide bf16 tiles therefore pass every strip
  // of 32 rows x 64 columns through a 4.5 KiB LDS buffer of the wavefront's own (row pitch
  // 144 bytes) and store it with 16 bytes per lane, 8 lanes per row: whole 128-byte lines.
  // The LDS instructions come from assembly: for LDS accesses it sees, the compiler would
  // first wait for every direct-to-LDS load in flight (the next item's operands).  A
  // wavefront's LDS instructions execute in order, so the read-back needs no wait after the
  // writes, nor the next strip's writes after the read-back.
  auto epilogue_staged = [&](const Ctx& cx) {
    constexpr int NO = GATED ? NJ / 2 : NJ;                 // output column subtiles of 32
    constexpr int kPairs = NO / 2 > 0 ? NO / 2 : 1;         // (instantiated for narrow tiles too, never called)
    constexpr int kStrips = MI * kPairs;                  // strip s: row subtile s / kPairs, column pair s % kPairs
    const uint32_t strip = (uint32_t)(uintptr_t)(lds_ptr_t)(smem + kStripBase) + wave * kStripBytes;
    const uint32_t wr = strip + r32 * kStripPitch + q * 8;  // + 2 (32 jl + 8 vg)
    const int rd_row = lane >> 3, rd_chunk = lane & 7;       // + 8 t rows
    const uint32_t rd = strip + rd_row * kStripPitch + rd_chunk * 16;
    const int col0 = (GATED ? cx.nt * (BN / 2) + wn * (WN / 2) : cx.nt * BN + wn * WN) + rd_chunk * 8;
    // the values of a strip as this lane holds them: 2 subtiles x 4 quads of 4 bf16
    auto strip_values = [&](int st, u32x2 (&o)[8]) {
      const int i = st / kPairs, jp = st % kPairs;
#pragma unroll
      for (int jl = 0; jl < 2; ++jl)
#pragma unroll
        for (int vg = 0; vg < 4; ++vg) {
          const int j = jp * 2 + jl;
          bf16x4 b;
#pragma unroll
          for (int e = 0; e < 4; ++e)
            b[e] = GATED ? (bf16_t)(silu(acc[i][j][vg * 4 + e]) * acc[i][j + NO][vg * 4 + e])
                         : (bf16_t)acc[i][j][vg * 4 + e];
          o[jl * 4 + vg] = __builtin_bit_cast(u32x2, b);
        }
    };
    // Strip st + 1 is computed while the writes of strip st are on their way.
    u32x2 cur[8], nxt[8];
    strip_values(0, cur);
#pragma unroll
    for (int st = 0; st < kStrips; ++st) {
      const int i = st / kPairs, jp = st % kPairs;
      const int row0 = (i * WGM + wm) * 32;
      const bool live = row0 < cx.row_count;                // wavefront-uniform
      // keep every strip's instructions together: moved up by the scheduler, the accumulator
      // reads of all strips would be live at once and push other values into scratch memory
      __builtin_amdgcn_sched_barrier(0);
      if (live) {
#pragma unroll
        for (int w8 = 0; w8 < 8; ++w8)
          asm volatile("ds_write_b64 %0, %1 offset:%2"
                       :: "v"(wr), "v"(cur[w8]), "n"(((w8 / 4) * 32 + (w8 % 4) * 8) * 2) : "memory");
      }
      if (st + 1 < kStrips) strip_values(st + 1, nxt);
      if (live) {
        // one statement up to the wait: the compiler takes an output for valid as soon as its
        // statement ends (and may copy it elsewhere right away)
        u32x4 v0, v1, v2, v3;
        asm volatile(
            "ds_read_b128 %0, %4 offset:%5\n\tds_read_b128 %1, %4 offset:%6\n\t"
            "ds_read_b128 %2, %4 offset:%7\n\tds_read_b128 %3, %4 offset:%8\n\ts_waitcnt lgkmcnt(0)"
            : "=&v"(v0), "=&v"(v1), "=&v"(v2), "=&v"(v3)
            : "v"(rd), "n"(0), "n"(8 * kStripPitch), "n"(16 * kStripPitch), "n"(24 * kStripPitch)
            : "memory");
        const u32x4 v[4] = {v0, v1, v2, v3};
        const int col = col0 + jp * 64;
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          const int row = row0 + t * 8 + rd_row;
          if (row < cx.row_count && col < p.N)
            *reinterpret_cast<u32x4*>(p.C + (size_t)(cx.row_start + row) * p.N + col) = v[t];
        }
      }
#pragma unroll
      for (int w8 = 0; w8 < 8; ++w8) cur[w8] = nxt[w8];
    }
  };
  auto epilogue = [&](const Ctx& cx) {
    if constexpr (SLICES) {
      // the accumulators as they are, an fp32 tile [BM][BN] in slot cx.part
      float* tile = p.Cpart + (size_t)cx.part * (BM * BN);
#pragma unroll
      for (int i = 0; i < MI; ++i) {
        if ((i * WGM + wm) * 32 >= cx.row_count) continue;    // wave-uniform
        const int row = (i * WGM + wm) * 32 + r32;
#pragma unroll
        for (int j = 0; j < NJ; ++j)
#pragma unroll
          for (int vg = 0; vg < 4; ++vg) {
            const int n = wn * WN + j * 32 + vg * 8 + q * 4;
            const f32x4 o = {acc[i][j][vg * 4], acc[i][j][vg * 4 + 1], acc[i][j][vg * 4 + 2],
                             acc[i][j][vg * 4 + 3]};
            *reinterpret_cast<f32x4*>(tile + (size_t)row * BN + n) = o;
          }
      }
      return;
    }
    if constexpr (kStagedStore) {
      epilogue_staged(cx);
      return;
    }
#pragma unroll
    for (int i = 0; i < MI; ++i) {
      const int row = (i * WGM + wm) * 32 + r32;
      if (row >= cx.row_count) continue;
      const size_t crow = (size_t)(cx.row_start + row);
      if (GATED) {
        constexpr int NH = NJ / 2;
        const int f0 = cx.nt * (BN / 2) + wn * (WN / 2);       // a multiple of 32
        uint16_t* const out = p.C + (p.c_tiled ? (crow >> 4) * (size_t)(p.N >> 5) * 512 + (size_t)(f0 >> 5) * 512 +
                                                     (crow & 15) * 32
                                               : crow * p.N + f0) + q * 4;
        const int col_step = p.c_tiled ? 512 : 32;             // elements from one column subtile to the next
#pragma unroll
        for (int j = 0; j < NH; ++j)
#pragma unroll
          for (int vg = 0; vg < 4; ++vg) {
            if (f0 + j * 32 + vg * 8 + q * 4 < p.N) {
              bf16x4 o;
#pragma unroll
              for (int e = 0; e < 4; ++e)
                o[e] = (bf16_t)(silu(acc[i][j][vg * 4 + e]) * acc[i][j + NH][vg * 4 + e]);
              *reinterpret_cast<bf16x4*>(out + j * col_step + vg * 8) = o;
            }
          }
      } else {
#pragma unroll
        for (int j = 0; j < NJ; ++j)
#pragma unroll
          for (int vg = 0; vg < 4; ++vg) {
            const int n = cx.nt * BN + wn * WN + j * 32 + vg * 8 + q * 4;
            if (n < p.N) {
              if (SPLITK) {
                const f32x4 o = {acc[i][j][vg * 4], acc[i][j][vg * 4 + 1], acc[i][j][vg * 4 + 2],
                                 acc[i][j][vg * 4 + 3]};
                *reinterpret_cast<f32x4*>(p.Cpart + ((size_t)split * p.c_rows + crow) * p.N + n) = o;
              } else {
                bf16x4 o;
#pragma unroll
                for (int e = 0; e < 4; ++e) o[e] = (bf16_t)acc[i][j][vg * 4 + e];
                *reinterpret_cast<bf16x4*>(p.C + crow * p.N + n) = o;
              }
            }
          }
      }
    }
  };

  // ---- walk the items ---------------------------------------------------------------
  // Item headers are fetched two items ahead and their pointers / source rows one
  // item ahead, so nothing on the critical path waits for them.
  int idx = slot;
  Item it_cur = fetch_item(idx);
  const Raw raw_cur = fetch_raw(it_cur);
  wait_vmcnt<0>();                       // the first item's source rows
  Ctx cur = make_ctx(it_cur, raw_cur);
  Item it_next = fetch_item(idx + slots);

#pragma unroll
  for (int s = 0; s < STAGES - 1; ++s) issue_loads(cur, min(s, cur.kt_n - 1), s, 0, LPS);
  wait_vmcnt<(STAGES - 2) * LPS>();
  __builtin_amdgcn_s_barrier();
  read_frags(0, 0, 0);

  while (true) {
    const bool has_next = idx + slots < count;
    const Item it_next2 = fetch_item(idx + 2 * slots);
    const Item& it_fill = has_next ? it_next : it_cur;
    const Raw raw_next = fetch_raw(it_fill);      // one more counted load, older than all that follow

    // refills still inside this item
    const int kt_n = SLICES ? cur.kt_n : KT;   // (every entry has at least STAGES - 1 k-tiles)
    // 256 x 256 tiles peel the first k-tile (4096 tokens of the 4096 x 14336 layer: layer 2075 -> 2065 us).  Lower ones have
    // 32 to 128 registers to clear, and the longer code costs as much as it saves (15 layers of 60 to 196 narrow experts at
    // 75 to 1016 tokens: layer 0.2 % slower with the peeled k-tile, up to 1 %).
    constexpr bool kFirst = MI * NJ == 16;
    if (kFirst && kt_n > STAGES - 1) {
      k_iteration(cur, STAGES - 1, std::true_type{});
    } else {
#pragma unroll
      for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j) acc[i][j] = kZero;
    }
    for (int kt = kFirst ? 1 : 0; kt + (STAGES - 1) < kt_n; ++kt) k_iteration(cur, kt + STAGES - 1, std::false_type{});
    // The source rows of the next item were requested before those iterations; loads
    // complete in order, so they have landed once enough younger loads have been
    // waited for, which the iterations above guarantee only if there were enough.
    if (GATED && KT < 2 * (STAGES - 1)) wait_vmcnt<0>();
    // refills that already belong to the next item (for the last item: a harmless
    // re-fetch of this item's first k-tiles, which keeps the vmcnt bookkeeping uniform)
    const Ctx nxt = make_ctx(it_fill, raw_next);
    for (int kt = max(kt_n - (STAGES - 1), 0); kt < kt_n; ++kt)
      k_iteration(nxt, min(kt + (STAGES - 1) - kt_n, (SLICES ? nxt.kt_n : KT) - 1), std::false_type{});

    epilogue(cur);
    if (!has_next) break;
    cur = nxt;
    it_cur = it_next;
    it_next = it_next2;
    idx += slots;
  }
  wait_vmcnt<0>();   // the last refills must land before this LDS allocation is released
#endif  // __HIP_DEVICE_COMPILE__
