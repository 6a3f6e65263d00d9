// Tile core of the bf16 grouped GEMMs for gfx950: matrix-core tiles (v_mfma_f32_16x16x32_bf16) with operands staged through
// LDS, and the epilogue of a tile, which the fp32 core (split_core.h) shares.
//
// The core computes, for one block, acc[nb][..] = sum over iterations of A_tile * B_tile(nb), and turns
// them into NOUT output matrices (with NAUX input matrices of the same shape) as an epilogue object says:
//     epi.apply(v, aux, scale, o)   v[nb][0..3] = C[m][n..n+3], aux[x][0..3], scale = epi.row_scale(m) -> o[out][0..3]
// Its members: NOUT, NAUX, OES (bytes per element of all those matrices), stream() (streaming stores);
// out[], in[] (origins of the tile in them), ldc (their row stride), rows, n_valid (valid extents of the tile).
// The sum over K runs over n_segs segments of nk iterations each (segments: the shared experts of
// a down projection, the two products of an input gradient); a segment functor supplies where the
// tiles of a segment start, and the core steps along K from there themselves.
#pragma once

#include <algorithm>
#include <utility>

#include "moe_common.h"
#include "trace.h"

namespace moe {
// 16 bytes through a bounds-checked buffer descriptor (reads beyond it return zero, writes are dropped)
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4_t;
__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void* base, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, bytes, 0x00020000);
}

// Start of one segment.  Pointers are already offset to the tile's first row/column at k = 0;
// "kc" (K-contiguous) operands are [rows][K] row-major, otherwise [K][rows] row-major.
template <typename T, int NB>
struct SegSrc {
  const T* a;        // A tile origin
  const T* b[NB];    // B tile origin(s)
  int k_len;         // values of K in the segment
  // bytes from the origins to the end of the valid data of the tile (used by the cores that load
  // through bounds-checked buffer descriptors: anything at or beyond reads as zero)
  int64_t a_bytes, b_bytes;
};

// Where row m of the A tile lives.  Plain tiles: row m of the tile (the tile origin is part of the
// operand pointers).  Gathered tiles (K-contiguous A only): row idx[row0 + m] / div of the whole
// operand, whose origin the pointers then are -- the token rows of X or dY read in grouped order
// without a permuted copy.
struct RowMap {
  const int32_t* idx;  // NULL: plain
  int32_t div, row0, rows;  // rows: valid rows of the tile (rows at or beyond read as zero)
  __device__ __forceinline__ bool gathered() const { return idx != nullptr; }
  __device__ __forceinline__ int operator()(int m) const { return idx[row0 + m] / div; }
};

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8_t;
typedef __attribute__((ext_vector_type(4))) short short4_t;
typedef __attribute__((ext_vector_type(8))) short short8_t;
typedef __attribute__((ext_vector_type(4))) float f32x4_t;

// f(integral_constant<int, 0>), ... f(integral_constant<int, N - 1>): the K loops are written out by it, so that every
// position in them is a constant (an unroll pragma gives up on loops whose bounds depend on an outer one's counter)
template <class F, int... I>
__device__ __forceinline__ void static_for_impl(F& f, std::integer_sequence<int, I...>) {
  (f(std::integral_constant<int, I>()), ...);
}
template <int N, class F>
__device__ __forceinline__ void static_for(F f) {
  static_for_impl(f, std::make_integer_sequence<int, (N > 0 ? N : 0)>());
}

// ------------------------------------------------------------------ epilogue of a tile
// Epilogue.  In the MFMA result layout a lane owns four consecutive columns of a row, so direct
// global accesses would be scatters of 8- or 16-byte pieces.  The arithmetic is done in that layout, on
// registers; the finished outputs, already in their final type, pass through a private LDS region of the
// wave in blocks of 32 rows and are picked up again as whole rows, 16 bytes per lane.  Inputs of the epilogue
// (the saved activations of a backward product, an output to add to) take the opposite way: whole rows
// into registers one block ahead, through the same region into the result layout.  The region's
// 16-byte pieces are XOR-swizzled by the row; LDS operations of one wave execute in order, so its reads and
// writes need no waits of their own, and the stores of a block are issued after the next block's
// arithmetic, under which their LDS reads return.
// What bounds it is instruction issue: one wave per SIMD, nothing to switch to.  (Staging fp32 values and
// doing arithmetic, rounding and addresses in row order, one pass of 4 rows after the other, took 10.5 k shader
// cycles per 256 x 256 tile of plain outputs, 13.8 k with SwiGLU, 50 k with its derivative; without the
// global stores still 9.9 k, 13.0 k, 39 k.  This form: 7.3 k, 12 k, 41 k, without the stores 4.5 k, 9.7 k, 34 k: what is
// left is arithmetic, two transcendentals per value, and the stores and loads of a launch's first tiles, which
// all CUs issue together.  Whole steps gain 1-3 % only, because the shader clock drops as the matrix pipe idles less.)
// NB products of TM x TN tiles a wave, NW waves; AGPR: the accumulators live in AGPRs, under inline assembly, and are
// copied out one by one.
// ROWS: rows of a block.  MT: rows of a tile, one per lane % MT; its columns are four for every lane of a row, lane / MT by lane / MT.
// AHEAD: the next block's inputs are loaded under a block's arithmetic (two blocks per CU have no registers for them).
template <int NB, int TM, int TN, int NW, int LDS, bool AGPR, int ROWS = 32, int MT = 16, bool AHEAD = true>
struct TileEpilogue {
  static constexpr int HP = 64 / MT, CT = 4 * HP;  // lanes of a row, columns of a tile
  // LDS that the staging regions of `waves` waves take
  template <class Epi> static constexpr int bytes(int waves) {
    return waves * (Epi::NOUT > Epi::NAUX ? Epi::NOUT : Epi::NAUX) * ROWS * TN * CT * Epi::OES;
  }
  template <class Epi>
  __device__ static __forceinline__ void run(char* smem, f32x4_t (&acc)[NB][TM][TN], const Epi& epi, int wave, int lane, int wm0, int wn0) {
    constexpr int OES = Epi::OES, NOUT = Epi::NOUT, NAUX = Epi::NAUX;
    constexpr int RB = TN * CT * OES;         // bytes per row of the wave's tile
    constexpr int LPR = RB / 16;              // lanes (16-byte pieces) per row
    constexpr int RPP = 64 / LPR;             // rows per wave-wide access
    constexpr int NPASS = ROWS / RPP;
    constexpr int SWZ = (LPR < 16 ? LPR : 16) - 1;
    constexpr int NI = TM * MT / ROWS;        // blocks of the wave's tile
    constexpr int BLOCK = ROWS * RB;          // one block of one matrix
    constexpr int NMAT = NOUT > NAUX ? NOUT : NAUX;
    constexpr int NA = NAUX > 0 ? NAUX : 1;
    static_assert(bytes<Epi>(NW) <= LDS, "the waves' staging regions fit into LDS");
    char* stage = smem + wave * (NMAT * BLOCK);
    // row order: row pass * RPP + lane / LPR, piece lane % LPR;  result layout: see MT
    const int rrow = lane / LPR, rpiece = lane % LPR;
    const uint32_t r_off = rrow * RB + ((rpiece ^ (rrow & SWZ)) << 4);
    constexpr int GR = ROWS / MT;             // tiles of a block's rows
    const int mrow = lane & (MT - 1), h = lane / MT;
    uint32_t m_off[GR];
#pragma unroll
    for (int rh = 0; rh < GR; rh++) m_off[rh] = (rh * MT + mrow) * RB + (((rh * MT + mrow) & SWZ) << 4);
    auto row_at = [&](int pass) __attribute__((always_inline)) {  // (rrow < RPP, so the row's other bits come from pass)
      return (r_off ^ (((pass * RPP) & SWZ) << 4)) + pass * RPP * RB;
    };
    // first of the lane's four columns: CT * j + 4 * h
    auto col_at = [&](int rh, int j) __attribute__((always_inline)) {
      return OES == 2 ? (m_off[rh] ^ ((HP / 2 * j + (h >> 1)) << 4)) + 8 * (h & 1) : (m_off[rh] ^ ((HP * j + h) << 4));
    };
    // global side: byte offsets from the tile's origin in every matrix
    const int c0 = wn0 + rpiece * (16 / OES);
    const uint32_t ldb = (uint32_t)epi.ldc * OES;
    const uint32_t g0 = (uint32_t)(wm0 + rrow) * ldb + (uint32_t)c0 * OES;
    const bool col_ok = c0 < epi.n_valid;
    const uint32_t extent = ((uint32_t)epi.rows - 1) * ldb + (uint32_t)epi.n_valid * OES;
    u32x4_t piece[NMAT][NPASS];
    auto load_aux = [&](int i) __attribute__((always_inline)) {
#pragma unroll
      for (int x = 0; x < NAUX; x++)
#pragma unroll
        for (int p = 0; p < NPASS; p++)
          piece[x][p] = __builtin_amdgcn_raw_buffer_load_b128(make_rsrc(epi.in[x], extent), g0 + (i * ROWS + p * RPP) * ldb, 0, 0);
    };
    // the row pieces of block i
    auto store_pieces = [&](const auto& r, int i) __attribute__((always_inline)) {
      auto put = [&](auto hint) __attribute__((always_inline)) {
#pragma unroll
        for (int x = 0; x < NOUT; x++)
#pragma unroll
          for (int p = 0; p < NPASS; p++)
            __builtin_amdgcn_raw_buffer_store_b128(r[x][p], make_rsrc(epi.out[x], extent), g0 + (i * ROWS + p * RPP) * ldb, 0,
                                                   decltype(hint)::value);
      };
      if (!col_ok) return;
      if (RB >= 128 && epi.stream()) put(std::integral_constant<int, 2>());
      else put(std::integral_constant<int, 0>());
    };
    if (NAUX > 0 && AHEAD) load_aux(0);
    float scale[TM];
#pragma unroll
    for (int i = 0; i < TM; i++) scale[i] = epi.row_scale(wm0 + i * MT + mrow);
#pragma unroll
    for (int i = 0; i < NI; i++) {
      if (NAUX > 0) {
        if (!AHEAD) load_aux(i);
#pragma unroll
        for (int x = 0; x < NAUX; x++)
#pragma unroll
          for (int p = 0; p < NPASS; p++) *reinterpret_cast<u32x4_t*>(stage + x * BLOCK + row_at(p)) = piece[x][p];
        asm volatile("" ::: "memory");
        if (AHEAD && i + 1 < NI) load_aux(i + 1);
      }
      // inputs are read one position ahead: every read behind the stores of the position before would wait for LDS with nothing to do
      // meanwhile (dH with dWd, T = 4096, d = 2048, 60 experts and four shared: 444 us so, 438 now; T = 16384 of the stress routing 827, 822)
      typename Epi::packed_t next[NA], a[NA];
      auto fetch = [&](int t) __attribute__((always_inline)) {
#pragma unroll
        for (int x = 0; x < NAUX; x++) next[x] = *reinterpret_cast<const typename Epi::packed_t*>(stage + x * BLOCK + col_at(t / TN, t % TN));
      };
      fetch(0);
#pragma unroll
      for (int t = 0; t < GR * TN; t++) {
        const int rh = t / TN, j = t % TN;
        float v[NB][4], in[NA][4], o[NOUT][4];
#pragma unroll
        for (int x = 0; x < NAUX; x++) a[x] = next[x];
        if (t + 1 < GR * TN) fetch(t + 1);
#pragma unroll
        for (int x = 0; x < NAUX; x++) Epi::unpack(a[x], in[x]);
#pragma unroll
        for (int nb = 0; nb < NB; nb++)
#pragma unroll
          for (int q = 0; q < 4; q++) {
            if constexpr (AGPR) asm volatile("v_accvgpr_read_b32 %0, %1" : "=v"(v[nb][q]) : "a"(acc[nb][GR * i + rh][j][q]));
            else v[nb][q] = acc[nb][GR * i + rh][j][q];
          }
        epi.apply(v, in, scale[GR * i + rh], o);
#pragma unroll
        for (int x = 0; x < NOUT; x++) Epi::pack(stage + x * BLOCK + col_at(rh, j), o[x]);
      }
      asm volatile("" ::: "memory");  // other lanes' values are read back below
      if (NAUX > 0) {
        // the registers of the row pieces hold the next block's inputs: pass the outputs through others
        u32x4_t r[NOUT][NPASS];
#pragma unroll
        for (int x = 0; x < NOUT; x++)
#pragma unroll
          for (int p = 0; p < NPASS; p++) r[x][p] = *reinterpret_cast<const u32x4_t*>(stage + x * BLOCK + row_at(p));
        store_pieces(r, i);
      } else {
        if (i > 0) store_pieces(piece, i - 1);
#pragma unroll
        for (int x = 0; x < NOUT; x++)
#pragma unroll
          for (int p = 0; p < NPASS; p++) piece[x][p] = *reinterpret_cast<const u32x4_t*>(stage + x * BLOCK + row_at(p));
      }
      asm volatile("" ::: "memory");
    }
    if (NAUX == 0) store_pieces(piece, NI - 1);
  }
};

// ------------------------------------------------------------------ MFMA core, LDS DMA loads
// Tiles travel HBM/L2 -> LDS directly (buffer_load_dwordx4 ... lds),
// so no registers stage them.  Lane l of a wave-wide load lands at lds_base + 16*l, which fixes
// each tile to whole 1 KB pieces per instruction; the swizzles are applied on the global side
// (which 16-byte piece a lane fetches).  Out-of-range pieces read as zero through the buffer
// descriptor's num_records, which provides the zero fill of ragged row tails and, for operands whose
// rows are K values, of the K tail.  A K tail inside the rows of a K-contiguous operand is masked with
// KTAIL: the lanes whose piece lies at or beyond K fetch from an offset no descriptor reaches.
//
// A tile row is 128 bytes of K (64 values), a k-step 32 values, and a lane's fragment of a k-step, 16 rows of it, is 16 bytes.
// The 32x32x16 instruction does the same work per cycle
// from the same fragment bytes, but it reads and writes every accumulator twice as often, and the chip's clock falls further under it:
// register-resident loops over normally distributed values sustain 1.73 PFLOP/s with it and 1.99 with 16x16x32.
// That alone changed nothing while the K loop was bound by issue (408 instructions per 128 MFMAs); with 225 (steps of
// three additions, M0 written by the addition that forms the address, the MFMA as its wait state, LDS addresses carried in bytes)
// whole training steps gain: T = 8192, d = 4096, 16 experts of 6400 7439 -> 7043 us, T = 8192, d = 7168, 256 experts 22830 -> 21837.
//
// LDS layouts, BK = 128 bytes of K, no padding:
//  K-contiguous operand [rows][BK]: 16-byte piece c of a row sits at position c ^ ((row/2)%8), so
//    that the 16 rows one phase of a 16-byte-per-lane read touches cover all banks once.
//  row-contiguous operand [BK][ROWS]: piece c (8 columns) of k-row k sits at position
//    c ^ (4*(k%4)) ^ (2*((k/8)%2)): the 32 lanes of two 16-lane groups of a transposing read, which take 16 columns of
//    four k rows and of the four k rows 8 further on, touch all banks once (64 columns, two k rows to the width of the banks:
//    c ^ (2*((k/2)%2)) ^ (4*((k/8)%2))).
template <int BM_, int BN_, int NB, bool A_KC, bool B_KC, int WM_ = 2, int WN_ = 2, int DEPTH = 1,
          bool KTAIL = false>
struct MfmaDmaCore {
  typedef bf16_t T;
  static constexpr int ES = sizeof(T);
  static constexpr int PE = 16 / ES;  // elements per 16-byte piece
  static constexpr int BM = BM_, BN = BN_, BK = 8 * PE;
  static constexpr int MT = 16;  // rows and columns of an accumulator tile
  static constexpr int KS = 2;   // MFMA k-steps per tile slot
  typedef bf16x8_t frag_t;
  typedef f32x4_t acc_t;
  static constexpr int AR = 4;   // registers of an accumulator tile
  static constexpr int WM = WM_, WN = WN_;
  static constexpr int NW = WM * WN, NT = 64 * NW;  // wavefronts and threads per block
  static constexpr int TM = BM / WM / MT, TN = BN / WN / MT;
  static constexpr int A_ELEMS = BM * BK, B_ELEMS = BN * BK;
  // Software pipeline of the K loop, by DEPTH:
  //  1  (tall tiles, bound by the matrix pipe): a ring of three A tiles and a ring of two B tile
  //     sets.  The A tile of iteration t+2 is requested while the B tiles of t+1 are still
  //     landing, so the memory pipeline never runs dry at the per-iteration barrier; MFMAs, LDS
  //     reads and tile loads are interleaved by hand.
  //  >= 2  (short tiles of ragged groups, bound by streaming the other operand from HBM): DEPTH + 1
  //     slots per operand and the loads of iteration t + DEPTH issued in iteration t, so that DEPTH
  //     whole K steps are in flight per CU; the latency of an HBM stream, not the matrix pipe, sets
  //     the pace there.
  //  0  (weight gradients of groups with a handful of rows: K is one step): one slot, no
  //     pipeline, small enough in LDS and registers for several blocks per CU, which is what hides
  //     latency when a block's life is one K iteration and an epilogue.
  static constexpr bool RING = DEPTH == 1;
  static constexpr bool REPEATS = DEPTH == 0;  // a block may compute several tiles (see w_gemm_block)
  static constexpr int A_SLOTS = DEPTH == 0 ? 1 : DEPTH == 1 ? 3 : DEPTH + 1;
  static constexpr int B_SLOTS = DEPTH == 0 ? 1 : DEPTH == 1 ? 2 : DEPTH + 1;
  static constexpr int B_SET_ELEMS = NB * B_ELEMS;
  static constexpr int TILE_BYTES = (A_SLOTS * A_ELEMS + B_SLOTS * B_SET_ELEMS) * ES;
  static constexpr int LDS_BYTES = TILE_BYTES;
  // blocks per CU the register allocation aims at (LDS allows as many)
  static constexpr int BLOCKS_PER_CU = LDS_BYTES > 80 * 1024 ? 1 : DEPTH == 0 ? 4 : NB * TM * TN * AR <= 64 ? 2 : 1;
  static constexpr int A_NI = BM / (8 * NW), B_NI = BN / (8 * NW);  // wave-wide loads per wave and tile
  static constexpr int PR_KC = 8;  // 16-byte pieces per row of a K-contiguous tile
  static_assert(NW == 4 || NW == 8, "four or eight wavefronts per block");
  static_assert(BM % (8 * NW) == 0 && BN % (8 * NW) == 0,
                "every wave issues the same number of 1 KB loads per tile");
  static_assert(BM % (32 * WM) == 0 && BN % (32 * WN) == 0, "wave tile must be a multiple of 32");
  static_assert((A_KC || BM * ES % 128 == 0) && (B_KC || BN * ES % 128 == 0),
                "swizzle of row-contiguous tiles needs >= 8 pieces per k row");
  static_assert(LDS_BYTES <= 160 * 1024, "LDS budget of a gfx950 CU");
  typedef __attribute__((address_space(3))) void* lds_vptr;

  // Byte offset (from the tile origin in memory) of the piece that lane `lane` fetches into the 1 KB piece `wave` of
  // the LDS tile (the j-th load of a wave fills piece wave + j * NW).  run() keeps one offset register per load, so that
  // the K loop spends no instructions on addresses and the whole offset stays inside the
  // descriptor's bounds check.
  __device__ static __forceinline__ int kc_swizzle(int row) { return ((row * PR_KC) >> 4) & (PR_KC - 1); }
  template <int ROWS>
  __device__ static __forceinline__ int rc_swizzle(int k) {
    return ROWS == 64 ? 2 * ((k >> 1) & 1) ^ 4 * ((k >> 3) & 1) : 4 * (k & 3) ^ 2 * ((k >> 3) & 1);
  }
  template <int ROWS, bool KC>
  __device__ static __forceinline__ uint32_t piece_offset(int wave, int lane, uint32_t ld) {
    const int q = wave * 64 + lane;  // linear 16-byte piece of the LDS tile
    if (KC) {
      const int row = q / PR_KC, pos = q % PR_KC;
      const int c = pos ^ kc_swizzle(row);
      return (uint32_t)row * ld * ES + (uint32_t)c * 16u;
    } else {
      constexpr int PR = ROWS / PE;
      const int k = q / PR, pos = q % PR;
      const int c = pos ^ rc_swizzle<ROWS>(k);
      return (uint32_t)k * ld * ES + (uint32_t)c * 16u;
    }
  }
  // first K value (within a tile) of the piece that a lane fetches from a K-contiguous operand: the same
  // for all of its loads
  __device__ static __forceinline__ int piece_k(int wave, int lane) {
    const int q = wave * 64 + lane;
    return ((q % PR_KC) ^ kc_swizzle(q / PR_KC)) * PE;
  }

  // One wave-wide 16-byte-per-lane load straight into LDS: the n-th 1 KB piece of this wave's share
  // of a tile.  Written as inline assembly so that the compiler does not serialise it against the
  // LDS reads of the other stage (it would wait for vmcnt(0) before every ds_read that may alias);
  // run() waits for the loads itself before its barrier.
  typedef __attribute__((ext_vector_type(4))) int rsrc_t;
  // `rsrc` is the raw buffer descriptor of the tile (48-bit base, stride 0, byte count, 32-bit data
  // format), `voff` the lane's byte offset from its base (piece_offset plus the rows of the earlier
  // loads of the tile), `dst` the LDS byte address of this wave's 1 KB piece.
  //
  // The compiler's hazard recogniser does not look inside inline assembly.  M0 must not be read by an
  // LDS-DMA load in the wait state after its write, hence the s_nop.  The descriptor words must not
  // have been written by a VALU instruction (v_readfirstlane and the like) in the five wait states
  // before the load: they are kept in scalar registers and stepped with scalar instructions only
  // (see Cursor), far from any vector instruction that could produce them.
  __device__ static __forceinline__ void issue_one(const rsrc_t& rsrc, uint32_t dst, uint32_t voff) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds"
                 :
                 : "s"(dst), "v"(voff), "s"(rsrc)
                 : "memory");
  }

  // ---- LDS -> MFMA fragment: lane l holds k = 32*ks + 8*(l/16) + 0..7 of row (row0 + l%16).
  // All lane-dependent address arithmetic is done once (lane_offsets); inside the K loop a
  // fragment address is a per-lane base plus a compile-time constant, which the LDS instructions
  // carry in their offset field.
  //   K-contiguous tile:   off[ks] for the wave's first MT rows; MT more rows = +MT*BK elements
  //                        (the swizzle repeats every 16 rows)
  //   row-contiguous tile: off[t] for the t-th group of MT columns at k-step 0;
  //                        k-step ks = +32*ks*ROWS elements, second half of the 8 k = +4*ROWS
  static constexpr int kOffs = 8;
  template <int ROWS, bool KC, int NTILE>
  __device__ static __forceinline__ void lane_offsets(int w0, int lane, uint32_t (&off)[kOffs]) {
    if (KC) {
      const int row = w0 + (lane & (MT - 1));
#pragma unroll
      for (int ks = 0; ks < KS; ks++) off[ks] = (row * BK + ((ks * (64 / MT) + lane / MT) ^ kc_swizzle(row)) * PE) * ES;
    } else {
      // transposing read: within 16 lanes, lane s points at 4 consecutive columns of k-row
      // kb + s/4, starting at column 4*(s%4); it receives k = kb..kb+3 of column s.
      const int s = lane & 15;
      const int k = 8 * (lane >> 4) + (s >> 2);
#pragma unroll
      for (int t = 0; t < NTILE; t++) {
        const int col = w0 + t * 16 + 4 * (s & 3);
        off[t] = (k * ROWS + (((col >> 3) ^ rc_swizzle<ROWS>(k)) << 3) + (col & 7)) * ES;
      }
    }
  }
  // how many of those offsets an operand has
  template <bool KC, int NTILE>
  static constexpr int n_offsets() { return KC ? KS : NTILE; }
  // fragment of tile t at k-step ks; `at`: LDS address of the operand's tile plus the lane's offsets, `plus` bytes further on
  template <typename P> __device__ static __forceinline__ const __attribute__((address_space(3))) P* lds_at(uint32_t a) {
    return (const __attribute__((address_space(3))) P*)(uintptr_t)a;
  }
  template <int ROWS, bool KC>
  __device__ static __forceinline__ frag_t frag(const uint32_t (&at)[kOffs], uint32_t plus, int t, int ks) {
    if constexpr (KC) {
      return __builtin_bit_cast(frag_t, *lds_at<u32x4_t>(at[ks] + (plus + t * MT * BK * ES)));
    } else {
      typedef __attribute__((address_space(3))) short4_t* lds_ptr;
      const uint32_t q = plus + ks * 32 * ROWS * ES;
      short4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(uintptr_t)(at[t] + q));
      short4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(uintptr_t)(at[t] + (q + 4 * ROWS * ES)));
      short8_t both = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
      return __builtin_bit_cast(frag_t, both);
    }
  }

  struct Frags {
    frag_t a[TM], b[NB][TN];
  };
  // the r-th fragment load of a k-step: first the TM fragments of A, then the NB*TN of B
  static constexpr int kFragLoads = TM + NB * TN;
  template <int ks, int r>
  __device__ static __forceinline__ void load_frag_n(const uint32_t (&la)[kOffs], const uint32_t (&lb)[kOffs], Frags& f) {
    if constexpr (r < TM) {
      f.a[r] = frag<BM, A_KC>(la, 0, r, ks);
    } else {
      constexpr int nb = (r - TM) / TN, j = (r - TM) % TN;
      f.b[nb][j] = frag<BN, B_KC>(lb, nb * B_ELEMS * ES, j, ks);
    }
  }
  // MFMA number m of a k-step.  Inline assembly with a memory clobber: the instruction stream of
  // the K loop is then exactly the order written in run() (LDS reads, tile loads and MFMAs
  // interleaved by hand), the compiler only allocates registers and inserts the waits.
  // Operands exchanged: result register r of lane l is C[m = l%16][n = 4*(l/16) + r]
  static constexpr int kMfma = NB * TM * TN;
  template <int m>
  __device__ static __forceinline__ void mfma_n(acc_t (&acc)[NB][TM][TN], const Frags& f) {
    constexpr int nb = m / (TM * TN), i = (m / TN) % TM, j = m % TN;
    asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0"
                 : "+a"(acc[nb][i][j])
                 : "v"(f.b[nb][j]), "v"(f.a[i])
                 : "memory");
  }

  // The same, with a tile load (see issue_one) in the instruction's shadow: the write of M0 before it, so that the
  // MFMA is the wait state that the load needs behind that write.  LDS address: base + plus.
  template <int m, int plus>
  __device__ static __forceinline__ void mfma_load_n(acc_t (&acc)[NB][TM][TN], const Frags& f, const rsrc_t& rsrc, uint32_t base,
                                                     uint32_t voff) {
    constexpr int nb = m / (TM * TN), i = (m / TN) % TM, j = m % TN;
    asm volatile("s_add_u32 m0, %3, %4\n\tv_mfma_f32_16x16x32_bf16 %0, %1, %2, %0\n\tbuffer_load_dwordx4 %5, %6, 0 offen lds"
                 : "+a"(acc[nb][i][j])
                 : "v"(f.b[nb][j]), "v"(f.a[i]), "s"(base), "n"(plus), "v"(voff), "s"(rsrc)
                 : "memory", "scc");
  }

  // Position of a stream of tile loads along K.  The K loop pays for every scalar instruction between
  // its MFMAs, so a step moves the descriptors' bases and byte counts by 32-bit constants, three additions each; the
  // segment functor is consulted only at the end of a run of steps (settle): where a segment starts, and before the steps add up
  // to more than 2 GiB (a byte count saturates at 4 GiB, and one iteration's tile spans at most 1 GiB of an operand whose
  // rows are K values).  Once the product is exhausted the steps are zero and the byte counts stay at
  // zero: loads issued from there on read nothing and deliver zeros.
  // byte offset beyond any descriptor's range (the operands of a tile span less than that: see the callers)
  static constexpr uint32_t kNowhere = 0xffffff00u;
  struct Cursor {
    rsrc_t ad, bd[NB];        // buffer descriptors of the A tile and the B tile(s) at this position
    uint32_t a_step, b_step;  // bytes by which one iteration moves the origins
    int k_left, k_step;       // valid values of K from the origins on
    int left;                 // steps until the run ends
    int end, sg;              // the iteration of segment sg where it does
  };
  // byte count of a descriptor: 32 bits, saturating (built from the halves: scalar instructions only)
  __device__ static __forceinline__ int clip_rem(int64_t v) {
    const int32_t hi = (int32_t)(v >> 32);
    return hi < 0 ? 0 : hi > 0 ? -1 : (int)(uint32_t)v;
  }
  __device__ static __forceinline__ rsrc_t make_desc(const T* base, int64_t bytes) {
    const uint64_t p = (uint64_t)base;
    rsrc_t r;
    r[0] = __builtin_amdgcn_readfirstlane((int)(uint32_t)p);
    r[1] = __builtin_amdgcn_readfirstlane((int)((uint32_t)(p >> 32) & 0xffffu));
    r[2] = __builtin_amdgcn_readfirstlane(clip_rem(bytes));
    r[3] = 0x00020000;
    return r;
  }
  // moves a descriptor by `step` bytes (the base stays below 2^48)
  __device__ static __forceinline__ void move_desc(rsrc_t& r, uint32_t step) {
    const uint64_t p = (((uint64_t)(uint32_t)r[1] << 32) | (uint32_t)r[0]) + step;
    r[0] = (int)(uint32_t)p;
    r[1] = (int)(uint32_t)(p >> 32);
    r[2] = (int)((uint32_t)r[2] - step);
  }
  // the run of steps that starts at iteration ki of segment sg
  template <class SegFn>
  __device__ static __forceinline__ void seek(Cursor& c, SegFn& segf, int sg, int ki, int n_segs, int nk, int64_t lda,
                                              int64_t ldb) {
    c.sg = sg;
    if (sg < n_segs && nk > 0) {
      const SegSrc<T, NB> g = segf(sg);
      const int64_t a_step = A_KC ? (int64_t)BK * ES : (int64_t)BK * ES * lda;
      const int64_t b_step = B_KC ? (int64_t)BK * ES : (int64_t)BK * ES * ldb;
      c.ad = make_desc((const T*)((const char*)g.a + ki * a_step), g.a_bytes - ki * a_step);
#pragma unroll
      for (int nb = 0; nb < NB; nb++) c.bd[nb] = make_desc((const T*)((const char*)g.b[nb] + ki * b_step), g.b_bytes - ki * b_step);
      // The words above come out of v_readfirstlane.  Five wait states must pass before a tile load reads
      // them, wherever the compiler places that load (a segment starts once or twice per tile, so this
      // costs nothing); the statements are tied to the descriptors and keep their order, so the wait
      // stands behind the last of those writes.
#pragma unroll
      for (int nb = 0; nb < NB; nb++) asm volatile("" : "+s"(c.bd[nb]) : : "memory");
      asm volatile("s_nop 4" : "+s"(c.ad) : : "memory");
      c.a_step = (uint32_t)a_step;
      c.b_step = (uint32_t)b_step;
      c.k_left = g.k_len - ki * BK;
      c.k_step = BK;
      const uint32_t most = A_KC && B_KC ? (uint32_t)(BK * ES) : max(c.a_step, c.b_step);
      c.left = nk - ki;
      if ((uint64_t)c.left * most > 0x80000000u) c.left = (int)(0x80000000u / most);
    } else {
      // exhausted (or nothing to do): zero-length descriptors that stay where they are
      c.a_step = c.b_step = 0;
      c.k_left = c.k_step = 0;
      c.left = 0x7fffffff;
      if (sg == 0) {
        c.ad = make_desc(nullptr, 0);
#pragma unroll
        for (int nb = 0; nb < NB; nb++) c.bd[nb] = make_desc(nullptr, 0);
      } else {
        c.ad[2] = 0;
#pragma unroll
        for (int nb = 0; nb < NB; nb++) c.bd[nb][2] = 0;
      }
    }
    c.end = ki + c.left;
  }
  // one iteration further (settle() must follow before the next load)
  __device__ static __forceinline__ void next(Cursor& c) {
    c.left--;
    move_desc(c.ad, c.a_step);
#pragma unroll
    for (int nb = 0; nb < NB; nb++) move_desc(c.bd[nb], c.b_step);
    c.k_left -= c.k_step;
  }
  template <class SegFn>
  __device__ static __forceinline__ void settle(Cursor& c, SegFn& segf, int n_segs, int nk, int64_t lda, int64_t ldb) {
    if (c.left == 0) {
      const bool done = c.end == nk;
      seek(c, segf, done ? c.sg + 1 : c.sg, done ? 0 : c.end, n_segs, nk, lda, ldb);
    }
  }

  // (the valid extents are not needed here: the descriptors' byte counts zero-fill the loads and bound
  // the epilogue's accesses)
  template <class SegFn, class Epi>
  __device__ static __forceinline__ void run(char* smem, int n_segs, int nk, SegFn segf, int64_t lda, int64_t ldb,
                                             const Epi& epi, const RowMap& amap) {
    const int n_iters = n_segs * nk;
    MOE_PHASE(0);
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wm0 = (wave / WN) * (BM / WM), wn0 = (wave % WN) * (BN / WN);

    acc_t acc[NB][TM][TN];
    // Called once the first tile loads are on their way, so that the AR * NB * TM * TN register
    // writes overlap their latency.
    auto zero_acc = [&]() __attribute__((always_inline)) {
#pragma unroll
      for (int nb = 0; nb < NB; nb++)
#pragma unroll
        for (int i = 0; i < TM; i++)
#pragma unroll
          for (int j = 0; j < TN; j++)
#pragma unroll
            for (int r = 0; r < AR; r++) acc[nb][i][j][r] = 0.f;
      // Pin the zeroing here.  Left alone, the compiler may materialise an accumulator's zeros right
      // in front of its first MFMA; that MFMA is inline assembly, so nobody would insert the wait
      // states a VALU write to an accumulator register needs before an MFMA reads it.
#pragma unroll
      for (int nb = 0; nb < NB; nb++)
#pragma unroll
        for (int i = 0; i < TM; i++)
#pragma unroll
          for (int j = 0; j < TN; j++) asm volatile("" : "+a"(acc[nb][i][j])::"memory");
      asm volatile("s_nop 7" ::: "memory");
    };

    // per-lane byte offsets of this wave's loads of a tile, fixed for the whole K loop
    uint32_t voa[A_NI], vob[B_NI];
#pragma unroll
    for (int j = 0; j < A_NI; j++)
      voa[j] = piece_offset<BM, A_KC>(wave + j * NW, lane, (uint32_t)lda);
    if constexpr (A_KC) {
      // gathered A rows: the same pieces, from the rows the map names.  The descriptor then spans the
      // whole operand, so the rows beyond the tile's valid ones get an offset no descriptor reaches
      // (they read as zero, as they do past the end of a plain tile).
      if (amap.gathered()) {
        const int q = wave * 64 + lane, row = q / PR_KC, c = (q % PR_KC) ^ kc_swizzle(row);
#pragma unroll
        for (int j = 0; j < A_NI; j++) {
          const int r = row + j * (64 / PR_KC) * NW;
          voa[j] = r < amap.rows ? (uint32_t)amap(r) * (uint32_t)lda * ES + (uint32_t)c * 16u : kNowhere;
        }
      }
    }
#pragma unroll
    for (int j = 0; j < B_NI; j++)
      vob[j] = piece_offset<BN, B_KC>(wave + j * NW, lane, (uint32_t)ldb);
    // LDS byte addresses: this wave's first piece of A slot 0 and of B slot 0
    const uint32_t lds_addr = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)smem;
    const uint32_t lds_a0 = lds_addr + (uint32_t)wave * 1024u;
    const uint32_t lds_b0 = lds_a0 + (uint32_t)(A_SLOTS * A_ELEMS * ES);
    // KTAIL: all-ones-like offsets for the lanes whose piece lies at or beyond the K values that are left (one
    // mask per stream of loads: the streams are at different iterations)
    const int pk = piece_k(wave, lane);
    uint32_t tail_a = 0, tail_b = 0;
    auto load_a = [&](const Cursor& c, int slot, int j) __attribute__((always_inline)) {
      issue_one(c.ad, lds_a0 + (uint32_t)(slot * A_ELEMS * ES) + (uint32_t)(j * NW) * 1024u,
                KTAIL && A_KC ? voa[j] | tail_a : voa[j]);
    };
    auto load_b = [&](const Cursor& c, int slot, int n) __attribute__((always_inline)) {
      const int nb = n / B_NI, j = n % B_NI;
      issue_one(c.bd[nb], lds_b0 + (uint32_t)((slot * B_SET_ELEMS + nb * B_ELEMS) * ES) + (uint32_t)(j * NW) * 1024u,
                KTAIL && B_KC ? vob[j] | tail_b : vob[j]);
    };
    // Loads beyond the last iteration still issue (the wait counts below stay constant and the K
    // loop free of branches): an exhausted cursor makes them read nothing.
    auto mask = [&](const Cursor& c, uint32_t& tail) __attribute__((always_inline)) {
      if (KTAIL) tail = pk < c.k_left ? 0u : kNowhere;
    };
    auto start = [&](Cursor& c) __attribute__((always_inline)) { seek(c, segf, 0, 0, n_segs, nk, lda, ldb); };
    auto settled = [&](Cursor& c) __attribute__((always_inline)) { settle(c, segf, n_segs, nk, lda, ldb); };
    auto step = [&](Cursor& c) __attribute__((always_inline)) {
      next(c);
      settled(c);
    };

    static_assert(TM <= kOffs && TN <= kOffs, "lane_offsets holds an offset per tile of an operand");
    uint32_t ao[kOffs], bo[kOffs];
    lane_offsets<BM, A_KC, TM>(wm0, lane, ao);
    lane_offsets<BN, B_KC, TN>(wn0, lane, bo);
    // LDS addresses of the fragments of the tile that is multiplied (`la`, `lb`), one of operand A or B at a time
    constexpr int kNA = n_offsets<A_KC, TM>(), kAddr = kNA + n_offsets<B_KC, TN>();
    uint32_t la[kOffs], lb[kOffs];
    auto set_address = [&](auto xc, uint32_t a_tile, uint32_t b_tile) __attribute__((always_inline)) {
      constexpr int x = decltype(xc)::value;
      if constexpr (x < kNA) la[x] = ao[x] + a_tile;
      else lb[x - kNA] = bo[x - kNA] + b_tile;
    };
    constexpr uint32_t kABytes = A_ELEMS * ES, kBBytes = B_SET_ELEMS * ES;
    const uint32_t lds_b = lds_addr + A_SLOTS * kABytes;
    static_for<kAddr>([&](auto x) __attribute__((always_inline)) { set_address(x, lds_addr, lds_b); });

    constexpr int kLoadsB = NB * B_NI;  // loads per wave for the B tiles of one iteration
    // Fragments are read a few MFMAs (16 cycles each) before the k-step that needs them starts.
    constexpr int kHalf = kMfma / 2, kLate = kMfma - kHalf;
    constexpr int kLead = kMfma / 8 < 8 ? kMfma / 8 : 8;
    constexpr int kSpan = kMfma - kLead, kLateSpan = kLate - kLead;
    // the loads of an iteration are spread over these MFMAs: all before the barrier
    constexpr int kSlots = (KS - 1) * kMfma + kHalf;
    Frags f[2];
    auto first_frags = [&]() __attribute__((always_inline)) {
      static_for<kFragLoads>([&](auto r) __attribute__((always_inline)) { load_frag_n<0, decltype(r)::value>(la, lb, f[0]); });
    };
    // What an iteration does ahead of its MFMA number `slot` besides tile loads: the fragments of the next k-step (of the last
    // one's: of the next tile, behind the barrier), spread over the k-step's MFMAs; ahead of the barrier the addresses of the
    // next tile's fragments.  (After the last tile this reads stale but in-bounds LDS data that is never used.)
    auto ahead = [&](auto slot_c, uint32_t a_next, uint32_t b_next, auto barrier) __attribute__((always_inline)) {
      constexpr int slot = decltype(slot_c)::value, ks = slot / kMfma, m = slot % kMfma;
      if constexpr (ks < KS - 1) {
        constexpr int r0 = std::min(m * kFragLoads / kSpan, kFragLoads), r1 = std::min((m + 1) * kFragLoads / kSpan, kFragLoads);
        static_for<r1 - r0>([&](auto r) __attribute__((always_inline)) {
          load_frag_n<ks + 1, r0 + decltype(r)::value>(la, lb, f[(ks + 1) & 1]);
        });
      } else if constexpr (m < kHalf) {
        constexpr int x0 = m * kAddr / kHalf, x1 = (m + 1) * kAddr / kHalf;
        static_for<x1 - x0>([&](auto x) __attribute__((always_inline)) {
          set_address(std::integral_constant<int, x0 + decltype(x)::value>(), a_next, b_next);
        });
      } else {
        if constexpr (m == kHalf) barrier();
        constexpr int h = m - kHalf;
        constexpr int r0 = std::min(h * kFragLoads / kLateSpan, kFragLoads), r1 = std::min((h + 1) * kFragLoads / kLateSpan, kFragLoads);
        static_for<r1 - r0>([&](auto r) __attribute__((always_inline)) { load_frag_n<0, r0 + decltype(r)::value>(la, lb, f[0]); });
      }
    };
    if constexpr (DEPTH >= 2) {
      // streaming pipeline: tiles t .. t+DEPTH-1 in flight while tile t is multiplied
      constexpr int L = A_NI + kLoadsB;  // loads per wave and iteration
      static_assert((DEPTH - 1) * L <= 63, "the wait count of the oldest tile must be encodable");
      Cursor s0;  // the next tile to request
      start(s0);
      auto issue_tile = [&](int it) __attribute__((always_inline)) {
        const int slot = it % (DEPTH + 1);
        mask(s0, tail_a);
        tail_b = tail_a;
#pragma unroll
        for (int j = 0; j < A_NI; j++) load_a(s0, slot, j);
#pragma unroll
        for (int n = 0; n < kLoadsB; n++) load_b(s0, slot, n);
        step(s0);
      };
      if (n_iters > 0) {
        for (int it = 0; it < DEPTH; it++) issue_tile(it);
      }
      zero_acc();
      // Tile t has landed once at most the DEPTH - 1 younger tiles are outstanding (loads complete in order).
      auto landed = [&]() __attribute__((always_inline)) {
        asm volatile("s_waitcnt vmcnt(%0)" ::"n"((DEPTH - 1) * L) : "memory");
        __syncthreads();
      };
      landed();
      // The instruction stream of an iteration t, as in the ring below: the L loads of tile t + DEPTH are spread
      // between the MFMAs, the fragments of the next k-step are read under those of the current one, and the
      // barrier stands half-way through the last k-step, so that the first fragments of tile t + 1 are read under
      // MFMAs too.  That barrier says that tile t + 1 is there and that every wave is done with tile t, whose slot the
      // loads of the next iteration overwrite.
      // (Reads before, then all loads, then all MFMAs of an iteration: the loads of four waves alone hold the
      // address unit for 16 cycles each, 768 of the 1950 cycles of a 128-row step.  Down product of 4 shared experts, T = 2777,
      // 176 tiles of 128 rows and 88 steps: 124 -> 79 us, 1.35 -> 0.83 us a step.)
      static_assert(L <= kSlots, "at most one load per MFMA");
      first_frags();
      int cur = 0;
      uint32_t fill_a = lds_a0 + DEPTH * kABytes, fill_b = lds_b0 + DEPTH * kBBytes;  // slot of tile t + DEPTH
      for (int it = 0; it < n_iters; it++) {
        const int nxt = cur == DEPTH ? 0 : cur + 1;
        mask(s0, tail_a);
        tail_b = tail_a;
        static_for<KS * kMfma>([&](auto slot_c) __attribute__((always_inline)) {
          constexpr int slot = decltype(slot_c)::value, ks = slot / kMfma, m = slot % kMfma, n = slot * L / kSlots;
          ahead(slot_c, lds_addr + nxt * kABytes, lds_b + nxt * kBBytes, landed);
          if constexpr (slot < kSlots && n < (slot + 1) * L / kSlots) {
            if constexpr (n < A_NI) {
              mfma_load_n<m, n * NW * 1024>(acc, f[ks & 1], s0.ad, fill_a, KTAIL && A_KC ? voa[n] | tail_a : voa[n]);
            } else {
              constexpr int nb = (n - A_NI) / B_NI, j = (n - A_NI) % B_NI;
              mfma_load_n<m, nb * B_ELEMS * ES + j * NW * 1024>(acc, f[ks & 1], s0.bd[nb], fill_b, KTAIL && B_KC ? vob[j] | tail_b : vob[j]);
            }
          } else {
            mfma_n<m>(acc, f[ks & 1]);
          }
          if constexpr (slot == kSlots) next(s0);  // behind the last load
        });
        settled(s0);
        fill_a = lds_a0 + cur * kABytes;
        fill_b = lds_b0 + cur * kBBytes;
        cur = nxt;
      }
    } else if constexpr (!RING) {
      // single slot: load a tile, wait, multiply; k-steps beyond the rows of K are skipped
      Cursor s0;
      start(s0);
      zero_acc();
      for (int it = 0; it < n_iters; it++) {
        if (it > 0) __syncthreads();
        mask(s0, tail_a);
        tail_b = tail_a;
#pragma unroll
        for (int j = 0; j < A_NI; j++) load_a(s0, 0, j);
#pragma unroll
        for (int n = 0; n < kLoadsB; n++) load_b(s0, 0, n);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        static_for<KS>([&](auto ks_c) __attribute__((always_inline)) {
          constexpr int ks = decltype(ks_c)::value;
          if (ks * (BK / KS) >= s0.k_left) return;  // uniform: the remaining k rows of the tile are zero
          // (one A fragment ahead, no more: the registers of four blocks per CU have no room for all of them)
          static_assert(NB == 1, "one row of accumulator tiles after the other");
          static_for<TN + 1>([&](auto r) __attribute__((always_inline)) { load_frag_n<ks, (decltype(r)::value + TM) % (TM + TN)>(la, lb, f[0]); });
          static_for<TM>([&](auto i) __attribute__((always_inline)) {
            if constexpr (decltype(i)::value + 1 < TM) load_frag_n<ks, decltype(i)::value + 1>(la, lb, f[0]);
            static_for<TN>([&](auto j) __attribute__((always_inline)) { mfma_n<decltype(i)::value * TN + decltype(j)::value>(acc, f[0]); });
          });
        });
        step(s0);
      }
    } else {
    Cursor s1, s2;  // s1: the B tiles of iteration it + 1; s2: the A tile of iteration it + 2
    start(s1);
    start(s2);
    mask(s1, tail_b);
    mask(s2, tail_a);
    if (n_iters > 0) {
#pragma unroll
      for (int j = 0; j < A_NI; j++) load_a(s2, 0, j);
#pragma unroll
      for (int n = 0; n < kLoadsB; n++) load_b(s1, 0, n);
      step(s1);
      step(s2);
      mask(s1, tail_b);
      mask(s2, tail_a);
#pragma unroll
      for (int j = 0; j < A_NI; j++) load_a(s2, 1, j);
      step(s2);
      mask(s2, tail_a);
    }
    zero_acc();
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    MOE_PHASE(1);

    // A wave issues in order and a tile load holds it for as long as the memory pipeline has no
    // free slot, so the overlap of loads, LDS reads and MFMAs is written into the instruction
    // stream itself.  Per K iteration t (KS k-steps
    // of kMfma MFMAs):
    //   - the fragments of k-step ks+1 are read from LDS during the MFMAs of ks;
    //   - the loads of B(t+1), then of A(t+2), are spread evenly between the MFMAs;
    //   - half-way through the last k-step all LDS reads of this iteration are done: wait until
    //     B(t+1) has landed (A(t+2) may still be in flight: loads complete in order), barrier, and
    //     read the first fragments of iteration t+1 under the remaining MFMAs.
    // What else an iteration needs is spread between the MFMAs too: a step of a cursor behind its last load, the addresses of
    // the next tile's fragments ahead of the barrier.
    constexpr int kLoads = kLoadsB + A_NI;
    static_assert(kLoads <= kSlots, "at most one load per MFMA");
    first_frags();
    auto landed = [&]() __attribute__((always_inline)) {
      // B(t+1) must have landed (the A_NI loads of A(t+2) issued after it may still be
      // outstanding), and every wave must be done reading this iteration's tiles
      asm volatile("s_waitcnt vmcnt(%0)" ::"n"(A_NI) : "memory");
      __syncthreads();
    };
    // slots: A(t+1) to multiply next, A(t+2) and B(t+1) to fill
    uint32_t a_nxt = kABytes, a_nn = 2 * kABytes, a_cur = 0, b_nxt = kBBytes;
    for (int it = 0; it < n_iters; it++) {
      static_for<KS * kMfma>([&](auto slot_c) __attribute__((always_inline)) {
        constexpr int slot = decltype(slot_c)::value, ks = slot / kMfma, m = slot % kMfma, n = slot * kLoads / kSlots;
        ahead(slot_c, lds_addr + a_nxt, lds_b + b_nxt, landed);
        if constexpr (slot < kSlots && n < (slot + 1) * kLoads / kSlots) {
          if constexpr (n < kLoadsB) {
            constexpr int nb = n / B_NI, j = n % B_NI;
            mfma_load_n<m, nb * B_ELEMS * ES + j * NW * 1024>(acc, f[ks & 1], s1.bd[nb], lds_b0 + b_nxt, KTAIL && B_KC ? vob[j] | tail_b : vob[j]);
          } else {
            constexpr int j = n - kLoadsB;
            mfma_load_n<m, j * NW * 1024>(acc, f[ks & 1], s2.ad, lds_a0 + a_nn, KTAIL && A_KC ? voa[j] | tail_a : voa[j]);
          }
          if constexpr (n == kLoadsB - 1) next(s1);
        } else {
          mfma_n<m>(acc, f[ks & 1]);
        }
        if constexpr (slot == kSlots) next(s2);
      });
      settled(s1);
      settled(s2);
      mask(s1, tail_b);
      mask(s2, tail_a);
      const uint32_t a_old = a_cur;
      a_cur = a_nxt;
      a_nxt = a_nn;
      a_nn = a_old;
      b_nxt = kBBytes - b_nxt;
    }
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // zero-length loads of the tail
    MOE_PHASE(2);
    // The accumulators live in AGPRs.  Each value is copied out right where it is needed (the
    // volatile asm pins the order); left to itself the compiler copies all 256 at the loop exit,
    // needs every arch VGPR for that and spills the loop's address registers.
    // The MFMAs above are opaque to the compiler's hazard recogniser, so the wait between the last
    // MFMA (4 passes of 4 cycles, plus write-back) and the first read of any accumulator is
    // explicit: 6 x 16 idle cycles, attached to the accumulator of the last MFMA.  The empty
    // statements make every other accumulator depend on a point after that wait (volatile asm
    // statements keep their order), so no compiler-generated accumulator copy can move above it.
    asm volatile("s_nop 15\n\ts_nop 15\n\ts_nop 15\n\ts_nop 15\n\ts_nop 15\n\ts_nop 15"
                 : "+a"(acc[NB - 1][TM - 1][TN - 1])
                 :
                 : "memory");
#pragma unroll
    for (int nb = 0; nb < NB; nb++)
#pragma unroll
      for (int i = 0; i < TM; i++)
#pragma unroll
        for (int j = 0; j < TN; j++) asm volatile("" : "+a"(acc[nb][i][j])::"memory");
    __syncthreads();  // every wave is done with the tile slots (stale fragment reads included)
    TileEpilogue<NB, TM, TN, NW, LDS_BYTES, true>::run(smem, acc, epi, wave, lane, wm0, wn0);
    MOE_PHASE(3);
  }
};

}  // namespace moe
