// Tile plan and argument blocks of the grouped GEMMs (device side).
#pragma once

#include "moe_common.h"

namespace moe {

// One row tile of a grouped GEMM whose C rows are token rows.
struct RowTile {
  int32_t group;     // expert that owns the rows
  int32_t row0_in;   // first row in the [n_rows, .] input/output of the call
  int32_t rows;      // valid rows (<= tile height) in bits 0..15, tile kind in bits 16..17 (height: that of the full tile >> kind)
  int32_t row0_out;  // first row in the per-group saved activations (differs in shared mode)
};

__host__ __device__ inline int tile_rows(const RowTile& t) { return t.rows & 0xffff; }
__host__ __device__ inline int tile_kind(const RowTile& t) { return (t.rows >> 16) & 3; }
// row tiles per band of the XCD-aware tile order of the LDS-DMA path
constexpr int kBandRows = 4;
// Launches of at most so many rounds of 256 row tiles deal them to the XCDs in short runs.  (Long runs above this line against short
// ones everywhere, training steps of d = d_ff = 4096, 8 experts, whose gate/up launch has twice the rounds given: 6.5 rounds 6475 and
// 6445 us, 7 6818 and 6846, 8 7711 and 7798, 9 8631 and 8726, 10 9576 and 9691; for launches below it see row_gemm_block.)
constexpr int kFineRounds = 6;

// Device-built plan, laid out in the workspace.
struct Plan {
  RowTile* tiles;      // [max_tiles]
  int32_t* n_tiles;    // [1]
  int4* ginfo;         // [n_groups] {group, rows, first row, compact slot} by descending row count
};

inline size_t plan_bytes(int n_groups, int max_tiles) {
  return align_up((size_t)max_tiles * sizeof(RowTile), 256) + 256 + align_up((size_t)n_groups * sizeof(int4), 256);
}

inline Plan carve_plan(void* ws, int /*n_groups*/, int max_tiles) {
  char* p = (char*)ws;
  Plan pl;
  pl.tiles = (RowTile*)p;
  p += align_up((size_t)max_tiles * sizeof(RowTile), 256);
  pl.n_tiles = (int32_t*)p;
  p += 256;
  pl.ginfo = (int4*)p;
  return pl;
}

// Bf16 calls of few rows whose products are short take small tiles (Cores<PATH_BF16_SMALL>): with four times as many, two on a CU,
// such launches fill the chip, and a tile's own latency is what counts.  Their plans have tiles of 64 rows only.  Three lines:
//  rows x d: below it tall tiles would not fill the chip.  (Passes before, on the full family's tiles, and now: T = 911, d = 128, 4 experts of
//    1088 and four shared, 0.1 million, training 173 and 98 us; T = 1190, top-4, d = 344, 85 experts of 400, 1.6 million, 177 and 146; T = 9871,
//    top-2, d = 128, 133 experts of 384, 2.4 million, 361 and 288; T = 243, top-6, d = 2304, 31 experts of 128, 3.2 million, 143 and 117; T = 6330,
//    d = 600, 166 experts of 384, 3.6 million, forward 101 and 104.)
//  bytes of a matrix of the groups that may have rows: above it the stream of the weights counts, and the full family reads twice as long
//    pieces of their rows.  A compromise: what decides is how many of the full family's tiles the groups have that do get rows, which the
//    host does not know.  (373 drawn passes with up to 128 of those in the smaller of the two forward products gain 20 %, 11 of them lose more than 1 %;
//    147 with more gain 3 %, 44 lose.)  Bytes rule out most of the latter: of 300 drawn passes 263 lie below the line and gain 19 %, 15 lose more
//    than 1 % and up to 11; 37 lie above, up to 2 GB, and would gain 7 %, 10 lose up to 10.  Near the line families take turns on either side
//    of it: T = 16 to 64, d = 2048, 48 to 128 experts of 1280 to 2048, 240 to 700 MB, forward, lose 8 % to gain 4 % without shared experts; with four
//    of 1408 beside them 330 MB takes 111 and 106 us, 352 MB 119 and 110.
//  arithmetic of a product: above it the matrix pipe counts.  (6 GFLOP, training 534 and 429 us; 14 GFLOP 747 and 758; 33 GFLOP, forward 377
//    and 418.)
constexpr int kFewRowValues = 13 << 18;
inline bool few_rows(int dtype, int64_t n_rows, int d) { return dtype != MOE_F32 && n_rows * d <= kFewRowValues; }
inline bool short_product(int64_t n_rows, int64_t d, int64_t d_ff) { return 2 * n_rows * d * d_ff <= 16000000000; }
inline bool small_tiles(int dtype, int n_groups, int n_rows, int d, int d_ff) {
  return few_rows(dtype, n_rows, d) && short_product(n_rows, d, d_ff) &&
         2 * (int64_t)(n_groups < n_rows ? n_groups : n_rows) * d * d_ff <= (int64_t)340 << 20;
}
// rows of the full row tiles of a plan
constexpr int kSmallTileRows = 64, kSmallTileKind = 2;  // (64-row tiles are kind 2 of the full family, too)
inline int plan_tile_rows(int dtype, int n_groups, int n_rows, int d, int d_ff) {
  return dtype == MOE_F32 ? 128 : small_tiles(dtype, n_groups, n_rows, d, d_ff) ? kSmallTileRows : 256;
}
// Room for the row tiles of any plan, whatever its tiles.  A dispatch and the calls that use its plan may disagree on those (they need not be
// given the same width), so the layout does not depend on them, and every family takes any plan.
inline int plan_cap(int n_groups, int n_rows) { return n_rows / 64 + 2 * n_groups; }
// upper bound of the row tiles that a plan can have (at most two remainder tiles per group; of 64-row tiles one)
inline int max_row_tiles(int dtype, int n_groups, int n_rows, int d) {
  const int g = n_groups < n_rows ? n_groups : n_rows, tall = n_rows / (dtype == MOE_F32 ? 128 : 256) + 2 * g;
  return few_rows(dtype, n_rows, d) && n_rows / kSmallTileRows + g > tall ? n_rows / kSmallTileRows + g : tall;
}

// One block of 1024 threads; thread e owns group e, which has c rows from row st on.  Bound by latency, nothing runs beside it: the pass
// for the group ranks takes four row counts per LDS read, the scans use one barrier each, and every tile has its own
// thread, which finds the group by bisection.  (Scans of ten steps with two barriers each, one row count per read and the
// tiles of a group written by one thread took: 60 groups 8.6 us, 64 groups 9.3, 8 groups 5.3; this form 6.6, 6.7, 3.7,
// as a launch of its own.)
__device__ __forceinline__ void build_plan(int c, int st, int n_groups, int BM, const Plan& pl, int32_t* active_ids, int32_t* n_active) {
  __shared__ __align__(16) int32_t rows_of[1024];                    // by group
  __shared__ int32_t cnt[1024], first[1024], tile0[1024], ord[1024];  // by rank
  __shared__ __align__(16) int32_t wsum[2][16];
  const int e = threadIdx.x;
  rows_of[e] = e < n_groups ? c : -1;
  int total_active;
  const int slot = block_scan_1024(e < n_groups && c > 0, wsum[0], total_active) - 1;
  if (e < n_groups) {
    // Launch order of the groups: descending row count (ties: ascending id), so that the short tiles
    // of the light groups fill the end of a launch.  Of the other wavefronts' groups the earlier ones precede
    // this one in a tie.
    const int own = e & ~(kWave - 1);
    int rank = 0;
    auto count = [&](int from, int to, int limit) __attribute__((always_inline)) {  // groups of more rows than `limit`
#pragma unroll 4
      for (int o = from; o < to; o += 4) {
        const int4 q = *reinterpret_cast<const int4*>(rows_of + o);
        rank += (q.x > limit) + (q.y > limit) + (q.z > limit) + (q.w > limit);
      }
    };
    count(0, own, c - 1);
#pragma unroll 4
    for (int o = own; o < min(own + kWave, n_groups); o++) rank += rows_of[o] > (o < e ? c - 1 : c);
    count(own + kWave, n_groups, c);
    ord[rank] = e;
    cnt[rank] = c;
    first[rank] = st;
    pl.ginfo[rank] = make_int4(e, c, st, c > 0 ? slot : -1);
    if (active_ids) {
      if (c > 0) active_ids[slot] = e;
      if (e >= total_active) active_ids[e] = -1;
    }
  }
  if (e == 0 && n_active) *n_active = total_active;
  __syncthreads();
  // Row tiles, groups in descending size: full tiles of BM rows, and the remainder r of a group cut into tiles of
  // BM/2, BM/4 and BM/8 rows so that little MFMA work is spent on padding; in eighths of BM: r > 6: one full tile;
  // (5,6]: 4 + 2; (4,5]: 4 + 1; (3,4]: 4; (2,3]: 2 + 1; (1,2]: 2; (0,1]: 1.  Tiles of one height: always a full one.
  auto eighths = [&](int rows) { return BM == kSmallTileRows ? (rows % BM ? 8 : 0) : ((rows % BM) * 8 + BM - 1) / BM; };
  const int cg = e < n_groups ? cnt[e] : 0;
  const int r8 = eighths(cg);
  const int nt = cg / BM + (r8 > 0) + (r8 == 3 || r8 == 5 || r8 == 6);
  int n_tiles;
  const int end = block_scan_1024(nt, wsum[1], n_tiles);
  tile0[e] = end - nt;
  if (e == 0) *pl.n_tiles = n_tiles;
  __syncthreads();
  for (int i = e; i < n_tiles; i += 1024) {
    int lo = 0, hi = n_groups;  // the last group whose tiles start at or before i (groups without tiles come last)
    while (hi - lo > 1) {
      const int mid = (lo + hi) >> 1;
      if (tile0[mid] <= i) lo = mid;
      else hi = mid;
    }
    const int rows = cnt[lo], full = rows / BM, r = eighths(rows), in_group = i - tile0[lo];
    const int k0 = r > 6 ? 0 : r > 3 ? 1 : r > 1 ? 2 : 3;  // kinds (heights BM >> kind) of the remainder's tiles
    const int k1 = r == 6 ? 2 : 3;
    const int kind = in_group < full ? 0 : in_group == full ? k0 : k1;
    const int row = min(in_group, full) * BM + (in_group > full ? BM >> k0 : 0);
    RowTile t;
    t.group = ord[lo];
    t.row0_in = first[lo] + row;
    t.rows = min(BM >> kind, rows - row) | ((BM == kSmallTileRows ? kSmallTileKind : kind) << 16);
    t.row0_out = t.row0_in;
    pl.tiles[i] = t;
  }
}

// C[rows, N] (+ second C when dual) = sum over (pair, seg) of A_seg[rows, K] * B_seg[K, N]
struct RowGemm {
  const RowTile* tiles;     // NULL: no plan, n_groups groups of n_rows rows in tiles of one height
  const int32_t* n_tiles;
  int32_t n_rows;
  // without a plan:
  int32_t n_groups;
  int32_t direct_kind;      // tile kind: height of the full tile >> kind
  int32_t n_parts, k_part;  // the values of K of a segment are summed in n_parts parts of k_part
  int32_t part_blocks;      // blocks of one part
  float* part;              // n_parts > 1: fp32 sums [n_parts][products][part_stride]
  int64_t part_stride;
  int32_t N, K;
  int32_t n_pairs, n_segs;
  const void* A[2];         // per pair; element (row, k) at A + seg*a_seg + row*lda + k
  int64_t lda, a_seg;
  int32_t a_rows_out;       // A rows are indexed by row0_out (saved activations) instead of row0_in
  // gathered A (pair 0, single segment, K-contiguous A only): row r of the call reads row
  // a_index[r] / a_index_div of A, which has a_src_rows rows (NULL: A is indexed by r itself)
  const int32_t* a_index;
  int32_t a_index_div, a_src_rows;
  const void* B[2];         // per pair; + group*b_group + seg*b_seg
  const void* Bdual;        // second B of a dual GEMM (pair 0 only)
  int64_t ldb, b_group, b_seg;
  // epilogue
  void* out[3];
  const void* in[2];
  // activation-backward epilogues: row r of the product is scaled by c_scale[a_index[r]] first (NULL: 1)
  const float* c_scale;
  int64_t ldc;
  int32_t c_rows_out;       // outputs indexed by row0_out
  int32_t wide;             // rows too long for the tile cores (see wide_rows)
};

// per group: C[M, N] = A_g^T B_g over the rows of the group (K = rows of the group)
struct WGemm {
  const int4* ginfo;        // per launch index (descending rows): {group, rows, first row, compact slot}; NULL: no plan
  int32_t n_rows, n_groups;
  // without a plan:
  int32_t n_parts, k_part;  // the rows are summed in n_parts parts of k_part
  float* part;              // n_parts > 1: fp32 sums [n_parts][products][part_stride]
  int64_t part_stride;
  int32_t *active_ids, *n_active;  // all groups, if not NULL
  int32_t M, N;
  const void* A;            // element (row, m) at A + row*lda + m
  int64_t lda;
  int32_t a_per_group;      // shared mode: A rows of group g start at g*n_rows
  const void* B[2];         // element (row, n) at B + row*ldb + n; B[1]: second product (dual GEMM, or second pass)
  int64_t ldb;
  int32_t b_per_group;
  void* C[2];
  int64_t c_slot;           // elements per slot
  int32_t k_min, k_max;     // only groups with k_min <= rows <= k_max are processed by this launch
  int32_t n_reps;           // consecutive column tiles per block (0 or 1: one)
  int32_t wide;             // rows too long for the tile cores (see wide_rows)
};

}  // namespace moe
