// moe_expert_fwd / moe_expert_bwd: the expert bodies of Eq. 3 (SwiGLU reading of Eq. 1) as
// grouped GEMMs over variable per-expert row counts, and their backward pass.
//
// Forward   F4: [G | U] = Xin_e [Wg_e | Wu_e],  H = silu(G) * U   (dual GEMM, fused epilogue)
//           F5: Yout_e = H_e Wd_e
// Backward  B2a: dH = dYin_e Wd_e^T, epilogue -> dG, dU           (reads the saved G, U)
//           B2b: dXin_e = dG_e Wg_e^T + dU_e Wu_e^T               (two K segments)
//           B3 : dWd_e = H_e^T dYin_e;  [dWg_e | dWu_e] = Xin_e^T [dG_e | dU_e]
// A device-built plan turns the row offsets into a list of row tiles (largest group first,
// groups without rows contribute nothing) so that no host synchronisation is needed.
#include <algorithm>
#include <atomic>

#include "gemm_cores.h"
#include "gemm_plan.h"

namespace moe {

// ------------------------------------------------------------------------------------ plan
__device__ __forceinline__ void block_scan_inclusive(int32_t* sc, int e) {
  for (int step = 1; step < 1024; step <<= 1) {
    int add = e >= step ? sc[e - step] : 0;
    __syncthreads();
    sc[e] += add;
    __syncthreads();
  }
}

// One block of 1024 threads; thread e owns group e.
__global__ __launch_bounds__(1024) void plan_kernel(const int32_t* __restrict__ offsets, int n_groups,
                                                    int n_rows, int BM, Plan pl, int32_t* active_ids,
                                                    int32_t* n_active) {
  __shared__ int32_t cnt[1024], sc[1024], ord[1024], st_[1024];
  const int e = threadIdx.x;
  int c = 0, st = 0;
  if (e < n_groups) {
    if (offsets) {
      st = offsets[e];
      c = offsets[e + 1] - st;
      if (c < 0) c = 0;
    } else {
      c = n_rows;
    }
  }
  cnt[e] = e < n_groups ? c : -1;
  st_[e] = st;
  sc[e] = (e < n_groups && c > 0) ? 1 : 0;
  __syncthreads();
  // Launch order of the groups: descending row count (ties: ascending id), so that the short tiles
  // of the light groups fill the end of a launch.
  int rank = 0;
  if (e < n_groups) {
    for (int o = 0; o < n_groups; o++) {
      int co = cnt[o];
      rank += (co > c) || (co == c && o < e);
    }
    ord[rank] = e;
  }
  __syncthreads();
  st_[e] = st;
  sc[e] = (e < n_groups && c > 0) ? 1 : 0;
  __syncthreads();
  block_scan_inclusive(sc, e);
  const int total_active = sc[1023];
  if (e < n_groups) {
    const int slot = c > 0 ? sc[e] - 1 : -1;
    if (active_ids) {
      if (slot >= 0) active_ids[slot] = e;
      if (e >= total_active) active_ids[e] = -1;
    }
  }
  if (e < n_groups) pl.ginfo[rank] = make_int4(e, c, st, c > 0 ? sc[e] - 1 : -1);
  if (e == 0 && n_active) *n_active = total_active;
  __syncthreads();
  // Row tiles, groups in descending size: full tiles of BM rows, and the remainder r of a group cut into tiles of
  // BM/2, BM/4 and BM/8 rows so that little MFMA work is spent on padding; in eighths of BM: r > 6: one full tile; (5,6]: 4 + 2; (4,5]: 4 + 1; (3,4]: 4; (2,3]: 2 + 1; (1,2]: 2; (0,1]: 1.
  const int g = e < n_groups ? ord[e] : 0;
  const int cg = e < n_groups ? cnt[g] : 0;
  const int full = cg / BM;
  int k0 = -1, k1 = -1;  // kinds (heights BM >> kind) of the up to two remainder tiles
  const int r8 = ((cg - full * BM) * 8 + BM - 1) / BM;  // eighths of BM, rounded up
  if (r8 > 6) k0 = 0;
  else if (r8 > 4) { k0 = 1; k1 = r8 == 6 ? 2 : 3; }
  else if (r8 == 4) k0 = 1;
  else if (r8 == 3) { k0 = 2; k1 = 3; }
  else if (r8 == 2) k0 = 2;
  else if (r8 == 1) k0 = 3;
  const int nt = full + (k0 >= 0) + (k1 >= 0);
  sc[e] = nt;
  __syncthreads();
  block_scan_inclusive(sc, e);
  const int base = sc[e] - nt;
  int row = 0;
  for (int i = 0; i < nt; i++) {
    const int kind = i < full ? 0 : (i == full ? k0 : k1);
    const int h = BM >> kind;
    RowTile t;
    t.group = g;
    t.row0_in = st_[g] + row;
    t.rows = min(h, cg - row) | (kind << 16);
    t.row0_out = offsets ? t.row0_in : g * n_rows + row;
    pl.tiles[base + i] = t;
    row += h;
  }
  if (e == 1023) *pl.n_tiles = sc[1023];
}

// ------------------------------------------------------------------------------- epilogues
enum { EPI_STORE = 0, EPI_SWIGLU_FWD = 1, EPI_SWIGLU_BWD = 2, EPI_STORE_F32 = 3, EPI_ADD = 4, EPI_GELU_FWD = 5,
       EPI_GELU_BWD = 6 };

// gelu(z) = z Phi(z) and its derivative Phi(z) + z phi(z) (Phi, phi: standard normal distribution
// function and density); the activation of the two-matrix expert.  `e` receives exp(-z^2 / 2).
// fp32 path: the library's erf and exp.  bf16 path (the result is rounded to bf16 anyway): the
// rational-times-exponential approximation of erf (Abramowitz & Stegun 7.1.26, absolute error below
// 1.5e-7) on the hardware's exp and reciprocal, a quarter of the instructions.
template <typename T> __device__ __forceinline__ float normal_cdf_(float z, float& e);
template <> __device__ __forceinline__ float normal_cdf_<float>(float z, float& e) {
  e = expf(-0.5f * z * z);
  return 0.5f * (1.f + erff(z * 0.70710678118654752f));
}
template <> __device__ __forceinline__ float normal_cdf_<bf16_t>(float z, float& e) {
  const float x = fabsf(z) * 0.70710678118654752f;
  const float t = __builtin_amdgcn_rcpf(1.f + 0.3275911f * x);
  e = __expf(-x * x);
  const float poly = t * (0.254829592f + t * (-0.284496736f + t * (1.421413741f + t * (-1.453152027f + t * 1.061405429f))));
  const float half_erfc = 0.5f * poly * e;  // (1 - erf(x)) / 2
  return z < 0.f ? half_erfc : 1.f - half_erfc;
}
template <typename T> __device__ __forceinline__ float gelu_f(float z) {
  float e;
  return z * normal_cdf_<T>(z, e);
}
template <typename T> __device__ __forceinline__ float gelu_grad_f(float z) {
  float e;
  const float cdf = normal_cdf_<T>(z, e);
  return cdf + z * 0.3989422804014327f * e;
}

// precise for the fp32 path; hardware exp and reciprocal where the result is rounded to bf16 anyway
template <typename T> __device__ __forceinline__ float sigmoidf_(float z);
template <> __device__ __forceinline__ float sigmoidf_<float>(float z) { return 1.f / (1.f + expf(-z)); }
template <> __device__ __forceinline__ float sigmoidf_<bf16_t>(float z) {
  return __builtin_amdgcn_rcpf(1.f + __expf(-z));
}

// Epilogue object of the tile cores (see gemm_cores.h): four consecutive values of every output from four of
// every product.
template <typename T, int NB, int EPI>
struct Epilogue {
  static constexpr int NOUT = EPI == EPI_SWIGLU_FWD ? 3 : (EPI == EPI_GELU_FWD || EPI == EPI_SWIGLU_BWD) ? 2
                              : EPI == EPI_STORE ? NB : 1;
  static constexpr int NAUX = EPI == EPI_SWIGLU_BWD ? 2 : (EPI == EPI_GELU_BWD || EPI == EPI_ADD) ? 1 : 0;
  static constexpr int OES = EPI == EPI_STORE_F32 ? 4 : sizeof(T);
  // bf16 outputs carry the streaming hint: every one is read again only by a later kernel, after gigabytes of
  // other traffic (2-3 % on the row GEMMs of the Qwen- and stress-shaped workloads)
  static constexpr bool NT = OES == 2;
  void* out[NOUT];
  const void* in[NAUX > 0 ? NAUX : 1];
  int64_t ldc;
  int rows, n_valid;
  // activation-backward epilogues of gathered rows: row m of the product is scaled by scale[index[m]]
  const float* scale = nullptr;
  const int32_t* index = nullptr;

  __device__ __forceinline__ float row_scale(int m) const {
    if (EPI != EPI_SWIGLU_BWD && EPI != EPI_GELU_BWD) return 1.f;
    return scale ? scale[index[min(m, rows - 1)]] : 1.f;
  }
  __device__ __forceinline__ static void pack(void* p, const float (&v)[4]) {
    if constexpr (OES == 2) *reinterpret_cast<uint2*>(p) = make_uint2(f32x2_to_bf16x2(v[0], v[1]), f32x2_to_bf16x2(v[2], v[3]));
    else *reinterpret_cast<float4*>(p) = make_float4(v[0], v[1], v[2], v[3]);
  }
  __device__ __forceinline__ static void unpack(const void* p, float (&v)[4]) {
    if constexpr (OES == 2) {
      const uint2 t = *reinterpret_cast<const uint2*>(p);
      v[0] = __uint_as_float(t.x << 16); v[1] = __uint_as_float(t.x & 0xffff0000u);
      v[2] = __uint_as_float(t.y << 16); v[3] = __uint_as_float(t.y & 0xffff0000u);
    } else {
      const float4 t = *reinterpret_cast<const float4*>(p);
      v[0] = t.x; v[1] = t.y; v[2] = t.z; v[3] = t.w;
    }
  }
  template <int NA>
  __device__ __forceinline__ void apply(const float (&v)[NB][4], const float (&a)[NA][4], float sc, float (&o)[NOUT][4]) const {
#pragma unroll
    for (int q = 0; q < 4; q++) {
      if constexpr (EPI == EPI_STORE) {
#pragma unroll
        for (int nb = 0; nb < NB; nb++) o[nb][q] = v[nb][q];
      } else if constexpr (EPI == EPI_STORE_F32) {  // fp32 output whatever the operand type (router logits)
        o[0][q] = v[0][q];
      } else if constexpr (EPI == EPI_ADD) {        // accumulate into the output
        o[0][q] = a[0][q] + v[0][q];
      } else if constexpr (EPI == EPI_GELU_FWD) {   // two-matrix expert: keep the pre-activation, store f of it
        o[0][q] = v[0][q];
        o[1][q] = gelu_f<T>(v[0][q]);
      } else if constexpr (EPI == EPI_GELU_BWD) {   // dZ = dH f'(Z)
        o[0][q] = sc * v[0][q] * gelu_grad_f<T>(a[0][q]);
      } else if constexpr (EPI == EPI_SWIGLU_FWD) {
        o[0][q] = v[0][q];
        o[1][q] = v[NB - 1][q];
        o[2][q] = v[0][q] * sigmoidf_<T>(v[0][q]) * v[NB - 1][q];
      } else {                                      // dU = dH g s,  dG = dH u (s + g s (1 - s)),  s = sigmoid(g)
        const float g = a[0][q], u = a[NA - 1][q];
        const float s = sigmoidf_<T>(g);
        const float dh = sc * v[0][q];
        const float t = g * s;
        o[1][q] = dh * t;
        o[0][q] = dh * u * fmaf(t, 1.f - s, s);
      }
    }
  }
};

// --------------------------------------------------------------------- row-tiled GEMM kernel
// CoreSet::tile<KIND> is the tile core of a tile kind; kinds differ in height only (same BN, BK), so
// one launch serves full tiles and the short tiles of ragged groups.
template <class Core, int NB, int EPI, bool B_KC>
__device__ __forceinline__ void row_gemm_tile(const RowGemm& p, const RowTile& t, int nt, char* smem) {
  typedef typename Core::T T;
  constexpr int BN = Core::BN, BK = Core::BK;
  const int rows = tile_rows(t);
  const int n0 = nt * BN;
  const int n_valid = min(BN, p.N - n0);
  const int a_row0 = p.a_rows_out ? t.row0_out : t.row0_in;
  const int nk = (p.K + BK - 1) / BK;
  // Where the tiles of this block start in each segment of the sum over K (segments: first all of
  // pair 0, then all of pair 1), and how many bytes of valid data follow the tile origins.
  constexpr int64_t es = sizeof(T);
  const int64_t b_tile = (int64_t)t.group * p.b_group + (B_KC ? (int64_t)n0 * p.ldb : (int64_t)n0);
  // gathered A: the operand pointer stays at the origin of the whole matrix and the row map names the rows
  const RowMap amap = {p.a_index, p.a_index ? p.a_index_div : 1, a_row0, rows};
  const int64_t a_tile = p.a_index ? 0 : (int64_t)a_row0 * p.lda;
  const int64_t a_end = ((int64_t)((p.a_index ? p.a_src_rows : rows) - 1) * p.lda + p.K) * es;
  const int64_t b_end = B_KC ? ((int64_t)(n_valid - 1) * p.ldb + p.K) * es : ((int64_t)(p.K - 1) * p.ldb + (p.N - n0)) * es;
  auto segf = [&](int sg) __attribute__((always_inline)) {
    SegSrc<T, NB> s;
    const int pair = sg >= p.n_segs ? 1 : 0;  // at most two pairs
    const int seg = sg - pair * p.n_segs;
    s.a = (const T*)p.A[pair] + a_tile + seg * p.a_seg;
    const int64_t boff = b_tile + seg * p.b_seg;
    s.b[0] = (const T*)p.B[pair] + boff;
    if (NB == 2) s.b[NB - 1] = (const T*)p.Bdual + boff;
    s.k_len = p.K;
    s.a_bytes = a_end;
    s.b_bytes = b_end;
    return s;
  };
  const int c_row0 = p.c_rows_out ? t.row0_out : t.row0_in;
  Epilogue<T, NB, EPI> epi;
  const int64_t c_off = ((int64_t)c_row0 * p.ldc + n0) * Epilogue<T, NB, EPI>::OES;
#pragma unroll
  for (int x = 0; x < epi.NOUT; x++) epi.out[x] = (char*)p.out[x] + c_off;
  if (EPI == EPI_ADD) epi.in[0] = epi.out[0];
  else if (epi.NAUX > 0) {
    epi.in[0] = (const char*)p.in[0] + c_off;
    if (epi.NAUX > 1) epi.in[epi.NAUX - 1] = (const char*)p.in[1] + c_off;
  }
  epi.ldc = p.ldc;
  epi.rows = rows;
  epi.n_valid = n_valid;
  epi.scale = p.c_scale;
  epi.index = p.a_index + a_row0;
  Core::run(smem, p.n_pairs * p.n_segs, nk, segf, p.lda, p.ldb, epi, amap);
}

template <class CoreSet, int NB, int EPI, bool B_KC>
__device__ __forceinline__ void row_gemm_block(const RowGemm& p, int block, char* smem) {
  typedef typename CoreSet::template tile<0> Core0;
  const int ntn = (p.N + Core0::BN - 1) / Core0::BN;
  // Blocks go to the XCDs round-robin (block b runs on XCD b % 8) and the 32 CUs of an XCD share
  // one L2, so the 32 blocks an XCD holds at a time should read as few different operand tiles as
  // possible.  Tiles are numbered band by band (a band: kBandRows consecutive row tiles), column
  // by column within a band, and each XCD takes runs of 32 consecutive tiles: 4 row tiles x 8
  // column tiles, 12 operand streams for 32 tiles.  What is left after the last whole round of 8 runs is
  // cut into 8 equal runs, so that no XCD is a run ahead of another (a training step with 4 shared experts on a
  // second stream, T = 4096, d = 2048: 2.40 -> 2.21 ms; launches of many rounds: the same).
  const int per_band = kBandRows * ntn;
  const int n_mt = p.tiles ? *p.n_tiles : (p.n_rows + (Core0::BM >> p.direct_kind) - 1) / (Core0::BM >> p.direct_kind);
  const int total = (n_mt + kBandRows - 1) / kBandRows * per_band;
  const int xcd = block & 7, j = block >> 3;
  const int whole = total >> 8, in_run = j & 31;
  int q = ((j >> 5) * 8 + xcd) * 32 + in_run;
  if ((j >> 5) >= whole) {
    const int run = (total - (whole << 8) + 7) >> 3;
    if ((j >> 5) > whole || in_run >= run) return;
    q = (whole << 8) + xcd * run + in_run;
    if (q >= total) return;
  }
  const int band = q / per_band, r = q - band * per_band;
  const int mt = band * kBandRows + r % kBandRows, nt = r / kBandRows;
  RowTile t;
  if (p.tiles) {
    if (mt >= *p.n_tiles) return;
    t = p.tiles[mt];
  } else {
    // direct tiling: tiles of one height (the caller may pick a shorter kind, so that a GEMM with few column
    // tiles still fills the chip)
    const int kind = p.direct_kind;
    const int bm = Core0::BM >> kind;
    t.group = 0;
    t.row0_in = mt * bm;
    if (t.row0_in >= p.n_rows) return;
    t.rows = min(bm, p.n_rows - t.row0_in) | (kind << 16);
    t.row0_out = t.row0_in;
  }
  MOE_TRACE_BEGIN();
  switch (tile_kind(t)) {  // uniform over the block
    case 0: row_gemm_tile<Core0, NB, EPI, B_KC>(p, t, nt, smem); break;
    case 1: row_gemm_tile<typename CoreSet::template tile<1>, NB, EPI, B_KC>(p, t, nt, smem); break;
    case 2: row_gemm_tile<typename CoreSet::template tile<2>, NB, EPI, B_KC>(p, t, nt, smem); break;
    default: row_gemm_tile<typename CoreSet::template tile<3>, NB, EPI, B_KC>(p, t, nt, smem); break;
  }
  MOE_TRACE_ROW_TILE(EPI | (NB << 4) | ((int)B_KC << 8), nt | (tile_kind(t) << 8) | (tile_rows(t) << 16));
}

// ------------------------------------------------------------------- weight-gradient kernel
// `block` counts the tiles of a group, then groups (by descending rows), then products
template <class Core, int NB>
__device__ __forceinline__ void w_gemm_block(const WGemm& p, int block, char* smem) {
  typedef typename Core::T T;
  constexpr int BM = Core::BM, BN = Core::BN, BK = Core::BK;
  const int ntn = (p.N + BN - 1) / BN;
  // a block computes n_reps consecutive column tiles of one row of tiles (n_reps > 1 only where a
  // tile is a single short K step: the block's set-up, its group record and the latency of its
  // first loads are then paid once for several tiles, and the stores of one tile overlap the loads
  // of the next)
  const int reps = p.n_reps > 1 ? p.n_reps : 1;
  const int ntb = (ntn + reps - 1) / reps;
  const int per_group = (p.M + BM - 1) / BM * ntb;
  const int item = block / per_group, tile = block - item * per_group;
  // single-product kernels serve the two products of a dual GEMM one after the other
  const int z = NB == 1 ? item / p.n_groups : 0;
  const int rank = item - z * p.n_groups, mt = tile / ntb, nt_first = (tile - mt * ntb) * reps;
  // {group, rows, first row, compact slot}; without records every group has n_rows rows and its own slot
  const int4 gi = p.ginfo ? p.ginfo[rank] : make_int4(rank, p.n_rows, 0, rank);
  // the record is the same for the whole block: keep it in scalar registers, and with it every
  // address computation of the K loop
  const int g = __builtin_amdgcn_readfirstlane(gi.x), K = __builtin_amdgcn_readfirstlane(gi.y),
            start = __builtin_amdgcn_readfirstlane(gi.z), slot = __builtin_amdgcn_readfirstlane(gi.w);
  if (K <= 0 || K < p.k_min || K > p.k_max) return;
  const int a_row0 = start + (p.a_per_group ? g * p.n_rows : 0);
  const int b_row0 = start + (p.b_per_group ? g * p.n_rows : 0);
  const int m0 = mt * BM;
  const int m_valid = min(BM, p.M - m0);
  for (int nt = nt_first; nt < min(nt_first + reps, ntn); nt++) {
  const int n0 = nt * BN;
  const int n_valid = min(BN, p.N - n0);
  if (nt > nt_first) __syncthreads();  // the previous tile's epilogue is done with LDS in every wave
  auto segf = [&](int) __attribute__((always_inline)) {  // one segment: the rows of the group
    SegSrc<T, NB> s;
    s.a = (const T*)p.A + (int64_t)a_row0 * p.lda + m0;
    s.b[0] = (const T*)p.B[z] + (int64_t)b_row0 * p.ldb + n0;
    if (NB == 2) s.b[NB - 1] = (const T*)p.B[1] + (int64_t)b_row0 * p.ldb + n0;
    s.k_len = K;
    const int64_t es = sizeof(T);
    s.a_bytes = ((int64_t)(K - 1) * p.lda + (p.M - m0)) * es;
    s.b_bytes = ((int64_t)(K - 1) * p.ldb + (p.N - n0)) * es;
    return s;
  };
  Epilogue<T, NB, EPI_STORE> epi;
#pragma unroll
  for (int x = 0; x < NB; x++) epi.out[x] = (T*)p.C[NB == 1 ? z : x] + (int64_t)slot * p.c_slot + (int64_t)m0 * p.N + n0;
  epi.ldc = p.N;
  epi.rows = m_valid;
  epi.n_valid = n_valid;
  MOE_TRACE_BEGIN();
  Core::run(smem, 1, (K + BK - 1) / BK, segf, p.lda, p.ldb, epi, RowMap{nullptr, 1, 0, 0});
  MOE_TRACE_W_TILE(0x1000 | NB | (BM << 4), g, min(K, 0xffff) << 16);
  }
}

// ---------------------------------------------------------------------------------- kernels
template <class CoreSet, int NB, int EPI, bool B_KC>
__global__ __launch_bounds__(CoreSet::template tile<0>::NT, CoreSet::template tile<0>::BLOCKS_PER_CU) void row_gemm_kernel(RowGemm p) {
  extern __shared__ __align__(16) char smem[];
  row_gemm_block<CoreSet, NB, EPI, B_KC>(p, blockIdx.x, smem);
}
template <class Core, int NB>
__global__ __launch_bounds__(Core::NT, Core::BLOCKS_PER_CU) void w_gemm_kernel(WGemm p) {
  extern __shared__ __align__(16) char smem[];
  w_gemm_block<Core, NB>(p, blockIdx.x, smem);
}
// An input gradient and a weight gradient that does not depend on it in one launch: the first `row_blocks` blocks
// are row tiles (the longer ones), the others weight-gradient tiles, which fill the compute units that the
// last row tiles leave idle.  (One launch per product against dH + dWd and dX + dWg + dWu, and one
// instead of two for the light groups: training steps of T = 2777, d = 2048, 60 experts, top-3: 1.87 -> 1.69 ms;
// T = 3001, d = 1000: 0.88 -> 0.76; T = 8192, d = 768 GELU: 1.08 -> 1.03; fp32 T = 2048, d = 1024: 2.32 -> 2.14.)
template <class CoreSet, int EPI, class WCore, int WNB>
__global__ __launch_bounds__(WCore::NT, CoreSet::template tile<0>::BLOCKS_PER_CU) void row_w_gemm_kernel(RowGemm p, WGemm w, int row_blocks) {
  extern __shared__ __align__(16) char smem[];
  if ((int)blockIdx.x < row_blocks) row_gemm_block<CoreSet, 1, EPI, true>(p, blockIdx.x, smem);
  else w_gemm_block<WCore, WNB>(w, (int)blockIdx.x - row_blocks, smem);
}
// The weight gradients of the groups with few rows: all matrices of an expert in one launch.
template <class Core>
__global__ __launch_bounds__(Core::NT, Core::BLOCKS_PER_CU) void w_light_kernel(WGemm a, WGemm b, int a_blocks) {
  extern __shared__ __align__(16) char smem[];
  if ((int)blockIdx.x < a_blocks) w_gemm_block<Core, 1>(a, blockIdx.x, smem);
  else w_gemm_block<Core, 1>(b, (int)blockIdx.x - a_blocks, smem);
}

// ------------------------------------------------------------------------------ host side
// Three families of tile cores: fp32 (MOE_F32), bf16 with d and d_ff multiples of 64, and bf16 with any
// multiples of 8.  The last differs in one point: the row GEMMs mask the K tail of their K-contiguous
// operands (a VALU instruction per tile load; the weight gradients have no such operands).  Before, such sizes
// ran on 128 x 128 tiles staged through registers: forward + backward of T = 3001, d = 1000, d_ff = 1368,
// 24 experts, top-3, one shared expert: 1.63 ms; on these cores 0.91 ms, with the same bits.
enum { PATH_F32 = 0, PATH_BF16_TAIL = 1, PATH_BF16 = 2 };
template <int PATH> struct Cores;
template <> struct Cores<PATH_F32> {
  static constexpr int BM = 64, BN = 128;
  // Bound by the fp32 matrix pipe (157 TFLOP/s).  An fp32 MFMA takes an eighth of the operand bytes per cycle of
  // a bf16 one, so even 64 x 128 tiles (dual GEMMs: 64 x 64 of each product) keep it fed from L2; small tiles
  // balance better and two blocks fit on a CU, one multiplying while the other stores.  Forward + backward of
  // T = 2048, d = 1024, 16 experts, top-2, d_ff = 2816: 4.85 ms with fp32 FMA tiles (44 TFLOP/s), 2.51 ms with
  // 128 x 128 MFMA tiles, 2.49 ms with 64 x 128 on the ring pipeline, 2.33 ms with two whole K steps in flight
  // (91 TFLOP/s; the ring requests B too late for an iteration of 32 MFMAs); d = 128, d_ff = 256, T = 256: 275 -> 121 us.
  template <int NB, bool A_KC, bool B_KC> using core = MfmaDmaCore<float, 128, 128 / NB, NB, A_KC, B_KC, 2, 2, 1, true>;
};
template <> struct Cores<PATH_BF16> {
  static constexpr int BM = 256, BN = 256;
  // one block of 4 wavefronts (one per SIMD, each with a 128 x 128 share: the fewest LDS reads and
  // scalar instructions per MFMA, which is what the K loop is short of) computes 256 x 256 outputs
  // (dual GEMMs: 256 x 128 of each product)
  template <int NB, bool A_KC, bool B_KC> using core = MfmaDmaCore<bf16_t, 256, 256 / NB, NB, A_KC, B_KC, 2, 2>;
  // weight gradients of groups with few rows: 128 x 128 outputs per product, one tile slot
  template <int NB> using core_light = MfmaDmaCore<bf16_t, 128, 128, NB, false, false, 2, 2, 0>;
};
template <> struct Cores<PATH_BF16_TAIL> : Cores<PATH_BF16> {};
constexpr int kLightGroupRows = 256;  // groups up to this many rows take the light dW kernel
constexpr int kLightReps = 2;         // column tiles per block of that kernel (1: +5 % time on the DeepSeek shape, 8: +3 %)

// The tile cores a row-tiled GEMM launch may use: tile kinds of heights BM, BM/2, BM/4, BM/8, so that ragged
// groups waste little MFMA work.
template <int PATH, int NB, bool B_KC> struct RowCores {
  // bf16: heights 256, 128, 64 and 32; the last two share the 64-row core (those tiles are bound by streaming the
  // weights, not by MFMA work).  Pipeline depth by height: the 128-row tile fits 3 slots per operand, the
  // 64-row one 4.
  template <int KIND>
  using tile = MfmaDmaCore<bf16_t, (KIND == 0 ? 256 : KIND == 1 ? 128 : 64), 256 / NB, NB, true, B_KC, 2, 2,
                           (KIND == 0 ? 1 : KIND == 1 ? 2 : 3), PATH == PATH_BF16_TAIL>;
};
template <int NB, bool B_KC> struct RowCores<PATH_F32, NB, B_KC> {
  // heights 64, 32, 16, 8
  template <int KIND>
  using tile = std::conditional_t<(KIND == 0 || NB == 2), MfmaDmaCore<float, 64, 128 / NB, NB, true, B_KC, 2, 2, 2, true>,
                                  MfmaDmaCore<float, 32, 128, NB == 2 ? 1 : NB, true, B_KC, 1, 4, 2, true>>;
};

static int pick_path(const moe_shape_t* s) {
  if (s->dtype == MOE_F32) return PATH_F32;
  return (s->d % 64 == 0 && s->d_ff % 64 == 0) ? PATH_BF16 : PATH_BF16_TAIL;
}

static inline int ceil_div(int a, int b) { return (a + b - 1) / b; }

// A kernel that wants more than 48 KB of dynamic LDS has to be told so once per device (the
// attribute belongs to the kernel's code object on that device); one instance per kernel.
struct LdsAttr {
  std::atomic<uint64_t> done{0};  // bit i: set on device i
  void ensure(const void* kern, int lds_bytes) {
    if (lds_bytes <= 48 * 1024) return;
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0) return;
    const uint64_t bit = 1ull << (dev & 63);
    if (dev < 64 && (done.load(std::memory_order_relaxed) & bit)) return;
    (void)hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, lds_bytes);
    if (dev < 64) done.fetch_or(bit, std::memory_order_relaxed);
  }
};

// upper bound of the row tiles the plan kernel may emit (at most two remainder tiles per group)
static int max_row_tiles(int n_groups, int n_rows, bool shared, int BM) {
  return shared ? n_groups * (n_rows / BM + 2) : n_rows / BM + 2 * n_groups;
}

// LDS of a launch: one block may run any of the tile kinds
template <class CoreSet> constexpr int row_lds_bytes() {
  constexpr int n0 = CoreSet::template tile<0>::LDS_BYTES;
  return std::max({n0, CoreSet::template tile<1>::LDS_BYTES, CoreSet::template tile<2>::LDS_BYTES, CoreSet::template tile<3>::LDS_BYTES});
}

// whole bands of kBandRows row tiles, handed out in runs of 32 tiles to 8 XCDs
template <class CoreSet> static unsigned row_blocks(const RowGemm& p, int max_tiles) {
  typedef typename CoreSet::template tile<0> Core;
  const int ntn = ceil_div(p.N, Core::BN);
  const int n_mt = p.tiles ? max_tiles : ceil_div(p.n_rows, Core::BM >> p.direct_kind);
  return (unsigned)ceil_div(ceil_div(n_mt, kBandRows) * kBandRows * ntn, 256) * 256u;
}
template <class Core> static unsigned w_blocks(const WGemm& p, int n_products = 1) {
  const int tiles = ceil_div(p.M, Core::BM) * ceil_div(ceil_div(p.N, Core::BN), p.n_reps > 1 ? p.n_reps : 1);
  return (unsigned)tiles * (unsigned)p.n_groups * (unsigned)n_products;
}

template <class CoreSet, int NB, int EPI, bool B_KC>
static void launch_row(const char* label, const RowGemm& p, int max_tiles, hipStream_t st) {
  const unsigned blocks = row_blocks<CoreSet>(p, max_tiles);
  if (blocks == 0) return;
  auto kern = row_gemm_kernel<CoreSet, NB, EPI, B_KC>;
  static LdsAttr attr;
  constexpr int kLds = row_lds_bytes<CoreSet>();
  attr.ensure((const void*)kern, kLds);
  ProfScope prof(label, st);
  hipLaunchKernelGGL(kern, dim3(blocks), dim3(CoreSet::template tile<0>::NT), kLds, st, p);
}

template <class Core, int NB>
static void launch_w(const char* label, const WGemm& p, hipStream_t st) {
  const unsigned blocks = w_blocks<Core>(p);
  if (blocks == 0) return;
  auto kern = w_gemm_kernel<Core, NB>;
  static LdsAttr attr;
  attr.ensure((const void*)kern, Core::LDS_BYTES);
  ProfScope prof(label, st);
  hipLaunchKernelGGL(kern, dim3(blocks), dim3(Core::NT), Core::LDS_BYTES, st, p);
}

template <class CoreSet, int EPI, class WCore, int WNB>
static void launch_row_w(const char* label, const RowGemm& p, int max_tiles, const WGemm& w, hipStream_t st) {
  const unsigned rb = row_blocks<CoreSet>(p, max_tiles), blocks = rb + w_blocks<WCore>(w);
  if (blocks == 0) return;
  auto kern = row_w_gemm_kernel<CoreSet, EPI, WCore, WNB>;
  static LdsAttr attr;
  constexpr int kLds = std::max(row_lds_bytes<CoreSet>(), WCore::LDS_BYTES);
  attr.ensure((const void*)kern, kLds);
  ProfScope prof(label, st);
  hipLaunchKernelGGL(kern, dim3(blocks), dim3(WCore::NT), kLds, st, p, w, (int)rb);
}

template <class Core>
static void launch_w_light(const char* label, const WGemm& a, const WGemm& b, int b_products, hipStream_t st) {
  const unsigned ab = w_blocks<Core>(a), blocks = ab + w_blocks<Core>(b, b_products);
  if (blocks == 0) return;
  auto kern = w_light_kernel<Core>;
  static LdsAttr attr;
  attr.ensure((const void*)kern, Core::LDS_BYTES);
  ProfScope prof(label, st);
  hipLaunchKernelGGL(kern, dim3(blocks), dim3(Core::NT), Core::LDS_BYTES, st, a, b, (int)ab);
}

struct FwdArgs {
  int d, F, n_groups, n_rows;
  const int32_t* offsets;
  const void *Xin, *Wg, *Wu, *Wd;
  void *G, *U, *H, *Yout;
  void* ws;
  // gathered input (moe_expert_fwd_gather): Xin is the token matrix [src_rows, d] and grouped row r reads
  // its row src_of[r] / src_div
  const int32_t* src_of = nullptr;
  int src_div = 1, src_rows = 0;
};

template <int PATH>
static void expert_fwd_impl(const FwdArgs& a, hipStream_t st) {
  const bool shared = a.offsets == nullptr;
  const int max_tiles = max_row_tiles(a.n_groups, a.n_rows, shared, Cores<PATH>::BM);
  Plan pl = carve_plan(a.ws, a.n_groups, max_tiles);
  {
    ProfScope prof("plan_kernel", st);
    hipLaunchKernelGGL(plan_kernel, dim3(1), dim3(1024), 0, st, a.offsets, a.n_groups, a.n_rows, Cores<PATH>::BM, pl,
                       (int32_t*)nullptr, (int32_t*)nullptr);
  }
  // F4: dual GEMM with the SwiGLU epilogue, or (two-matrix expert, Wu == NULL) one GEMM with the GELU epilogue
  RowGemm p = {};
  p.tiles = pl.tiles; p.n_tiles = pl.n_tiles; p.n_rows = a.n_rows;
  p.N = a.F; p.K = a.d; p.n_pairs = 1; p.n_segs = 1;
  p.A[0] = a.Xin; p.lda = a.d; p.a_seg = 0; p.a_rows_out = 0;
  p.a_index = a.src_of; p.a_index_div = a.src_div; p.a_src_rows = a.src_rows;
  p.B[0] = a.Wg; p.Bdual = a.Wu; p.ldb = a.F; p.b_group = (int64_t)a.d * a.F; p.b_seg = 0;
  p.out[0] = a.G; p.out[1] = a.Wu ? a.U : a.H; p.out[2] = a.H; p.ldc = a.F; p.c_rows_out = 1;
  if (a.Wu) launch_row<RowCores<PATH, 2, false>, 2, EPI_SWIGLU_FWD, false>("gemm_fwd_gate_up", p, max_tiles, st);
  else launch_row<RowCores<PATH, 1, false>, 1, EPI_GELU_FWD, false>("gemm_fwd_gate_up", p, max_tiles, st);
  // F5: Yout = H Wd (shared mode: summed over groups through K segments)
  RowGemm q = {};
  q.n_rows = a.n_rows; q.N = a.d; q.K = a.F; q.n_pairs = 1;
  q.A[0] = a.H; q.lda = a.F; q.a_rows_out = 1;
  q.B[0] = a.Wd; q.ldb = a.d;
  q.out[0] = a.Yout; q.ldc = a.d; q.c_rows_out = 0;
  if (shared) {
    q.tiles = nullptr; q.n_segs = a.n_groups; q.a_seg = (int64_t)a.n_rows * a.F; q.b_seg = (int64_t)a.F * a.d;
    q.b_group = 0;
  } else {
    q.tiles = pl.tiles; q.n_tiles = pl.n_tiles; q.n_segs = 1; q.b_group = (int64_t)a.F * a.d;
  }
  launch_row<RowCores<PATH, 1, false>, 1, EPI_STORE, false>("gemm_fwd_down", q, max_tiles, st);
}

struct BwdArgs {
  int d, F, n_groups, n_rows;
  const int32_t* offsets;
  const void *Xin, *Wg, *Wu, *Wd, *G, *U, *H, *dYin;
  void* dXin;
  int32_t *active_ids, *n_active;
  void *dWg, *dWu, *dWd;
  void* ws;
  size_t plan_sz;
  // gathered upstream gradient (moe_expert_bwd_gather): the product dH reads row src_of[r] / src_div of
  // dY [src_rows, d] and scales row r by row_w[src_of[r]]; the weight gradient of Wd still reads dYin
  const void* dY = nullptr;
  const int32_t* src_of = nullptr;
  const float* row_w = nullptr;
  int src_div = 1, src_rows = 0;
};

template <int PATH>
static void expert_bwd_impl(const BwdArgs& a, hipStream_t st) {
  typedef Cores<PATH> C;
  const bool shared = a.offsets == nullptr;
  const size_t es = PATH == PATH_F32 ? 4 : 2;
  const int max_tiles = max_row_tiles(a.n_groups, a.n_rows, shared, Cores<PATH>::BM);
  Plan pl = carve_plan(a.ws, a.n_groups, max_tiles);
  const size_t act_rows = (size_t)(shared ? a.n_groups : 1) * a.n_rows;
  char* dG = (char*)a.ws + a.plan_sz;
  char* dU = dG + align_up(act_rows * a.F * es, 256);
  {
    ProfScope prof("plan_kernel", st);
    hipLaunchKernelGGL(plan_kernel, dim3(1), dim3(1024), 0, st, a.offsets, a.n_groups, a.n_rows, Cores<PATH>::BM, pl,
                       a.active_ids, a.n_active);
  }
  // B2a: dH = dYin Wd^T, epilogue turns it into dG, dU
  RowGemm p = {};
  p.tiles = pl.tiles; p.n_tiles = pl.n_tiles; p.n_rows = a.n_rows;
  p.N = a.F; p.K = a.d; p.n_pairs = 1; p.n_segs = 1;
  p.A[0] = a.dYin; p.lda = a.d; p.a_rows_out = 0;
  if (a.src_of) {
    p.A[0] = a.dY; p.a_index = a.src_of; p.a_index_div = a.src_div; p.a_src_rows = a.src_rows; p.c_scale = a.row_w;
  }
  p.B[0] = a.Wd; p.ldb = a.d; p.b_group = (int64_t)a.F * a.d;
  p.in[0] = a.G; p.in[1] = a.U; p.out[0] = dG; p.out[1] = dU; p.ldc = a.F; p.c_rows_out = 1;
  const bool gated = a.Wu != nullptr;  // two-matrix expert otherwise: dG is dZ, no dU
  // B2b: dXin = dG Wg^T + dU Wu^T
  RowGemm q = {};
  q.n_rows = a.n_rows; q.N = a.d; q.K = a.F; q.n_pairs = gated ? 2 : 1;
  q.A[0] = dG; q.A[1] = dU; q.lda = a.F; q.a_rows_out = 1;
  q.B[0] = a.Wg; q.B[1] = a.Wu; q.ldb = a.F;
  q.out[0] = a.dXin; q.ldc = a.d; q.c_rows_out = 0;
  if (shared) {
    q.tiles = nullptr; q.n_segs = a.n_groups; q.a_seg = (int64_t)a.n_rows * a.F; q.b_seg = (int64_t)a.d * a.F;
    q.b_group = 0;
  } else {
    q.tiles = pl.tiles; q.n_tiles = pl.n_tiles; q.n_segs = 1; q.b_group = (int64_t)a.d * a.F;
  }
  // B3: weight gradients, compacted to active groups, largest group first
  WGemm w = {};
  w.ginfo = pl.ginfo; w.n_rows = a.n_rows; w.n_groups = a.n_groups;
  w.M = a.F; w.N = a.d;
  w.A = a.H; w.lda = a.F; w.a_per_group = shared;
  w.B[0] = a.dYin; w.ldb = a.d; w.b_per_group = 0;
  w.C[0] = a.dWd; w.c_slot = (int64_t)a.F * a.d;
  WGemm v = {};
  v.ginfo = pl.ginfo; v.n_rows = a.n_rows; v.n_groups = a.n_groups;
  v.M = a.d; v.N = a.F;
  v.A = a.Xin; v.lda = a.d; v.a_per_group = 0;
  v.B[0] = dG; v.B[1] = dU; v.ldb = a.F; v.b_per_group = shared;
  v.C[0] = a.dWg; v.C[1] = a.dWu; v.c_slot = (int64_t)a.d * a.F;
  w.k_min = v.k_min = 1;
  w.k_max = v.k_max = 0x7fffffff;
  WGemm wl_ = w, vl_ = v;  // groups with few rows
  bool light = false;
  if constexpr (PATH != PATH_F32) {
    // groups with few rows are bound by writing their gradient, not by MFMA work: they go to a
    // kernel that keeps several blocks per CU in flight
    if (!shared) {
      light = true;
      const int light_rows = MOE_KNOB("MOE_LIGHT_ROWS", kLightGroupRows);
      w.k_min = v.k_min = light_rows + 1;
      wl_.k_min = vl_.k_min = 1;
      wl_.k_max = vl_.k_max = light_rows;
      // column tiles per block: at most kLightReps, and the same for every block of a row of tiles (11
      // column tiles go 6 + 5, not 8 + 3: consecutive blocks run on different XCDs, and unequal blocks
      // would load the XCDs unequally)
      const int reps_max = MOE_KNOB("MOE_LIGHT_REPS", kLightReps);
      auto even_reps = [&](int n_cols) {
        const int ntn = ceil_div(n_cols, C::template core_light<1>::BN);
        return ceil_div(ntn, ceil_div(ntn, reps_max));
      };
      wl_.n_reps = even_reps(wl_.N);
      vl_.n_reps = even_reps(vl_.N);
    }
  }
  // dH with dWd (which needs nothing that dH produces), then dX with dWg and dWu
  typedef RowCores<PATH, 1, true> Rows;
  typedef typename C::template core<1, false, false> W1;
  typedef typename C::template core<2, false, false> W2;
  if (gated) {
    launch_row_w<Rows, EPI_SWIGLU_BWD, W1, 1>("gemm_bwd_dh_dwd", p, max_tiles, w, st);
    launch_row_w<Rows, EPI_STORE, W2, 2>("gemm_bwd_dx_dwgu", q, max_tiles, v, st);
  } else {
    launch_row_w<Rows, EPI_GELU_BWD, W1, 1>("gemm_bwd_dh_dwd", p, max_tiles, w, st);
    launch_row_w<Rows, EPI_STORE, W1, 1>("gemm_bwd_dx_dwgu", q, max_tiles, v, st);
  }
  if constexpr (PATH != PATH_F32) {
    if (light) launch_w_light<typename C::template core_light<1>>("gemm_bwd_dw_light", wl_, vl_, gated ? 2 : 1, st);
  }
}

static size_t plan_size_for(int n_groups, int n_rows, bool shared) {
  // sized for the smallest row tile of any path, so the query does not depend on the path taken
  const int bound = max_row_tiles(n_groups, n_rows, shared, 64);
  return align_up(plan_bytes(n_groups, bound + 1), 256);
}

static int check_expert_args(const moe_shape_t* s, int n_groups, int n_rows, const char* who) {
  int rc = check_shape(s, who);
  if (rc) return rc;
  if (n_groups < 1 || n_groups > MOE_MAX_EXPERTS || n_rows < 0 || (int64_t)n_groups * n_rows >= (int64_t)1 << 31) {
    set_error("%s: bad n_groups=%d n_rows=%d", who, n_groups, n_rows);
    return MOE_EINVAL;
  }
  return MOE_OK;
}

}  // namespace moe

extern "C" size_t moe_expert_fwd_workspace_bytes(const moe_shape_t* shape, int32_t n_groups, int32_t n_rows,
                                                 int32_t shared) {
  using namespace moe;
  if (!shape || n_groups < 1 || n_rows < 0) return 0;
  return plan_size_for(n_groups, n_rows, shared != 0);
}

// plan + dG + dU ([n_rows, d_ff] each; shared mode keeps them per group)
extern "C" size_t moe_expert_bwd_workspace_bytes(const moe_shape_t* shape, int32_t n_groups, int32_t n_rows,
                                                 int32_t shared) {
  using namespace moe;
  if (!shape || n_groups < 1 || n_rows < 0) return 0;
  const size_t rows = (size_t)(shared ? n_groups : 1) * (size_t)n_rows;
  return plan_size_for(n_groups, n_rows, shared != 0) +
         2 * align_up(rows * shape->d_ff * elem_size(shape->dtype), 256);
}

extern "C" int moe_expert_fwd(const moe_shape_t* shape, int32_t n_groups, const int32_t* offsets, int32_t n_rows,
                              const void* Xin, const void* Wg, const void* Wu, const void* Wd, void* G, void* U,
                              void* H, void* Yout, void* ws, size_t ws_bytes, void* stream) {
  using namespace moe;
  int rc = check_expert_args(shape, n_groups, n_rows, "moe_expert_fwd");
  if (rc) return rc;
  if (!Wg || !Wd || !ws || (n_rows > 0 && (!Xin || !G || (Wu && !U) || !H || !Yout))) {
    set_error("moe_expert_fwd: null pointer");
    return MOE_EINVAL;
  }
  const void* ptrs[] = {Xin, Wg, Wu, Wd, G, U, H, Yout, ws};
  for (const void* p : ptrs)
    if (!aligned16(p)) {
      set_error("moe_expert_fwd: every tensor must be 16-byte aligned");
      return MOE_EINVAL;
    }
  if (ws_bytes < moe_expert_fwd_workspace_bytes(shape, n_groups, n_rows, offsets == nullptr)) {
    set_error("moe_expert_fwd: workspace of %zu bytes, need %zu", ws_bytes,
              moe_expert_fwd_workspace_bytes(shape, n_groups, n_rows, offsets == nullptr));
    return MOE_EWS;
  }
  if (n_rows == 0) return MOE_OK;
  FwdArgs a = {shape->d, shape->d_ff, n_groups, n_rows, offsets, Xin, Wg, Wu, Wd, G, U, H, Yout, ws};
  switch (pick_path(shape)) {
    case PATH_F32: expert_fwd_impl<PATH_F32>(a, (hipStream_t)stream); break;
    case PATH_BF16_TAIL: expert_fwd_impl<PATH_BF16_TAIL>(a, (hipStream_t)stream); break;
    default: expert_fwd_impl<PATH_BF16>(a, (hipStream_t)stream); break;
  }
  return launch_status("moe_expert_fwd");
}

extern "C" int moe_expert_bwd(const moe_shape_t* shape, int32_t n_groups, const int32_t* offsets, int32_t n_rows,
                              const void* Xin, const void* Wg, const void* Wu, const void* Wd, const void* G,
                              const void* U, const void* H, const void* dYin, void* dXin, int32_t* active_ids,
                              int32_t* n_active, void* dWg_c, void* dWu_c, void* dWd_c, void* ws,
                              size_t ws_bytes, void* stream) {
  using namespace moe;
  int rc = check_expert_args(shape, n_groups, n_rows, "moe_expert_bwd");
  if (rc) return rc;
  if (!Wg || !Wd || !ws || !active_ids || !n_active || !dWg_c || (Wu && !dWu_c) || !dWd_c ||
      (n_rows > 0 && (!Xin || !G || (Wu && !U) || !H || !dYin || !dXin))) {
    set_error("moe_expert_bwd: null pointer");
    return MOE_EINVAL;
  }
  const void* ptrs[] = {Xin, Wg, Wu, Wd, G, U, H, dYin, dXin, dWg_c, dWu_c, dWd_c, ws};
  for (const void* p : ptrs)
    if (!aligned16(p)) {
      set_error("moe_expert_bwd: every tensor must be 16-byte aligned");
      return MOE_EINVAL;
    }
  const size_t need = moe_expert_bwd_workspace_bytes(shape, n_groups, n_rows, offsets == nullptr);
  if (ws_bytes < need) {
    set_error("moe_expert_bwd: workspace of %zu bytes, need %zu", ws_bytes, need);
    return MOE_EWS;
  }
  BwdArgs a = {shape->d, shape->d_ff, n_groups, n_rows, offsets, Xin, Wg, Wu, Wd, G, U, H, dYin, dXin,
               active_ids, n_active, dWg_c, dWu_c, dWd_c, ws, plan_size_for(n_groups, n_rows, offsets == nullptr)};
  switch (pick_path(shape)) {
    case PATH_F32: expert_bwd_impl<PATH_F32>(a, (hipStream_t)stream); break;
    case PATH_BF16_TAIL: expert_bwd_impl<PATH_BF16_TAIL>(a, (hipStream_t)stream); break;
    default: expert_bwd_impl<PATH_BF16>(a, (hipStream_t)stream); break;
  }
  return launch_status("moe_expert_bwd");
}

// The same two calls reading token rows in place (grouped mode only): see include/moe_hip.h.
extern "C" int moe_expert_fwd_gather(const moe_shape_t* shape, const int32_t* offsets, const int32_t* src_of,
                                     const void* X, const void* Wg, const void* Wu, const void* Wd, void* G, void* U,
                                     void* H, void* Yout, void* ws, size_t ws_bytes, void* stream) {
  using namespace moe;
  int rc = check_shape(shape, "moe_expert_fwd_gather");
  if (rc) return rc;
  const int n_groups = shape->E, n_rows = shape->T * shape->k;
  if (!offsets || !Wg || !Wd || !ws || (n_rows > 0 && (!src_of || !X || !G || (Wu && !U) || !H || !Yout))) {
    set_error("moe_expert_fwd_gather: null pointer");
    return MOE_EINVAL;
  }
  const void* ptrs[] = {X, Wg, Wu, Wd, G, U, H, Yout, ws};
  for (const void* p : ptrs)
    if (!aligned16(p)) {
      set_error("moe_expert_fwd_gather: every tensor must be 16-byte aligned");
      return MOE_EINVAL;
    }
  if ((int64_t)shape->T * shape->d * (int64_t)elem_size(shape->dtype) >= ((int64_t)1 << 32) - 4096) {
    set_error("moe_expert_fwd_gather: X must be smaller than 4 GiB (32-bit byte offsets); use moe_expert_fwd on a permuted copy");
    return MOE_EINVAL;
  }
  const size_t need = moe_expert_fwd_workspace_bytes(shape, n_groups, n_rows, 0);
  if (ws_bytes < need) {
    set_error("moe_expert_fwd_gather: workspace of %zu bytes, need %zu", ws_bytes, need);
    return MOE_EWS;
  }
  if (n_rows == 0) return MOE_OK;
  FwdArgs a = {shape->d, shape->d_ff, n_groups, n_rows, offsets, X, Wg, Wu, Wd, G, U, H, Yout, ws};
  a.src_of = src_of; a.src_div = shape->k; a.src_rows = shape->T;
  switch (pick_path(shape)) {
    case PATH_F32: expert_fwd_impl<PATH_F32>(a, (hipStream_t)stream); break;
    case PATH_BF16_TAIL: expert_fwd_impl<PATH_BF16_TAIL>(a, (hipStream_t)stream); break;
    default: expert_fwd_impl<PATH_BF16>(a, (hipStream_t)stream); break;
  }
  return launch_status("moe_expert_fwd_gather");
}

extern "C" int moe_expert_bwd_gather(const moe_shape_t* shape, const int32_t* offsets, const int32_t* src_of,
                                     const void* Xp, const void* Wg, const void* Wu, const void* Wd, const void* G,
                                     const void* U, const void* H, const void* dY, const float* topk_w, const void* dYp,
                                     void* dXp, int32_t* active_ids, int32_t* n_active, void* dWg_c, void* dWu_c,
                                     void* dWd_c, void* ws, size_t ws_bytes, void* stream) {
  using namespace moe;
  int rc = check_shape(shape, "moe_expert_bwd_gather");
  if (rc) return rc;
  const int n_groups = shape->E, n_rows = shape->T * shape->k;
  if (!offsets || !Wg || !Wd || !ws || !active_ids || !n_active || !dWg_c || (Wu && !dWu_c) || !dWd_c ||
      (n_rows > 0 && (!src_of || !Xp || !G || (Wu && !U) || !H || !dY || !topk_w || !dYp || !dXp))) {
    set_error("moe_expert_bwd_gather: null pointer");
    return MOE_EINVAL;
  }
  const void* ptrs[] = {Xp, Wg, Wu, Wd, G, U, H, dY, dYp, dXp, dWg_c, dWu_c, dWd_c, ws};
  for (const void* p : ptrs)
    if (!aligned16(p)) {
      set_error("moe_expert_bwd_gather: every tensor must be 16-byte aligned");
      return MOE_EINVAL;
    }
  if ((int64_t)shape->T * shape->d * (int64_t)elem_size(shape->dtype) >= ((int64_t)1 << 32) - 4096) {
    set_error("moe_expert_bwd_gather: dY must be smaller than 4 GiB (32-bit byte offsets); use moe_expert_bwd");
    return MOE_EINVAL;
  }
  const size_t need = moe_expert_bwd_workspace_bytes(shape, n_groups, n_rows, 0);
  if (ws_bytes < need) {
    set_error("moe_expert_bwd_gather: workspace of %zu bytes, need %zu", ws_bytes, need);
    return MOE_EWS;
  }
  BwdArgs a = {shape->d, shape->d_ff, n_groups, n_rows, offsets, Xp, Wg, Wu, Wd, G, U, H, dYp, dXp,
               active_ids, n_active, dWg_c, dWu_c, dWd_c, ws, plan_size_for(n_groups, n_rows, false)};
  a.dY = dY; a.src_of = src_of; a.row_w = topk_w; a.src_div = shape->k; a.src_rows = shape->T;
  switch (pick_path(shape)) {
    case PATH_F32: expert_bwd_impl<PATH_F32>(a, (hipStream_t)stream); break;
    case PATH_BF16_TAIL: expert_bwd_impl<PATH_BF16_TAIL>(a, (hipStream_t)stream); break;
    default: expert_bwd_impl<PATH_BF16>(a, (hipStream_t)stream); break;
  }
  return launch_status("moe_expert_bwd_gather");
}

// ------------------------------------------------------------------------------------ router
// The gating network read as one linear map: logits = X Wr, and its adjoint.  E is arbitrary, so
// the GEMMs run on copies padded to Ep = E rounded up to 64 columns (zeros), which live in the
// workspace; when E is already a multiple of 64 the caller's buffers are used directly.
namespace moe {

template <typename TI, typename TO>
__device__ __forceinline__ TO cvt_elem(TI v);
template <> __device__ __forceinline__ float cvt_elem<float, float>(float v) { return v; }
template <> __device__ __forceinline__ bf16_t cvt_elem<bf16_t, bf16_t>(bf16_t v) { return v; }
template <> __device__ __forceinline__ bf16_t cvt_elem<float, bf16_t>(float v) { return f32_to_bf16(v); }

// dst[r][c] = c < cols_in ? src[r][c] : 0 for c < cols_out (cols_out >= cols_in: pad; the other way: strip)
template <typename TI, typename TO>
__global__ __launch_bounds__(256) void recolumn_kernel(const TI* __restrict__ src, TO* __restrict__ dst, int64_t rows,
                                                       int cols_in, int cols_out) {
  const int64_t n = rows * cols_out;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
    const int64_t r = i / cols_out;
    const int c = (int)(i - r * cols_out);
    dst[i] = c < cols_in ? cvt_elem<TI, TO>(src[r * cols_in + c]) : cvt_elem<TI, TO>(TI(0));
  }
}
template <typename TI, typename TO>
static void recolumn(const char* label, const void* src, void* dst, int64_t rows, int cols_in, int cols_out, hipStream_t st) {
  const int64_t n = rows * cols_out;
  if (n == 0) return;
  ProfScope prof(label, st);
  hipLaunchKernelGGL((recolumn_kernel<TI, TO>), dim3((unsigned)std::min<int64_t>((n + 255) / 256, 4096)), dim3(256), 0, st,
                     (const TI*)src, (TO*)dst, rows, cols_in, cols_out);
}

static int router_path(const moe_shape_t* s) {
  if (s->dtype == MOE_F32) return PATH_F32;
  return s->d % 64 == 0 ? PATH_BF16 : PATH_BF16_TAIL;
}
static int padded_experts(const moe_shape_t* s) { return (s->E + 63) / 64 * 64; }

template <int PATH>
static void router_fwd_impl(const moe_shape_t* s, const void* X, const void* Wr, float* logits, char* ws, hipStream_t st) {
  typedef typename Cores<PATH>::template core<1, true, false>::T T;
  const int Ep = padded_experts(s);
  const bool padded = Ep != s->E;
  const void* B = Wr;
  float* out = logits;
  if (padded) {
    T* WrP = (T*)ws;
    out = (float*)(ws + align_up((size_t)s->d * Ep * sizeof(T), 256));
    recolumn<T, T>("router_pad", Wr, WrP, s->d, s->E, Ep, st);
    B = WrP;
  }
  RowGemm p = {};
  p.n_rows = s->T; p.direct_kind = 2;  // quarter-height tiles: E is small, so the rows have to fill the chip
  p.N = Ep; p.K = s->d; p.n_pairs = 1; p.n_segs = 1;
  p.A[0] = X; p.lda = s->d;
  p.B[0] = B; p.ldb = Ep;
  p.out[0] = out; p.ldc = Ep;
  launch_row<RowCores<PATH, 1, false>, 1, EPI_STORE_F32, false>("gemm_router_fwd", p, 0, st);
  if (padded) recolumn<float, float>("router_pad", out, logits, s->T, Ep, s->E, st);
}

template <int PATH>
static void router_bwd_impl(const moe_shape_t* s, const void* X, const void* Wr, const float* dlogits, void* dWr, void* dX,
                            bool accumulate, char* ws, hipStream_t st) {
  typedef typename Cores<PATH>::template core<1, true, false>::T T;
  typedef Cores<PATH> C;
  const int Ep = padded_experts(s);
  const bool padded = Ep != s->E;
  // workspace: dlogits in the operand type [T, Ep]; then, when padded, Wr [d, Ep] and dWr [d, Ep]
  T* dlP = (T*)ws;
  char* q0 = ws + align_up((size_t)s->T * Ep * sizeof(T), 256);
  T* WrP = (T*)q0;
  T* dWrP = (T*)(q0 + align_up((size_t)s->d * Ep * sizeof(T), 256));
  recolumn<float, T>("router_pad", dlogits, dlP, s->T, s->E, Ep, st);
  const void* B = Wr;
  void* dW = dWr;
  if (padded) {
    recolumn<T, T>("router_pad", Wr, WrP, s->d, s->E, Ep, st);
    B = WrP;
    dW = dWrP;
  }
  // dWr = X^T dlogits  (one group of T rows)
  WGemm w = {};
  w.ginfo = nullptr; w.n_rows = s->T; w.n_groups = 1;
  w.M = s->d; w.N = Ep;
  w.A = X; w.lda = s->d; w.a_per_group = 0;
  w.B[0] = dlP; w.ldb = Ep; w.b_per_group = 0;
  w.C[0] = dW; w.c_slot = (int64_t)s->d * Ep;
  w.k_min = 1; w.k_max = 0x7fffffff;
  launch_w<typename C::template core<1, false, false>, 1>("gemm_router_dw", w, st);
  if (padded) recolumn<T, T>("router_pad", dWrP, dWr, s->d, Ep, s->E, st);
  // dX (+)= dlogits Wr^T
  RowGemm p = {};
  p.n_rows = s->T; p.direct_kind = 0;
  p.N = s->d; p.K = Ep; p.n_pairs = 1; p.n_segs = 1;
  p.A[0] = dlP; p.lda = Ep;
  p.B[0] = B; p.ldb = Ep;
  p.out[0] = dX; p.ldc = s->d;
  if (accumulate) launch_row<RowCores<PATH, 1, true>, 1, EPI_ADD, true>("gemm_router_dx", p, 0, st);
  else launch_row<RowCores<PATH, 1, true>, 1, EPI_STORE, true>("gemm_router_dx", p, 0, st);
}

}  // namespace moe

extern "C" size_t moe_router_fwd_workspace_bytes(const moe_shape_t* shape) {
  using namespace moe;
  if (!shape || shape->E < 1 || shape->d < 1 || shape->T < 0) return 0;
  const int Ep = padded_experts(shape);
  if (Ep == shape->E) return 256;
  return align_up((size_t)shape->d * Ep * elem_size(shape->dtype), 256) + align_up((size_t)shape->T * Ep * 4, 256);
}

extern "C" size_t moe_router_bwd_workspace_bytes(const moe_shape_t* shape) {
  using namespace moe;
  if (!shape || shape->E < 1 || shape->d < 1 || shape->T < 0) return 0;
  const int Ep = padded_experts(shape);
  const size_t es = elem_size(shape->dtype);
  return align_up((size_t)shape->T * Ep * es, 256) + 2 * align_up((size_t)shape->d * Ep * es, 256);
}

extern "C" int moe_router_fwd(const moe_shape_t* shape, const void* X, const void* Wr, float* logits, void* ws,
                              size_t ws_bytes, void* stream) {
  using namespace moe;
  int rc = check_shape(shape, "moe_router_fwd");
  if (rc) return rc;
  if (shape->T == 0) return MOE_OK;
  if (!X || !Wr || !logits || !ws) {
    set_error("moe_router_fwd: null pointer");
    return MOE_EINVAL;
  }
  if (!aligned16(X) || !aligned16(Wr) || !aligned16(logits) || !aligned16(ws)) {
    set_error("moe_router_fwd: every tensor must be 16-byte aligned");
    return MOE_EINVAL;
  }
  if (ws_bytes < moe_router_fwd_workspace_bytes(shape)) {
    set_error("moe_router_fwd: workspace of %zu bytes, need %zu", ws_bytes, moe_router_fwd_workspace_bytes(shape));
    return MOE_EWS;
  }
  switch (router_path(shape)) {
    case PATH_F32: router_fwd_impl<PATH_F32>(shape, X, Wr, logits, (char*)ws, (hipStream_t)stream); break;
    case PATH_BF16_TAIL: router_fwd_impl<PATH_BF16_TAIL>(shape, X, Wr, logits, (char*)ws, (hipStream_t)stream); break;
    default: router_fwd_impl<PATH_BF16>(shape, X, Wr, logits, (char*)ws, (hipStream_t)stream); break;
  }
  return launch_status("moe_router_fwd");
}

extern "C" int moe_router_bwd(const moe_shape_t* shape, const void* X, const void* Wr, const float* dlogits, void* dWr,
                              void* dX, int32_t accumulate, void* ws, size_t ws_bytes, void* stream) {
  using namespace moe;
  int rc = check_shape(shape, "moe_router_bwd");
  if (rc) return rc;
  if (!Wr || !dWr || !ws || (shape->T > 0 && (!X || !dlogits || !dX))) {
    set_error("moe_router_bwd: null pointer");
    return MOE_EINVAL;
  }
  if (!aligned16(X) || !aligned16(Wr) || !aligned16(dlogits) || !aligned16(dWr) || !aligned16(dX) || !aligned16(ws)) {
    set_error("moe_router_bwd: every tensor must be 16-byte aligned");
    return MOE_EINVAL;
  }
  if (ws_bytes < moe_router_bwd_workspace_bytes(shape)) {
    set_error("moe_router_bwd: workspace of %zu bytes, need %zu", ws_bytes, moe_router_bwd_workspace_bytes(shape));
    return MOE_EWS;
  }
  if (shape->T == 0) {  // no tokens: the weight gradient is zero, there is no dX
    if (shape->dtype == MOE_F32) recolumn<float, float>("router_pad", nullptr, dWr, shape->d, 0, shape->E, (hipStream_t)stream);
    else recolumn<bf16_t, bf16_t>("router_pad", nullptr, dWr, shape->d, 0, shape->E, (hipStream_t)stream);
    return launch_status("moe_router_bwd");
  }
  switch (router_path(shape)) {
    case PATH_F32: router_bwd_impl<PATH_F32>(shape, X, Wr, dlogits, dWr, dX, accumulate != 0, (char*)ws, (hipStream_t)stream); break;
    case PATH_BF16_TAIL: router_bwd_impl<PATH_BF16_TAIL>(shape, X, Wr, dlogits, dWr, dX, accumulate != 0, (char*)ws, (hipStream_t)stream); break;
    default: router_bwd_impl<PATH_BF16>(shape, X, Wr, dlogits, dWr, dX, accumulate != 0, (char*)ws, (hipStream_t)stream); break;
  }
  return launch_status("moe_router_bwd");
}

MOE_TRACE_DEFINE_READER
