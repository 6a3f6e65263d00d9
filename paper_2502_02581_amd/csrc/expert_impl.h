// Kernels and host side of the expert and router GEMMs, instantiated once per family of tile cores
// (expert_f32.hip, expert_bf16.hip, expert_tail.hip, expert_small.hip: four translation units, so that they compile side by side).
#pragma once

#include <algorithm>
#include <atomic>
#include <cmath>
#include <iterator>

#include "gemm_cores.h"
#include "gemm_plan.h"
#include "split_core.h"

namespace moe {

// ------------------------------------------------------------------------------- epilogues
enum { EPI_STORE = 0, EPI_SWIGLU_FWD = 1, EPI_SWIGLU_BWD = 2, EPI_STORE_F32 = 3, EPI_ADD = 4, EPI_GELU_FWD = 5,
       EPI_GELU_BWD = 6, EPI_PART = 7 };

// gelu(z) = z Phi(z) and its derivative Phi(z) + z phi(z) (Phi, phi: standard normal distribution
// function and density); the activation of the two-matrix expert.
// fp32 path: the library's erf and exp.  bf16 path (the result is rounded to bf16 anyway): the
// rational-times-exponential approximation of erf (Abramowitz & Stegun 7.1.26, absolute error below
// 1.5e-7) on the hardware's base-2 exp and reciprocal, a quarter of the instructions:
//   1 - Phi(|z|) = e p(t) t,  e = exp(-z^2 / 2) = 2^-(y^2),  y = |z| sqrt(log2(e) / 2),  t = 1 / (1 + 0.3275911 |z| / sqrt(2)),
// its factor of a half and the change of base folded into the constants.  The epilogue is bound by the number of its instructions
// (T = 8192, d = 768, 64 experts of 3072: gate/up 178 -> 173 us, dH with dWd 308 -> 303 against constants and selections one by one).
__device__ __forceinline__ float upper_tail_(float z, float& e) {  // p(t) t; e as above
  const float y = fabsf(z) * 0.8493218f;
  const float t = __builtin_amdgcn_rcpf(fmaf(y, 0.2727374809f, 1.f));
  e = __builtin_amdgcn_exp2f(-y * y);
  return t * fmaf(t, fmaf(t, fmaf(t, fmaf(t, 0.5307027145f, -0.7265760135f), 0.7107068705f), -0.142248368f), 0.127414796f);
}
template <typename T> __device__ __forceinline__ float gelu_f(float z) {
  if constexpr (sizeof(T) == 4) return z * (0.5f * (1.f + erff(z * 0.70710678118654752f)));
  float e;
  const float h = upper_tail_(z, e) * e;
  return z * (z < 0.f ? h : 1.f - h);
}
template <typename T> __device__ __forceinline__ float gelu_grad_f(float z) {
  if constexpr (sizeof(T) == 4) {
    const float e = expf(-0.5f * z * z), cdf = 0.5f * (1.f + erff(z * 0.70710678118654752f));
    return cdf + z * 0.3989422804014327f * e;
  }
  float e;
  const float p = upper_tail_(z, e);
  const float w = e * fmaf(fabsf(z), -0.3989422804014327f, p);  // the derivative at -|z|; at |z| it is one minus that
  return z < 0.f ? w : 1.f - w;
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
                              : EPI == EPI_STORE || EPI == EPI_PART ? NB : 1;
  static constexpr int NAUX = EPI == EPI_SWIGLU_BWD ? 2 : (EPI == EPI_GELU_BWD || EPI == EPI_ADD) ? 1 : 0;
  static constexpr int OES = EPI == EPI_STORE_F32 || EPI == EPI_PART ? 4 : sizeof(T);
  // bf16 outputs carry the streaming hint: every one is read again only by a later kernel, after gigabytes of
  // other traffic (2-3 % on the row GEMMs of the Qwen- and stress-shaped workloads; all launches without it: +0.8 % on a training
  // step of T = 4096, d = 2048, the light weight gradients +2 to 3 %).  Not where rows are no whole cache lines: two tiles
  // write parts of the same line then, and the hint sends each part on to memory by itself (T = 3001, d = 1000, width 1368:
  // 603 us a training step with it, 584 without; the light weight gradients alone 588).
  __device__ __forceinline__ bool stream() const { return OES == 2 && ldc % 64 == 0; }
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
  typedef std::conditional_t<OES == 2, uint2, float4> packed_t;  // four values
  __device__ __forceinline__ static void unpack(const packed_t& t, float (&v)[4]) {
    if constexpr (OES == 2) {
      v[0] = __uint_as_float(t.x << 16); v[1] = __uint_as_float(t.x & 0xffff0000u);
      v[2] = __uint_as_float(t.y << 16); v[3] = __uint_as_float(t.y & 0xffff0000u);
    } else {
      v[0] = t.x; v[1] = t.y; v[2] = t.z; v[3] = t.w;
    }
  }
  template <int NA>
  __device__ __forceinline__ void apply(const float (&v)[NB][4], const float (&a)[NA][4], float sc, float (&o)[NOUT][4]) const {
#pragma unroll
    for (int q = 0; q < 4; q++) {
      if constexpr (EPI == EPI_STORE || EPI == EPI_PART) {  // EPI_PART: fp32 sums of a part of K (see reduce_kernel)
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
// one launch serves full tiles and the short tiles of ragged groups.  EPI_PART: part `part` of p.n_parts, which
// sums p.k_part values of K of every segment.
template <class Core, int NB, int EPI, bool B_KC>
__device__ __forceinline__ void row_gemm_tile(const RowGemm& p, const RowTile& t, int nt, int part, char* smem) {
  typedef typename Core::T T;
  constexpr int BN = Core::BN, BK = Core::BK;
  const int rows = tile_rows(t);
  const int n0 = nt * BN;
  const int n_valid = min(BN, p.N - n0);
  const int a_row0 = p.a_rows_out ? t.row0_out : t.row0_in;
  const int k0 = EPI == EPI_PART ? part * p.k_part : 0;
  const int K = EPI == EPI_PART ? min(p.k_part, p.K - k0) : p.K;
  const int nk = (K + BK - 1) / BK;
  // Where the tiles of this block start in each segment of the sum over K (segments: first all of
  // pair 0, then all of pair 1), and how many bytes of valid data follow the tile origins.
  constexpr int64_t es = sizeof(T);
  const int64_t b_tile = (int64_t)t.group * p.b_group + (B_KC ? (int64_t)n0 * p.ldb + k0 : (int64_t)k0 * p.ldb + n0);
  // gathered A: the operand pointer stays at the origin of the whole matrix and the row map names the rows
  const RowMap amap = {p.a_index, p.a_index ? p.a_index_div : 1, a_row0, rows};
  const int64_t a_tile = (p.a_index ? 0 : (int64_t)a_row0 * p.lda) + k0;
  const int64_t a_end = ((int64_t)((p.a_index ? p.a_src_rows : rows) - 1) * p.lda + K) * es;
  const int64_t b_end = B_KC ? ((int64_t)(n_valid - 1) * p.ldb + K) * es : ((int64_t)(K - 1) * p.ldb + (p.N - n0)) * es;
  auto segf = [&](int sg) __attribute__((always_inline)) {
    SegSrc<T, NB> s;
    const int pair = sg >= p.n_segs ? 1 : 0;  // at most two pairs
    const int seg = sg - pair * p.n_segs;
    s.a = (const T*)p.A[pair] + a_tile + seg * p.a_seg;
    const int64_t boff = b_tile + seg * p.b_seg;
    s.b[0] = (const T*)p.B[pair] + boff;
    if (NB == 2) s.b[NB - 1] = (const T*)p.Bdual + boff;
    s.k_len = K;
    s.a_bytes = a_end;
    s.b_bytes = b_end;
    return s;
  };
  const int c_row0 = p.c_rows_out ? t.row0_out : t.row0_in;
  Epilogue<T, NB, EPI> epi;
  const int64_t c_off = ((int64_t)c_row0 * p.ldc + n0) * Epilogue<T, NB, EPI>::OES;
#pragma unroll
  for (int x = 0; x < epi.NOUT; x++)
    epi.out[x] = (EPI == EPI_PART ? (char*)(p.part + (int64_t)(part * NB + x) * p.part_stride) : (char*)p.out[x]) + c_off;
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

// PLAN: the tiles are those of a device-built plan; otherwise the host knows the row counts: p.n_groups groups
// of p.n_rows rows, cut into tiles of one height, possibly in parts along K (block: part by part).
template <class CoreSet, int NB, int EPI, bool B_KC, bool PLAN>
__device__ __forceinline__ void row_gemm_block(const RowGemm& p, int block, char* smem) {
  typedef typename CoreSet::template tile<0> Core0;
  const int ntn = (p.N + Core0::BN - 1) / Core0::BN;
  // Blocks go to the XCDs round-robin (block b runs on XCD b % 8) and the 32 CUs of an XCD share
  // one L2, so the 32 blocks an XCD holds at a time should read as few different operand tiles as
  // possible.  Tiles are numbered band by band (a band: kBandRows consecutive row tiles), column
  // by column within a band, and dealt to the XCDs 256 at a time.  Launches of many such rounds deal runs
  // of 32 consecutive tiles: 4 row tiles x 8 column tiles, 12 operand streams for 32 tiles.  The tiles come longest first,
  // though, and XCD 0 always gets the first run: in launches of a few rounds, and in the last round, that costs more
  // than the streams save, so there the runs are of 8 tiles, and a round that is not full is dealt tile by tile.  (Runs of 32 and
  // eighths of the last round against this, training steps: T = 3001, d = 1000, one shared expert 603 -> 580 us; T = 8192,
  // d = 768 1029 -> 1004; T = 4096, d = 2048, four shared 2148 -> 2106; T = 2777 of those 1515 -> 1484.  Runs of 8 throughout cost
  // T = 8192, d = 4096, width 6400, 12 rounds and more, 0.8 %.)
  const int per_band = kBandRows * ntn;
  const int bm = Core0::BM >> p.direct_kind;
  const int per_group = PLAN ? 0 : (p.n_rows + bm - 1) / bm;
  const int n_mt = PLAN ? *p.n_tiles : p.n_groups * per_group;
  const int part = PLAN || p.n_parts == 1 ? 0 : block / p.part_blocks;
  if (!PLAN) block -= part * p.part_blocks;
  const int total = n_mt * ntn, rounds = total >> 8;
  const int xcd = block & 7, round = block >> 8, i = (block >> 3) & 31;
  int q = round << 8;
  if (round < rounds) q += rounds > kFineRounds && round < rounds - 1 ? (xcd << 5) + i : ((i >> 3) << 6) + (xcd << 3) + (i & 7);
  else q += (i << 3) + xcd;
  if (q >= total) return;
  // (the last band may have fewer rows)
  const int band = q / per_band, r = q - band * per_band;
  const int high = min(kBandRows, n_mt - band * kBandRows);
  const int mt = band * kBandRows + r % high, nt = r / high;
  RowTile t;
  if (PLAN) {
    t = p.tiles[mt];
  } else {
    t.group = mt / per_group;
    t.row0_in = (mt - t.group * per_group) * bm;
    t.rows = min(bm, p.n_rows - t.row0_in) | (p.direct_kind << 16);
    t.row0_out = t.group * p.n_rows + t.row0_in;
  }
  MOE_TRACE_BEGIN();
  auto tile = [&](auto epi) __attribute__((always_inline)) {
    constexpr int E = decltype(epi)::value;
    if constexpr (CoreSet::KINDS == 1) {  // (a plan may have taller tiles: see plan_cap)
      for (int r0 = 0; r0 < tile_rows(t); r0 += Core0::BM) {
        if (r0 > 0) __syncthreads();  // the epilogue before is done with LDS in every wave
        RowTile u = t;
        u.row0_in += r0; u.row0_out += r0; u.rows = min(Core0::BM, tile_rows(t) - r0);
        row_gemm_tile<Core0, NB, E, B_KC>(p, u, nt, part, smem);
      }
    } else switch (tile_kind(t)) {  // uniform over the block
      case 0: row_gemm_tile<Core0, NB, E, B_KC>(p, t, nt, part, smem); break;
      case 1: row_gemm_tile<typename CoreSet::template tile<1>, NB, E, B_KC>(p, t, nt, part, smem); break;
      case 2: row_gemm_tile<typename CoreSet::template tile<2>, NB, E, B_KC>(p, t, nt, part, smem); break;
      default: row_gemm_tile<typename CoreSet::template tile<3>, NB, E, B_KC>(p, t, nt, part, smem); break;
    }
  };
  if (!PLAN && p.n_parts > 1) tile(std::integral_constant<int, EPI_PART>());
  else tile(std::integral_constant<int, EPI>());
  MOE_TRACE_ROW_TILE(EPI | (NB << 4) | ((int)B_KC << 8), nt | (tile_kind(t) << 8) | (tile_rows(t) << 16));
}

// ------------------------------------------------------------------- weight-gradient kernel
// `block` counts the tiles of a group, then groups (by descending rows), then products; without a plan (groups of
// p.n_rows rows each) then parts of the rows
template <class Core, int NB, bool PLAN>
__device__ __forceinline__ void w_gemm_block(const WGemm& p, int block, char* smem) {
  typedef typename Core::T T;
  constexpr int BM = Core::BM, BN = Core::BN, BK = Core::BK;
  const int ntn = (p.N + BN - 1) / BN;
  // a block computes n_reps consecutive column tiles of one row of tiles (n_reps > 1 only where a
  // tile is a single short K step: the block's set-up, its group record and the latency of its
  // first loads are then paid once for several tiles, and the stores of one tile overlap the loads
  // of the next)
  const int reps = Core::REPEATS && p.n_reps > 1 ? p.n_reps : 1;
  const int ntb = (ntn + reps - 1) / reps;
  const int per_group = (p.M + BM - 1) / BM * ntb;
  if (!PLAN && p.active_ids && block == 0)  // what plan_kernel writes when there is a plan
    for (int i = threadIdx.x; i < p.n_groups; i += Core::NT) {
      p.active_ids[i] = i;
      if (i == 0) *p.n_active = p.n_groups;
    }
  const int part = PLAN ? 0 : block / (p.n_groups * per_group);
  if (!PLAN) {
    if (part >= p.n_parts) return;  // the launch is rounded up
    block -= part * (p.n_groups * per_group);
  }
  const int item = block / per_group, tile = block - item * per_group;
  // single-product kernels serve the two products of a dual GEMM one after the other
  const int z = NB == 1 ? item / p.n_groups : 0;
  const int rank = item - z * p.n_groups, mt = tile / ntb, nt_first = (tile - mt * ntb) * reps;
  // {group, rows, first row, compact slot}; without a plan every group has n_rows rows and its own slot
  const int k0 = part * p.k_part;
  const int4 gi = PLAN ? p.ginfo[rank] : make_int4(rank, p.n_parts == 1 ? p.n_rows : min(p.k_part, p.n_rows - k0), k0, rank);
  // the record is the same for the whole block: keep it in scalar registers, and with it every
  // address computation of the K loop
  const int g = __builtin_amdgcn_readfirstlane(gi.x), K = __builtin_amdgcn_readfirstlane(gi.y),
            start = __builtin_amdgcn_readfirstlane(gi.z), slot = __builtin_amdgcn_readfirstlane(gi.w);
  if (K <= 0 || K < p.k_min || K > p.k_max) return;
  const int a_row0 = start + (p.a_per_group ? g * p.n_rows : 0);
  const int b_row0 = start + (p.b_per_group ? g * p.n_rows : 0);
  const int m0 = mt * BM;
  const int m_valid = min(BM, p.M - m0);
  // (one trip where the core's tiles are long: what a loop would hoist has no registers there)
  for (int nt = nt_first; nt < (Core::REPEATS ? min(nt_first + reps, ntn) : nt_first + 1); nt++) {
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
  const int64_t c_off = (int64_t)slot * p.c_slot + (int64_t)m0 * p.N + n0;
  auto tile_of = [&](auto epi) __attribute__((always_inline)) {
    epi.ldc = p.N;
    epi.rows = m_valid;
    epi.n_valid = n_valid;
    Core::run(smem, 1, (K + BK - 1) / BK, segf, p.lda, p.ldb, epi, RowMap{nullptr, 1, 0, 0});
  };
  MOE_TRACE_BEGIN();
  if (!PLAN && p.n_parts > 1) {
    Epilogue<T, NB, EPI_PART> epi;
#pragma unroll
    for (int x = 0; x < NB; x++) epi.out[x] = p.part + (int64_t)(part * NB + x) * p.part_stride + c_off;
    tile_of(epi);
  } else {
    Epilogue<T, NB, EPI_STORE> epi;
#pragma unroll
    for (int x = 0; x < NB; x++) epi.out[x] = (T*)p.C[NB == 1 ? z : x] + c_off;
    tile_of(epi);
  }
  MOE_TRACE_W_TILE(0x1000 | NB | (BM << 4), g, min(K, 0xffff) << 16);
  }
}

// ---------------------------------------------------------------------------------- kernels
// A product over the rows of routed experts (PLAN), of shared ones or of the router (no plan).
template <class CoreSet, int NB, int EPI, bool B_KC, bool PLAN>
__global__ __launch_bounds__(CoreSet::template tile<0>::NT, CoreSet::template tile<0>::BLOCKS_PER_CU) void row_gemm_kernel(RowGemm p) {
  extern __shared__ __align__(16) char smem[];
  row_gemm_block<CoreSet, NB, EPI, B_KC, PLAN>(p, blockIdx.x, smem);
}
// The same product over the rows of shared experts, `s_blocks` blocks, and over those of the routed ones, in one launch.  The shared
// tiles are full and even, so
// they come first: the light tiles of the routed groups end the launch.  (In launches of their own the shared experts' few tiles leave
// compute units idle, and so do the last routed ones.  Before and now, whole passes: training, T = 3001, d = 1000, one shared
// 673 -> 603 us, T = 2777, d = 2048, four shared 1629 -> 1518; 16 tokens through 4 shared of width 1408 and 60 experts, d = 2048,
// forward, with the plan from the dispatch and the cheaper marshalling of the calls, 128 -> 114, by box from 139 -> 129 to 125 -> 110.
// Against the shared experts on a second stream: training, T = 4096, d = 2048, four shared 2188 -> 2162.)
template <class CoreSet, int NB, int EPI, bool B_KC>
__global__ __launch_bounds__(CoreSet::template tile<0>::NT, CoreSet::template tile<0>::BLOCKS_PER_CU) void both_row_gemm_kernel(RowGemm s, RowGemm r, int s_blocks) {
  extern __shared__ __align__(16) char smem[];
  const int b = (int)blockIdx.x - s_blocks;
  if (b < 0) row_gemm_block<CoreSet, NB, EPI, B_KC, false>(s, blockIdx.x, smem);
  else row_gemm_block<CoreSet, NB, EPI, B_KC, true>(r, b, smem);
}
// An input gradient and a weight gradient that does not depend on it in one launch: first the row tiles (the longer
// ones), then weight-gradient tiles, which fill the compute units that the last row tiles leave idle.
// (One launch per product against dH + dWd and dX + dWg + dWu, and one
// instead of two for the light groups: training steps of T = 2777, d = 2048, 60 experts, top-3: 1.87 -> 1.69 ms;
// T = 3001, d = 1000: 0.88 -> 0.76; T = 8192, d = 768 GELU: 1.08 -> 1.03; fp32 T = 2048, d = 1024: 2.32 -> 2.14.)
// Blocks in this order, all counts but the last multiples of 8: weight gradients of shared experts where their tiles
// are the longest, row tiles of shared experts, weight gradients of shared experts where their tiles are at least half as long as
// the routed experts' full row tiles (T = 4096, d = 2048, four shared experts: 2148 -> 2108 us a training step against the end), row
// tiles of routed experts, weight gradients of shared experts otherwise, of routed experts.
struct RowWOrder {
  int32_t first_sw, s_rows, mid_sw, r_rows, last_sw;
};
// of one set (of the router, without a plan): only the first of those places for weight gradients, and the end
template <class CoreSet, int EPI, class WCore, int WNB, bool PLAN>
__global__ __launch_bounds__(WCore::NT, CoreSet::template tile<0>::BLOCKS_PER_CU) void row_w_gemm_kernel(RowGemm p, WGemm w, int first_w, int rows) {
  extern __shared__ __align__(16) char smem[];
  const int b = blockIdx.x, row = b - (PLAN ? 0 : first_w);
  if (row >= 0 && row < rows) row_gemm_block<CoreSet, 1, EPI, true, PLAN>(p, row, smem);
  else w_gemm_block<WCore, WNB, PLAN>(w, row < 0 ? b : row - rows, smem);
}
template <class CoreSet, int EPI, class WCore, int WNB>
__global__ __launch_bounds__(WCore::NT, CoreSet::template tile<0>::BLOCKS_PER_CU) void both_row_w_gemm_kernel(RowGemm s, RowGemm r, WGemm sw, WGemm rw, RowWOrder o) {
  extern __shared__ __align__(16) char smem[];
  // positions from the start of each section on
  const int b = blockIdx.x, srow = b - o.first_sw, mid = srow - o.s_rows, rrow = mid - o.mid_sw, last = rrow - o.r_rows;
  if (srow < 0 || (mid >= 0 && rrow < 0) || (last >= 0 && last < o.last_sw)) w_gemm_block<WCore, WNB, false>(sw, srow < 0 ? b : rrow < 0 ? mid : last, smem);
  else if (mid < 0) row_gemm_block<CoreSet, 1, EPI, true, false>(s, srow, smem);
  else if (last < 0) row_gemm_block<CoreSet, 1, EPI, true, true>(r, rrow, smem);
  else w_gemm_block<WCore, WNB, true>(rw, last - o.last_sw, smem);
}
// The weight gradients of the groups with few rows: all matrices of an expert in one launch.
template <class Core>
__global__ __launch_bounds__(Core::NT, Core::BLOCKS_PER_CU) void w_light_kernel(WGemm a, WGemm b, int a_blocks) {
  extern __shared__ __align__(16) char smem[];
  if ((int)blockIdx.x < a_blocks) w_gemm_block<Core, 1, true>(a, blockIdx.x, smem);
  else w_gemm_block<Core, 1, true>(b, (int)blockIdx.x - a_blocks, smem);
}

// Sums the parts of a product in their order and applies the epilogue that its tiles left out: `n` values per
// output matrix, `part` holds [n_parts][NB][n].
struct Reduce {
  const float* part;
  int32_t n_parts;
  int64_t n;          // a multiple of 4
  void* out[3];
  const void* in[2];
};
template <typename T, int NB, int EPI>
__global__ __launch_bounds__(256) void reduce_kernel(Reduce p) {
  typedef Epilogue<T, NB, EPI> Epi;
  constexpr int NA = Epi::NAUX > 0 ? Epi::NAUX : 1;
  Epi epi;
  for (int64_t i = ((int64_t)blockIdx.x * 256 + threadIdx.x) * 4; i < p.n; i += (int64_t)gridDim.x * 1024) {
    float v[NB][4] = {}, a[NA][4], o[Epi::NOUT][4];
#pragma unroll 4
    for (int s = 0; s < p.n_parts; s++)
#pragma unroll
      for (int nb = 0; nb < NB; nb++) {
        const float4 t = *reinterpret_cast<const float4*>(p.part + (int64_t)(s * NB + nb) * p.n + i);
        v[nb][0] += t.x; v[nb][1] += t.y; v[nb][2] += t.z; v[nb][3] += t.w;
      }
#pragma unroll
    for (int x = 0; x < Epi::NAUX; x++) Epi::unpack(*reinterpret_cast<const typename Epi::packed_t*>((const char*)(EPI == EPI_ADD ? p.out[0] : p.in[x]) + i * Epi::OES), a[x]);
    epi.apply(v, a, 1.f, o);
#pragma unroll
    for (int x = 0; x < Epi::NOUT; x++) Epi::pack((char*)p.out[x] + i * Epi::OES, o[x]);
  }
}

// ------------------------------------------------------------------------------ host side
// Four families of tile cores: fp32 (MOE_F32), bf16 with d and d_ff multiples of 64, bf16 with any multiples of 8, and
// bf16 calls of few rows (small_tiles).  The third differs from the second in one point: the row GEMMs mask the K tail of their
// K-contiguous operands (a VALU instruction per tile load; the weight gradients have no such operands).  Before, such sizes
// ran on 128 x 128 tiles staged through registers: forward + backward of T = 3001, d = 1000, d_ff = 1368,
// 24 experts, top-3, one shared expert: 1.63 ms; on these cores 0.91 ms, with the same bits.
enum { PATH_F32 = 0, PATH_BF16_TAIL = 1, PATH_BF16 = 2, PATH_BF16_SMALL = 3 };
template <int PATH> struct Cores;
template <> struct Cores<PATH_F32> {
  // 128 x 128 outputs (dual GEMMs: 128 x 64 of each product), two blocks per CU, one multiplying while the other stores its planes
  // or its outputs
  static constexpr int BM = 128, BN = 128;  // (BM: see plan_tile_rows)
  template <int NB, bool A_KC, bool B_KC> using core = SplitCore<128, 128 / NB, NB, A_KC, B_KC, 2, 2>;
};
template <> struct Cores<PATH_BF16> {
  static constexpr int BM = 256, BN = 256;
  // one block of 4 wavefronts (one per SIMD, each with a 128 x 128 share: the fewest LDS reads and
  // scalar instructions per MFMA, which is what the K loop is short of) computes 256 x 256 outputs
  // (dual GEMMs: 256 x 128 of each product)
  template <int NB, bool A_KC, bool B_KC> using core = MfmaDmaCore<256, 256 / NB, NB, A_KC, B_KC, 2, 2>;
  // weight gradients of groups with few rows: 128 x 128 outputs per product, one tile slot
  template <int NB> using core_light = MfmaDmaCore<128, 128, NB, false, false, 2, 2, 0>;
};
template <> struct Cores<PATH_BF16_TAIL> : Cores<PATH_BF16> {};
// Calls of few rows and short products (small_tiles): 64 x 128 outputs (dual GEMMs: 64 x 64 of each product), weight gradients 128 x 128, two blocks
// per CU.  Takes any multiples of 8.
template <> struct Cores<PATH_BF16_SMALL> : Cores<PATH_BF16> {
  static constexpr int BM = kSmallTileRows, BN = 128;
  template <int NB, bool A_KC, bool B_KC> using core = MfmaDmaCore<128, 128 / NB, NB, A_KC, B_KC, 2, 2>;
};
// Groups up to this many rows, one K step, take the light dW kernel.  (256 and 64, training steps: T = 3001, d = 1000,
// 24 experts 603 and 589 us; T = 8192, d = 768, 64 experts 1029 and 1019; T = 16384, d = 2048, stress routing 3696 and 3676; T = 8192,
// d = 4096, 16 experts 7178 and 7149; the others within 0.3 %.)
constexpr int kLightGroupRows = 64;
constexpr int kLightReps = 2;         // column tiles per block of that kernel (1: +5 % time on the DeepSeek shape, 8: +3 %)

// The tile cores a row-tiled GEMM launch may use: tile kinds of heights BM, BM/2, BM/4, BM/8, so that ragged
// groups waste little MFMA work.
template <int PATH, int NB, bool B_KC> struct RowCores {
  static constexpr int KINDS = 4;
  // bf16: heights 256, 128, 64 and 32; the last two share the 64-row core (those tiles are bound by streaming the
  // weights, not by MFMA work).  Pipeline depth by height: the 128-row tile fits 3 slots per operand, the
  // 64-row one 4.
  template <int KIND>
  using tile = MfmaDmaCore<(KIND == 0 ? 256 : KIND == 1 ? 128 : 64), 256 / NB, NB, true, B_KC, 2, 2,
                           (KIND == 0 ? 1 : KIND == 1 ? 2 : 3), PATH == PATH_BF16_TAIL>;
};
template <int NB, bool B_KC> struct RowCores<PATH_BF16_SMALL, NB, B_KC> {
  static constexpr int KINDS = 1;
  template <int KIND> using tile = MfmaDmaCore<kSmallTileRows, 128 / NB, NB, true, B_KC, 2, 2, 2, true>;
};
template <int NB, bool B_KC, int TERMS> struct SplitRows {
  static constexpr int KINDS = 4;
  // heights 128, 64, 32 and 16; the last two share the 32-row core
  template <int KIND>
  using tile = std::conditional_t<KIND == 0, SplitCore<128, 128 / NB, NB, true, B_KC, 2, 2, TERMS>,
                                  std::conditional_t<KIND == 1, SplitCore<64, 128 / NB, NB, true, B_KC, 2, 2, TERMS>,
                                                     SplitCore<32, 128 / NB, NB, true, B_KC, 1, 4, TERMS>>>;
};
template <int NB, bool B_KC> struct RowCores<PATH_F32, NB, B_KC> : SplitRows<NB, B_KC, 6> {};
// The cores of the gradient of the router's input.  In fp32 with eight terms: the gradients of the logits may be zero outside the selected
// experts, of which there may be one, and a sum of one product gains nothing that would make up for the two products left out.  (T = 8192,
// d = 2048, 64 experts, backward 49.4 us with six terms, 50.9 with eight.)
template <int PATH> struct RouterDx { typedef RowCores<PATH, 1, true> Rows; };
template <> struct RouterDx<PATH_F32> { typedef SplitRows<1, true, 8> Rows; };

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

void launch_plan(const int32_t* offsets, int n_groups, int BM, const Plan& pl, int32_t* active_ids, int32_t* n_active, hipStream_t st);

// LDS of a launch: one block may run any of the tile kinds
template <class CoreSet> constexpr int row_lds_bytes() {
  constexpr int n0 = CoreSet::template tile<0>::LDS_BYTES;
  return std::max({n0, CoreSet::template tile<1>::LDS_BYTES, CoreSet::template tile<2>::LDS_BYTES, CoreSet::template tile<3>::LDS_BYTES});
}

// --------------------------------------------------------------------------------- long rows
// The tile cores address their operands and outputs by 32-bit byte offsets from a tile's first row.  A tile is up to
// 256 rows high, rows beyond its valid ones included (those offsets only have to lie outside the descriptor's byte count),
// so where 256 rows of a matrix reach 4 GiB an offset wraps around into the valid rows: fp32 d or d_ff from 4.2 million,
// bf16 from 8.4 million.  Those products run on the two kernels of expert_wide.hip: 64-bit addresses, a wavefront per four outputs, its
// lanes splitting K.  Nothing about them is fast; they read an operand once per output row or column.
inline bool wide_rows(int64_t ld, size_t es) { return 256 * ld * (int64_t)es > ((int64_t)1 << 32) - 4096; }
template <typename T, int NB, int EPI, bool B_KC>
void launch_wide_row(const char* label, const RowGemm& p, int bm, int max_tiles, hipStream_t st);
template <typename T>
void launch_wide_w(const char* label, const WGemm& p, int n_products, hipStream_t st);

// whole rounds of 256 tiles (see row_gemm_block)
static unsigned row_block_count(int n_tiles, int N, int bn) { return (unsigned)ceil_div(n_tiles * ceil_div(N, bn), 256) * 256u; }
template <class Core> static unsigned w_block_count(const WGemm& p, int n_products = 1) {
  const int tiles = ceil_div(p.M, Core::BM) * ceil_div(ceil_div(p.N, Core::BN), p.n_reps > 1 ? p.n_reps : 1);
  return (unsigned)tiles * (unsigned)p.n_groups * (unsigned)n_products;
}

// Products without a plan: the host knows how many tiles there are, and picks the tile height and the number of
// parts along K.  A layer's few shared experts and the router have few, long products: 16 tokens through 4 shared
// experts of width 1408 (d = 2048) gave the down product 8 blocks of 88 K steps, 112 us, in parts 21 + 5 us (the sums);
// gate/up 30 -> 19 + 5 us.  The router of d = 7168, E = 256, T = 8192: forward 83 -> 47 + 8 us; the weight
// gradient had 28 tiles of 128 steps, 145 us, and followed dX, 51 us: now in one launch 74 + 6 us.  Shared
// expert of T = 3001, d = 1000, d_ff = 712, backward: 65 + 67 -> 38 + 44 us (and 11 us of sums).
//
// The choice minimises an estimate, in microseconds: a K step of a tile, by height (`iter`), what a tile costs besides
// (`fixed`: first loads, epilogue), a launch with the sums of the parts at 5 TB/s.  Measured for comparison with 256 tiles, one
// per compute unit, 16 and 64 K steps, operands in cache (dual products in brackets): bf16 1.53, 0.83, 0.60 and 0.54 (1.45, 0.79,
// 0.51, 0.48) a step of 256, 128, 64 and 32 rows, and 12 to 7 (16 to 8) besides, launch included; the table's steps are within a fifth
// of that, those of the short tiles up to half above it.  The weight gradients' and those of the small tiles (PATH_BF16_SMALL) were not
// measured apart.  fp32 (SplitCore, operands from memory): 1.52, 0.89 and 0.67 a step of 32 values of K and 128, 64 and 32 rows, 9 to 5
// besides; the table holds 0.5 to 0.6 of that at any height, and only the heights' ratio matters where it is used.  Neither has a term for the rate
// at which weights arrive (decode's gate/up and down products over 16 rows: 9 and 10 us by the estimate, 19 and 21 by
// measure); hence the 8 % that a choice has to promise over one part of full tiles, 20 % for the small tiles.
struct TileCost {
  int bm, bn, bk;
  float iter[4], fixed[4];
  int slots = 256;  // blocks that run side by side at these costs
};
// fp32 has two tables.  A sum in parts is rounded less often, so the parts of fp32 products are those of the tiles that computed them on the
// fp32 matrix instructions (64 rows, 64 and 128 columns: 1.07 us a step of 64 rows, 0.61 of fewer, 1.02 of dual ones, measured as above), to
// which the results' errors are held (with parts chosen by the costs of SplitCore's tiles, fewer, and all products in one sum, shared results
// were up to 1.6 times as far off, T = 1, d = 320, width 896: 3.1e-7 -> 4.8e-7); the height is chosen by row_cost and w_cost, those of SplitCore.
template <int PATH, int NB> constexpr TileCost part_cost() {
  if (PATH == PATH_BF16_SMALL) return TileCost{64, 128 / NB, 64, {0.45f, 0.45f, 0.45f, 0.45f}, {4, 4, 4, 4}, 512};
  if (PATH == PATH_F32)
    return NB == 2 ? TileCost{64, 64, 32, {0.9f, 0.9f, 0.9f, 0.9f}, {3, 3, 3, 3}}
                   : TileCost{64, 128, 32, {0.9f, 0.5f, 0.5f, 0.5f}, {3, 2, 2, 2}};
  return TileCost{256, 256 / NB, 64, {1.45f, 0.85f, 0.7f, 0.7f}, {7, 5, 4, 4}};
}
template <int PATH, int NB> constexpr TileCost w_part_cost() {
  if (PATH == PATH_BF16_SMALL) return TileCost{128, 128 / NB, 64, {0.6f, 0, 0, 0}, {5, 0, 0, 0}, 512};
  if (PATH == PATH_F32) return TileCost{128, 128 / NB, 32, {1.8f, 0, 0, 0}, {5, 0, 0, 0}};
  return TileCost{256, 256 / NB, 64, {1.45f, 0, 0, 0}, {7, 0, 0, 0}};
}
template <int PATH, int NB> constexpr TileCost row_cost() {
  if (PATH == PATH_BF16_SMALL) return part_cost<PATH, NB>();
  if (PATH == PATH_F32)  // two blocks per CU share the matrix pipe: figures of one block that has it for itself
    return TileCost{128, 128 / NB, 32, {0.9f, 0.5f, 0.35f, 0.35f}, {5, 4, 3, 3}};
  return TileCost{256, 256 / NB, 64, {1.45f, 0.85f, 0.7f, 0.7f}, {7, 5, 4, 4}};
}
template <int PATH, int NB> constexpr TileCost w_cost() {
  if (PATH == PATH_BF16_SMALL) return w_part_cost<PATH, NB>();
  if (PATH == PATH_F32) return TileCost{128, 128 / NB, 32, {0.9f, 0, 0, 0}, {5, 0, 0, 0}};
  return TileCost{256, 256 / NB, 64, {1.45f, 0, 0, 0}, {7, 0, 0, 0}};
}
struct DirectShape {      // one product (or pair of products, `nb` = 2) without a plan
  TileCost cost, tiles;        // by which the parts are chosen, and then the height
  int groups, rows, N, K, nb;  // (weight gradient: rows is M)
  int sums;                    // segments times pairs: how often K values are summed
  int64_t out_elems;           // elements of an output matrix
  double routed_us;            // the launch's tiles of routed experts, summed (an estimate: their row counts are on the device)
};
struct DirectChoice {
  int kind = 0, n_parts = 1, k_part = 0;
  double block_us = 0, reduce_us = 0;
  int64_t blocks = 0;
  size_t part_bytes = 0;
};
static DirectChoice direct_option(const DirectShape& s, const TileCost& cost, int kind, int parts) {
  DirectChoice c;
  const int nk = ceil_div(s.K, cost.bk), per = ceil_div(nk, parts);
  c.kind = kind;
  c.n_parts = ceil_div(nk, per);
  c.k_part = per * cost.bk;
  c.blocks = (int64_t)s.groups * ceil_div(s.rows, cost.bm >> kind) * ceil_div(s.N, cost.bn) * c.n_parts;
  c.block_us = cost.fixed[kind] + s.sums * per * cost.iter[kind];
  if (c.n_parts > 1) {
    c.part_bytes = align_up((size_t)c.n_parts * s.nb * s.out_elems * 4, 256);
    c.reduce_us = (cost.slots > 256 ? 7 : 4) + 2e-6 / 5 * c.part_bytes;  // (short launches: the launch as well)
  }
  return c;
}
// r: row product or NULL, w: weight gradient of the same launch or NULL; `avail`: bytes for the parts
static void choose_direct(const DirectShape* r, const DirectShape* w, size_t avail, DirectChoice* rc, DirectChoice* wc) {
  static const int kParts[] = {1, 2, 3, 4, 5, 6, 8, 10, 12, 16};
  const double routed = r ? r->routed_us : 0;
  const int slots = r ? r->cost.slots : w->cost.slots;
  if (routed > 0) {
    // No more room than the same product takes alone, which is what the size queries ask for: a larger workspace must not
    // change the parts, and with them the results' last bits.
    DirectShape alone = *r;
    alone.routed_us = 0;
    choose_direct(&alone, w, avail, rc, wc);
    avail = rc->part_bytes + wc->part_bytes;
  }
  double best = 0;
  bool first = true;
  DirectChoice w_options[std::size(kParts)];
  for (size_t i = 0; w && i < std::size(kParts); i++) w_options[i] = direct_option(*w, w->cost, 0, kParts[i]);
  for (int kind = 0; kind < (r ? 4 : 1); kind++)
    for (int pr : kParts) {
      const DirectChoice a = r ? direct_option(*r, r->cost, kind, pr) : DirectChoice();
      if (pr > 1 && (!r || a.n_parts == 1 || a.part_bytes > avail)) continue;
      for (size_t i = 0; i < std::size(kParts); i++) {
        const DirectChoice& b = w_options[i];
        if (i > 0 && (!w || b.n_parts == 1 || a.part_bytes + b.part_bytes > avail)) continue;
        double us;
        if (!w && routed == 0) us = (double)((a.blocks + slots - 1) / slots) * a.block_us;
        else {
          const double longest = std::max(a.block_us, b.block_us);
          us = std::max(longest, (a.blocks * a.block_us + b.blocks * b.block_us + routed) / slots + 0.3 * longest);
        }
        us += a.reduce_us + b.reduce_us;
        if (first || us < best) {
          best = first ? us * (slots > 256 ? 0.8 : 0.92) : us;
          *rc = a;
          *wc = b;
        }
        first = false;
      }
    }
  // the same parts in the tiles that compute them
  if (r && r->tiles.bm != r->cost.bm) {
    const int parts = rc->n_parts;
    best = 0;
    for (int kind = 0; kind < 3; kind++) {
      const DirectChoice a = direct_option(*r, r->tiles, kind, parts);
      const double us = (double)((a.blocks + slots - 1) / slots) * a.block_us;
      if (kind == 0 || us < best) {
        best = us;
        *rc = a;
      }
    }
  }
  if (w) *wc = direct_option(*w, w->tiles, 0, wc->n_parts);
}

template <typename T, int NB, int EPI>
static void launch_reduce(const float* part, int n_parts, int64_t n, void* const* out, const void* const* in, hipStream_t st) {
  Reduce q = {};
  q.part = part;
  q.n_parts = n_parts;
  q.n = n;
  for (int x = 0; x < Epilogue<T, NB, EPI>::NOUT; x++) q.out[x] = out[x];
  for (int x = 0; x < Epilogue<T, NB, EPI>::NAUX && in; x++) q.in[x] = in[x];
  ProfScope prof("gemm_reduce", st);
  hipLaunchKernelGGL((reduce_kernel<T, NB, EPI>), dim3((unsigned)std::min<int64_t>((n / 4 + 255) / 256, 4096)), dim3(256), 0, st, q);
}

// The shared side of a launch: the product without a plan (filled but for the choice) and room for its parts.
struct Direct {
  RowGemm p;
  DirectShape shape;
  WGemm w;
  DirectShape w_shape;
  char* parts;
  size_t avail;
};
static void set_choice(RowGemm& p, const DirectShape& s, const DirectChoice& c, char* parts, int bm, int bn) {
  p.direct_kind = c.kind; p.n_parts = c.n_parts; p.k_part = c.k_part;
  p.part = (float*)parts; p.part_stride = s.out_elems;
  p.part_blocks = (int)row_block_count(s.groups * ceil_div(s.rows, bm >> c.kind), p.N, bn);
}

template <auto KERNEL, class... Args>
static void launch_gemm(const char* label, unsigned blocks, int threads, int lds_bytes, hipStream_t st, Args... args) {
  static LdsAttr attr;
  attr.ensure((const void*)KERNEL, lds_bytes);
  ProfScope prof(label, st);
  hipLaunchKernelGGL(KERNEL, dim3(blocks), dim3(threads), lds_bytes, st, args...);
}
// launches of the router, which never have routed rows beside them, by their epilogue or their cores
template <int EPI, class CoreSet> constexpr bool kRouterOnly = EPI == EPI_STORE_F32 || EPI == EPI_ADD || std::is_same_v<CoreSet, RouterDx<PATH_F32>::Rows>;

// One product over the shared rows (sd), the routed rows (r, at most r_tiles tiles), or both.
// Launches of one set have kernels of their own, with one argument block and without the other set's code: short ones are bound by how
// fast they start.  (A call of one set in the kernels of both and in these, us, forward / backward: routed, T = 300, d = 1024, 16
// experts 32.6 / 63.2 and 32.2 / 63.0; T = 1500, d = 384, 4 experts 37.8 / 62.3 and 37.4 / 61.8; T = 2048, d = 1024, 8 experts
// 54.0 / 86.0 and 52.8 / 86.0; shared, 300 rows, 2 of 1024 31.6 / 34.8 and 30.5 / 34.5; 16 rows, 4 of 1408, d = 2048 41.0 / 54.8 and
// 40.3 / 54.4.  The router, T = 300, d = 2048, 64 experts: the product 17.1 and 15.8.)
template <class CoreSet, int NB, int EPI, bool B_KC>
static void launch_row(const char* label, const Direct* sd, const RowGemm* r, int r_tiles, hipStream_t st) {
  typedef typename CoreSet::template tile<0> Core;
  if (sd && sd->p.wide)
    launch_wide_row<typename Core::T, NB, EPI, B_KC>(label, sd->p, Core::BM, sd->shape.groups * ceil_div(sd->shape.rows, Core::BM), st);
  if (r && r->wide) launch_wide_row<typename Core::T, NB, EPI, B_KC>(label, *r, Core::BM, r_tiles, st);
  if (sd && sd->p.wide) sd = nullptr;
  if (r && r->wide) r = nullptr;
  DirectChoice c, none;
  RowGemm p = {};
  if (sd) {
    choose_direct(&sd->shape, nullptr, sd->avail, &c, &none);
    p = sd->p;
    set_choice(p, sd->shape, c, sd->parts, Core::BM, Core::BN);
  }
  const unsigned sb = (unsigned)p.part_blocks * c.n_parts, rb = r ? row_block_count(r_tiles, r->N, Core::BN) : 0;
  if (sb + rb == 0) return;
  constexpr int kLds = row_lds_bytes<CoreSet>();
  if (rb == 0) {
    launch_gemm<row_gemm_kernel<CoreSet, NB, EPI, B_KC, false>>(label, sb, Core::NT, kLds, st, p);
  } else if constexpr (!kRouterOnly<EPI, CoreSet>) {
    if (sb == 0) launch_gemm<row_gemm_kernel<CoreSet, NB, EPI, B_KC, true>>(label, rb, Core::NT, kLds, st, *r);
    else launch_gemm<both_row_gemm_kernel<CoreSet, NB, EPI, B_KC>>(label, sb + rb, Core::NT, kLds, st, p, *r, (int)sb);
  }
  if (c.n_parts > 1) launch_reduce<typename Core::T, NB, EPI>(p.part, c.n_parts, sd->shape.out_elems, p.out, p.in, st);
}

// The same with a weight gradient that does not depend on the product.
template <class CoreSet, int EPI, class WCore, int WNB>
static void launch_row_w(const char* label, const Direct* sd, const RowGemm* r, int r_tiles, const WGemm* rw, hipStream_t st) {
  typedef typename CoreSet::template tile<0> Core;
  typedef typename Core::T T;
  if (sd && sd->p.wide) {
    launch_wide_row<T, 1, EPI, true>(label, sd->p, Core::BM, sd->shape.groups * ceil_div(sd->shape.rows, Core::BM), st);
    launch_wide_w<T>(label, sd->w, WNB, st);
    sd = nullptr;
  }
  if (r && r->wide) {
    launch_wide_row<T, 1, EPI, true>(label, *r, Core::BM, r_tiles, st);
    launch_wide_w<T>(label, *rw, WNB, st);
    r = nullptr;
  }
  DirectChoice rc, wc;
  RowGemm p = {};
  WGemm w = {};
  RowWOrder o = {};
  if (sd) {
    choose_direct(&sd->shape, &sd->w_shape, sd->avail, &rc, &wc);
    p = sd->p;
    set_choice(p, sd->shape, rc, sd->parts, Core::BM, Core::BN);
    w = sd->w;
    w.n_parts = wc.n_parts; w.k_part = wc.k_part;
    w.part = (float*)(sd->parts + rc.part_bytes); w.part_stride = sd->w_shape.out_elems;
    o.s_rows = p.part_blocks * rc.n_parts;
    const int wb = (int)((w_block_count<WCore>(w) * (unsigned)wc.n_parts + 7) / 8 * 8);
    const TileCost& c = sd->shape.tiles;
    const double routed_us = r ? c.fixed[0] + (double)r->n_pairs * r->n_segs * ceil_div(r->K, c.bk) * c.iter[0] : 0;
    (wc.block_us > rc.block_us ? o.first_sw : r && 2 * wc.block_us >= routed_us ? o.mid_sw : o.last_sw) = wb;
  }
  if (r) o.r_rows = (int)row_block_count(r_tiles, r->N, Core::BN);
  const unsigned blocks = (unsigned)(o.first_sw + o.s_rows + o.mid_sw + o.r_rows + o.last_sw) + (r ? w_block_count<WCore>(*rw) : 0);
  if (blocks == 0) return;
  constexpr int kLds = std::max(row_lds_bytes<CoreSet>(), WCore::LDS_BYTES);
  if (!r) {
    launch_gemm<row_w_gemm_kernel<CoreSet, EPI, WCore, WNB, false>>(label, blocks, WCore::NT, kLds, st, p, w, o.first_sw, o.s_rows);
  } else if constexpr (!kRouterOnly<EPI, CoreSet>) {
    if (!sd) launch_gemm<row_w_gemm_kernel<CoreSet, EPI, WCore, WNB, true>>(label, blocks, WCore::NT, kLds, st, *r, *rw, 0, o.r_rows);
    else launch_gemm<both_row_w_gemm_kernel<CoreSet, EPI, WCore, WNB>>(label, blocks, WCore::NT, kLds, st, p, *r, w, *rw, o);
  }
  if (rc.n_parts > 1) launch_reduce<T, 1, EPI>(p.part, rc.n_parts, sd->shape.out_elems, p.out, p.in, st);
  if (wc.n_parts > 1) launch_reduce<T, WNB, EPI_STORE>(w.part, wc.n_parts, sd->w_shape.out_elems, w.C, nullptr, st);
}

template <class Core>
static void launch_w_light(const char* label, const WGemm& a, const WGemm& b, int b_products, hipStream_t st) {
  const unsigned ab = w_block_count<Core>(a), blocks = ab + w_block_count<Core>(b, b_products);
  if (blocks == 0) return;
  auto kern = w_light_kernel<Core>;
  static LdsAttr attr;
  attr.ensure((const void*)kern, Core::LDS_BYTES);
  ProfScope prof(label, st);
  hipLaunchKernelGGL(kern, dim3(blocks), dim3(Core::NT), Core::LDS_BYTES, st, a, b, (int)ab);
}

// The products without a plan: of a shared call, then of the router.
template <int PATH, int NB>
static DirectShape row_shape(int groups, int rows, int N, int K, int sums = 1) {
  return {part_cost<PATH, NB>(), row_cost<PATH, NB>(), groups, rows, N, K, NB, sums, (int64_t)groups * rows * N, 0.};
}
template <int PATH, int NB>
static DirectShape w_shape(int groups, int M, int N, int rows) {
  return {w_part_cost<PATH, NB>(), w_cost<PATH, NB>(), groups, M, N, rows, NB, 1, (int64_t)groups * M * N, 0.};
}
// The routed experts' share of a launch, in microseconds of one compute unit: n_rows rows over groups of unknown sizes.
// It makes for fewer parts (prefill of 192 tokens, one shared expert, d = 7168: 1085 us a pass without it, 1035 with it; training, T = 3001,
// d = 1000: 580 and 543), and so for longer sums.  In bf16 the results' rounding hides that (errors against 64 bits the same to
// four digits over sizes of T = 16 to 3001, d = 128 to 7168); in fp32 shared results were up to 2.6 times as far off (T = 1743,
// d = 832, width 64: 3.1e-7 -> 8.1e-7), so fp32 products are in the same parts beside routed rows as alone.
template <int PATH> constexpr bool kPartsSeeRouted = PATH != PATH_F32;
template <int PATH, int NB> static double routed_row_us(int n_groups, int n_rows, int N, int K, int sums = 1) {
  constexpr TileCost c = row_cost<PATH, NB>();
  const double steps = (double)sums * ceil_div(K, c.bk);
  if (PATH == PATH_BF16_SMALL)  // rows that fall on the groups at random
    return ceil_div(N, c.bn) * ((double)(n_rows / c.bm) + n_groups * (1 - std::exp(-(double)n_rows / n_groups))) * (c.fixed[0] + steps * c.iter[0]);
  return ceil_div(N, c.bn) * ((double)(n_rows / c.bm) * (c.fixed[0] + steps * c.iter[0]) +
                              std::min(n_groups, n_rows) * (c.fixed[2] + steps * c.iter[2]));
}
template <int PATH, int NB> static double routed_w_us(int n_rows, int M, int N) {
  constexpr TileCost c = w_cost<PATH, NB>();
  return (double)ceil_div(M, c.bm) * ceil_div(N, c.bn) * ceil_div(n_rows, c.bk) * c.iter[0];
}
template <int PATH> struct Products {
  int d, F, groups, rows;
  template <int NB> DirectShape gate_up() const { return row_shape<PATH, NB>(groups, rows, F, d); }
  DirectShape down() const { return row_shape<PATH, 1>(1, rows, d, F, groups); }
  DirectShape dh() const { return row_shape<PATH, 1>(groups, rows, F, d); }
  DirectShape dwd() const { return w_shape<PATH, 1>(groups, F, d, rows); }
  template <int NB> DirectShape dx() const { return row_shape<PATH, 1>(1, rows, d, F, NB * groups); }
  template <int NB> DirectShape dwgu() const { return w_shape<PATH, NB>(groups, d, F, rows); }
};
static size_t part_bytes_of(const DirectShape& r, const DirectShape* w) {
  DirectChoice a, b;
  choose_direct(&r, w, SIZE_MAX, &a, &b);
  return a.part_bytes + b.part_bytes;
}
// bytes for parts that a shared call can use, whatever its activation
template <int PATH> size_t expert_part_bytes(int d, int F, int n_groups, int n_rows, bool bwd) {
  const Products<PATH> s = {d, F, n_groups, n_rows};
  if (n_rows == 0) return 0;
  if (!bwd) return std::max({part_bytes_of(s.template gate_up<1>(), nullptr), part_bytes_of(s.template gate_up<2>(), nullptr), part_bytes_of(s.down(), nullptr)});
  const DirectShape wd = s.dwd(), w1 = s.template dwgu<1>(), w2 = s.template dwgu<2>();
  return std::max({part_bytes_of(s.dh(), &wd), part_bytes_of(s.template dx<1>(), &w1), part_bytes_of(s.template dx<2>(), &w2)});
}

struct FwdArgs {
  int d, F, n_groups, n_rows;
  const int32_t* offsets;
  const void *Xin, *Wg, *Wu, *Wd;
  void *G, *U, *H, *Yout;
  char* ws;
  char* parts;  // behind the plan
  size_t part_avail;
  // gathered input (moe_expert_fwd_gather): Xin is the token matrix [src_rows, d] and grouped row r reads
  // its row src_of[r] / src_div
  const int32_t* src_of = nullptr;
  int src_div = 1, src_rows = 0;
  void* plan = nullptr;  // a plan that moe_route_dispatch_plan has built
};

// The forward pass of the routed experts (r), of the shared ones (s), or of both in common launches.
template <int PATH>
void expert_fwd_impl(const FwdArgs* r, const FwdArgs* s, hipStream_t st) {
  struct Gemms {
    RowGemm gate_up, down;
  };
  auto fill = [](const FwdArgs& a, const Plan& pl) {
    const bool shared = a.offsets == nullptr;
    // F4: dual GEMM with the SwiGLU epilogue, or (two-matrix expert, Wu == NULL) one GEMM with the GELU epilogue
    RowGemm p = {};
    p.tiles = pl.tiles; p.n_tiles = pl.n_tiles; p.n_rows = a.n_rows; p.n_groups = a.n_groups;
    p.N = a.F; p.K = a.d; p.n_pairs = 1; p.n_segs = 1;
    p.A[0] = a.Xin; p.lda = a.d; p.a_seg = 0; p.a_rows_out = 0;
    p.a_index = a.src_of; p.a_index_div = a.src_div; p.a_src_rows = a.src_rows;
    p.B[0] = a.Wg; p.Bdual = a.Wu; p.ldb = a.F; p.b_group = (int64_t)a.d * a.F; p.b_seg = 0;
    p.out[0] = a.G; p.out[1] = a.Wu ? a.U : a.H; p.out[2] = a.H; p.ldc = a.F; p.c_rows_out = 1;
    // F5: Yout = H Wd (shared mode: summed over groups through K segments)
    RowGemm q = {};
    q.tiles = pl.tiles; q.n_tiles = pl.n_tiles;
    q.n_rows = a.n_rows; q.n_groups = 1; q.N = a.d; q.K = a.F; q.n_pairs = 1;
    q.A[0] = a.H; q.lda = a.F; q.a_rows_out = 1;
    q.B[0] = a.Wd; q.ldb = a.d;
    q.out[0] = a.Yout; q.ldc = a.d; q.c_rows_out = 0;
    q.n_segs = shared ? a.n_groups : 1;
    if (shared) { q.a_seg = (int64_t)a.n_rows * a.F; q.b_seg = (int64_t)a.F * a.d; }
    else q.b_group = (int64_t)a.F * a.d;
    p.wide = q.wide = wide_rows(std::max(a.d, a.F), sizeof(typename Cores<PATH>::template core<1, true, false>::T));
    return Gemms{p, q};
  };
  const bool gated = (r ? r->Wu : s->Wu) != nullptr;  // (the same for both)
  Gemms rg;
  int max_tiles = 0;
  if (r) {
    constexpr int dtype = PATH == PATH_F32 ? MOE_F32 : MOE_BF16;
    const int bm = plan_tile_rows(dtype, r->n_groups, r->n_rows, r->d, r->F);
    max_tiles = max_row_tiles(dtype, r->n_groups, r->n_rows, r->d);
    const Plan pl = carve_plan(r->plan ? r->plan : r->ws, r->n_groups, plan_cap(r->n_groups, r->n_rows));
    if (!r->plan) launch_plan(r->offsets, r->n_groups, bm, pl, nullptr, nullptr, st);
    rg = fill(*r, pl);
  }
  Direct up = {}, down = {};
  if (s) {
    const Gemms sg = fill(*s, Plan{});
    const Products<PATH> ps = {s->d, s->F, s->n_groups, s->n_rows};
    up.p = sg.gate_up; up.shape = gated ? ps.template gate_up<2>() : ps.template gate_up<1>();
    down.p = sg.down; down.shape = ps.down();
    up.parts = down.parts = s->parts; up.avail = down.avail = s->part_avail;
    if (r && kPartsSeeRouted<PATH>) {
      up.shape.routed_us = gated ? routed_row_us<PATH, 2>(r->n_groups, r->n_rows, r->F, r->d) : routed_row_us<PATH, 1>(r->n_groups, r->n_rows, r->F, r->d);
      down.shape.routed_us = routed_row_us<PATH, 1>(r->n_groups, r->n_rows, r->d, r->F);
    }
  }
  const Direct *su = s ? &up : nullptr, *sd = s ? &down : nullptr;
  typedef RowCores<PATH, 1, false> Rows1;
  typedef RowCores<PATH, 2, false> Rows2;
  if (gated) launch_row<Rows2, 2, EPI_SWIGLU_FWD, false>("gemm_fwd_gate_up", su, r ? &rg.gate_up : nullptr, max_tiles, st);
  else launch_row<Rows1, 1, EPI_GELU_FWD, false>("gemm_fwd_gate_up", su, r ? &rg.gate_up : nullptr, max_tiles, st);
  launch_row<Rows1, 1, EPI_STORE, false>("gemm_fwd_down", sd, r ? &rg.down : nullptr, max_tiles, st);
}

struct BwdArgs {
  int d, F, n_groups, n_rows;
  const int32_t* offsets;
  const void *Xin, *Wg, *Wu, *Wd, *G, *U, *H, *dYin;
  void* dXin;
  int32_t *active_ids, *n_active;
  void *dWg, *dWu, *dWd;
  char* ws;
  char *dG, *dU, *parts;  // behind the plan
  size_t part_avail;
  // gathered upstream gradient (moe_expert_bwd_gather): the product dH reads row src_of[r] / src_div of
  // dY [src_rows, d] and scales row r by row_w[src_of[r]]; the weight gradient of Wd still reads dYin
  const void* dY = nullptr;
  const int32_t* src_of = nullptr;
  const float* row_w = nullptr;
  int src_div = 1, src_rows = 0;
  void* plan = nullptr;
};

// The backward pass of the routed experts (r), of the shared ones (s), or of both in common launches.  With both, either
// all row counts are positive or the calls come one by one.
template <int PATH>
void expert_bwd_impl(const BwdArgs* r, const BwdArgs* s, hipStream_t st) {
  typedef Cores<PATH> C;
  struct Gemms {
    RowGemm dh, dx;
    WGemm dwd, dwgu;
  };
  auto fill = [](const BwdArgs& a, const Plan& pl) {
    const bool shared = a.offsets == nullptr;
    // B2a: dH = dYin Wd^T, epilogue turns it into dG, dU
    RowGemm p = {};
    p.tiles = pl.tiles; p.n_tiles = pl.n_tiles; p.n_rows = a.n_rows; p.n_groups = a.n_groups;
    p.N = a.F; p.K = a.d; p.n_pairs = 1; p.n_segs = 1;
    p.A[0] = a.dYin; p.lda = a.d; p.a_rows_out = 0;
    if (a.src_of) {
      p.A[0] = a.dY; p.a_index = a.src_of; p.a_index_div = a.src_div; p.a_src_rows = a.src_rows; p.c_scale = a.row_w;
    }
    p.B[0] = a.Wd; p.ldb = a.d; p.b_group = (int64_t)a.F * a.d;
    p.in[0] = a.G; p.in[1] = a.U; p.out[0] = a.dG; p.out[1] = a.dU; p.ldc = a.F; p.c_rows_out = 1;
    // B2b: dXin = dG Wg^T + dU Wu^T (two-matrix expert: dG is dZ, there is no dU)
    RowGemm q = {};
    q.tiles = pl.tiles; q.n_tiles = pl.n_tiles;
    q.n_rows = a.n_rows; q.n_groups = 1; q.N = a.d; q.K = a.F; q.n_pairs = a.Wu ? 2 : 1;
    q.A[0] = a.dG; q.A[1] = a.dU; q.lda = a.F; q.a_rows_out = 1;
    q.B[0] = a.Wg; q.B[1] = a.Wu; q.ldb = a.F;
    q.out[0] = a.dXin; q.ldc = a.d; q.c_rows_out = 0;
    q.n_segs = shared ? a.n_groups : 1;
    if (shared) { q.a_seg = (int64_t)a.n_rows * a.F; q.b_seg = (int64_t)a.d * a.F; }
    else q.b_group = (int64_t)a.d * a.F;
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
    v.B[0] = a.dG; v.B[1] = a.dU; v.ldb = a.F; v.b_per_group = shared;
    v.C[0] = a.dWg; v.C[1] = a.dWu; v.c_slot = (int64_t)a.d * a.F;
    w.k_min = v.k_min = 1;
    w.k_max = v.k_max = 0x7fffffff;
    p.wide = q.wide = w.wide = v.wide = wide_rows(std::max(a.d, a.F), sizeof(typename C::template core<1, true, false>::T));
    return Gemms{p, q, w, v};
  };
  const bool gated = (r ? r->Wu : s->Wu) != nullptr;  // (the same for both)
  Gemms rg;
  int max_tiles = 0;
  if (r) {
    constexpr int dtype = PATH == PATH_F32 ? MOE_F32 : MOE_BF16;
    const int bm = plan_tile_rows(dtype, r->n_groups, r->n_rows, r->d, r->F);
    max_tiles = max_row_tiles(dtype, r->n_groups, r->n_rows, r->d);
    const Plan pl = carve_plan(r->plan ? r->plan : r->ws, r->n_groups, plan_cap(r->n_groups, r->n_rows));
    if (!r->plan) launch_plan(r->offsets, r->n_groups, bm, pl, r->active_ids, r->n_active, st);
    if (r->n_rows == 0) return;  // no group is active
    rg = fill(*r, pl);
  }
  if (s && s->n_rows == 0) {
    launch_plan(nullptr, s->n_groups, C::BM, carve_plan(s->ws, s->n_groups, plan_cap(s->n_groups, 0)), s->active_ids, s->n_active, st);
    return;
  }
  // groups with few rows are bound by writing their gradient, not by MFMA work: they go to a
  // kernel that keeps several blocks per CU in flight
  WGemm wl_ = rg.dwd, vl_ = rg.dwgu;
  bool light = false;
  if constexpr (PATH != PATH_F32) {
    if (r && !rg.dwd.wide) {
      light = true;
      const int light_rows = MOE_KNOB("MOE_LIGHT_ROWS", kLightGroupRows);
      rg.dwd.k_min = rg.dwgu.k_min = light_rows + 1;
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
  Direct dh = {}, dx = {};
  if (s) {
    const Gemms sg = fill(*s, Plan{});
    const Products<PATH> ps = {s->d, s->F, s->n_groups, s->n_rows};
    dh.p = sg.dh; dh.shape = ps.dh(); dh.w = sg.dwd; dh.w_shape = ps.dwd();
    dh.w.active_ids = s->active_ids;
    dh.w.n_active = s->n_active;
    dx.p = sg.dx; dx.shape = gated ? ps.template dx<2>() : ps.template dx<1>();
    dx.w = sg.dwgu; dx.w_shape = gated ? ps.template dwgu<2>() : ps.template dwgu<1>();
    dh.parts = dx.parts = s->parts; dh.avail = dx.avail = s->part_avail;
    if (r && kPartsSeeRouted<PATH>) {
      dh.shape.routed_us = routed_row_us<PATH, 1>(r->n_groups, r->n_rows, r->F, r->d) + routed_w_us<PATH, 1>(r->n_rows, r->F, r->d);
      dx.shape.routed_us = routed_row_us<PATH, 1>(r->n_groups, r->n_rows, r->d, r->F, gated ? 2 : 1) +
                           (gated ? routed_w_us<PATH, 2>(r->n_rows, r->d, r->F) : routed_w_us<PATH, 1>(r->n_rows, r->d, r->F));
    }
  }
  const Direct *sh = s ? &dh : nullptr, *sx = s ? &dx : nullptr;
  const RowGemm *rh = r ? &rg.dh : nullptr, *rx = r ? &rg.dx : nullptr;
  // dH with dWd (which needs nothing that dH produces), then dX with dWg and dWu
  typedef RowCores<PATH, 1, true> Rows;
  typedef typename C::template core<1, false, false> W1;
  typedef typename C::template core<2, false, false> W2;
  if (gated) {
    launch_row_w<Rows, EPI_SWIGLU_BWD, W1, 1>("gemm_bwd_dh_dwd", sh, rh, max_tiles, &rg.dwd, st);
    launch_row_w<Rows, EPI_STORE, W2, 2>("gemm_bwd_dx_dwgu", sx, rx, max_tiles, &rg.dwgu, st);
  } else {
    launch_row_w<Rows, EPI_GELU_BWD, W1, 1>("gemm_bwd_dh_dwd", sh, rh, max_tiles, &rg.dwd, st);
    launch_row_w<Rows, EPI_STORE, W1, 1>("gemm_bwd_dx_dwgu", sx, rx, max_tiles, &rg.dwgu, st);
  }
  if constexpr (PATH != PATH_F32) {
    if (light) launch_w_light<typename C::template core_light<1>>("gemm_bwd_dw_light", wl_, vl_, gated ? 2 : 1, st);
  }
}

// ------------------------------------------------------------------------------------ router
// The gating network read as one linear map: logits = X Wr, and its adjoint.  E is arbitrary, so
// the GEMMs run on copies padded to Ep = E rounded up to 64 columns (zeros), which live in the
// workspace; when E is already a multiple of 64 the caller's buffers are used directly.
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

static inline int padded_experts(const moe_shape_t* s) { return (s->E + 63) / 64 * 64; }

template <int PATH> DirectShape router_fwd_shape(const moe_shape_t* s) { return row_shape<PATH, 1>(1, s->T, padded_experts(s), s->d); }
template <int PATH> DirectShape router_dx_shape(const moe_shape_t* s) { return row_shape<PATH, 1>(1, s->T, s->d, padded_experts(s)); }
template <int PATH> DirectShape router_dw_shape(const moe_shape_t* s) { return w_shape<PATH, 1>(1, s->d, padded_experts(s), s->T); }
template <int PATH> size_t router_part_bytes(const moe_shape_t* s, bool bwd) {
  if (s->T == 0) return 0;
  const DirectShape w = router_dw_shape<PATH>(s);
  return bwd ? part_bytes_of(router_dx_shape<PATH>(s), &w) : part_bytes_of(router_fwd_shape<PATH>(s), nullptr);
}

template <int PATH>
void router_fwd_impl(const moe_shape_t* s, const void* X, const void* Wr, float* logits, char* ws, char* parts, size_t part_avail, hipStream_t st) {
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
  p.n_rows = s->T; p.n_groups = 1;
  p.N = Ep; p.K = s->d; p.n_pairs = 1; p.n_segs = 1;
  p.A[0] = X; p.lda = s->d;
  p.B[0] = B; p.ldb = Ep;
  p.out[0] = out; p.ldc = Ep;
  p.wide = wide_rows(std::max(s->d, Ep), sizeof(T));
  Direct all = {};
  all.p = p; all.shape = router_fwd_shape<PATH>(s); all.parts = parts; all.avail = part_avail;
  launch_row<RowCores<PATH, 1, false>, 1, EPI_STORE_F32, false>("gemm_router_fwd", &all, nullptr, 0, st);
  if (padded) recolumn<float, float>("router_pad", out, logits, s->T, Ep, s->E, st);
}

template <int PATH>
void router_bwd_impl(const moe_shape_t* s, const void* X, const void* Wr, const float* dlogits, void* dWr, void* dX,
                     bool accumulate, char* ws, char* parts, size_t part_avail, hipStream_t st) {
  typedef typename Cores<PATH>::template core<1, true, false>::T T;
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
  // dX (+)= dlogits Wr^T
  RowGemm p = {};
  p.n_rows = s->T; p.n_groups = 1;
  p.N = s->d; p.K = Ep; p.n_pairs = 1; p.n_segs = 1;
  p.A[0] = dlP; p.lda = Ep;
  p.B[0] = B; p.ldb = Ep;
  p.out[0] = dX; p.ldc = s->d;
  p.wide = w.wide = wide_rows(std::max(s->d, Ep), sizeof(T));
  typedef typename RouterDx<PATH>::Rows Rows;
  typedef typename Cores<PATH>::template core<1, false, false> W1;
  const Direct all = {p, router_dx_shape<PATH>(s), w, router_dw_shape<PATH>(s), parts, part_avail};
  if (accumulate) launch_row_w<Rows, EPI_ADD, W1, 1>("gemm_router_bwd", &all, nullptr, 0, nullptr, st);
  else launch_row_w<Rows, EPI_STORE, W1, 1>("gemm_router_bwd", &all, nullptr, 0, nullptr, st);
  if (padded) recolumn<T, T>("router_pad", dWrP, dWr, s->d, Ep, s->E, st);
}

}  // namespace moe
