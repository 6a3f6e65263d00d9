// Tile core of the fp32 products: fp32 operands on the bf16 matrix pipe.
//
// Every fp32 value is the exact sum of three bf16 values, a = a1 + a2 + a3 (each the rounding of what the ones before
// leave; the second is at most 2^-8, the third at most 2^-17 of the first).  Of the nine products of two such sums the six
// of at least 2^-18 are computed, exactly and added in fp32, by v_mfma_f32_16x16x32_bf16; the other three together are
// below the rounding of an fp32 product.  Six of those instructions take 96 cycles for 16 x 16 x 32 products, an fp32
// instruction (v_mfma_f32_16x16x4_f32) 256, and a sum over K is rounded 6 times per 32 values instead of 32 times, so
// the results are closer to the exact ones than those of the fp32 instructions.
//
// Infinities, NaNs and sums that overflow come out as NaN or infinity somewhere among the partial products.  A tile that ends with
// such a value in any lane is computed again with the fp32 instruction, which treats them as fp32 arithmetic does (EXACT below).
// Operands below 2^-102 in magnitude (2e-31) lose the last bits of their third part to bf16's range, whose end is that of fp32.
//
// Measured, training steps, before (v_mfma_f32_32x32x2_f32 on 64 x 128 tiles) and now: T = 2048, d = 1024, 16 experts, top-2, width 2816
// 1940 -> 1450 to 1480 us (108 -> 145 TFLOP/s of fp32 products; the matrix pipe is busy 45 % of the time, stores to LDS and their barriers
// and the splitting itself take the rest); T = 256, d = 128, 8 experts of width 256 92.4 -> 87.6.  Errors against 64 bits 0.72 to 0.92 of the
// former ones over 40 drawn layers (weight gradients of T = 2048, d = 1024: 9.8e-7 -> 8.3e-7).
// Also tried: A from memory to the registers of its wavefront, without LDS, B in two tiles of planes with one barrier a step: on 256 x 128 tiles,
// one block per CU, 1575 us (the compiler moves accumulators between the register files), on 128 x 128, two blocks, 1488 (the weight
// gradients run out of registers).
#pragma once

#include "gemm_cores.h"

namespace moe {

// Same interface as MfmaDmaCore.  One block of 4 wavefronts, two blocks per CU; K step 32.  Operand tiles go from memory to registers (16 bytes per
// lane, one K step ahead), are split there, once per block, and stored to LDS as three bf16 planes.
// LDS layouts of a plane:
//  K-contiguous operand: 1 KB per 16 rows, in the order in which a wave reads them as MFMA fragments: piece p (8 values of K, lane
//    group p) of row r at p * 256 + (r ^ 4p) * 16.  The eight values are K = 4p..4p+3 and 16+4p..16+4p+3 (any order of K serves as long as
//    both operands have it), so that the four lanes that load a row read 64 consecutive bytes.
//  row-contiguous operand: [32][COLS], rows 32 bytes longer than their values, so that the 32 lanes of a transposing read (8 rows of
//    K, 32 bytes each) use different banks; lane group p takes the same K values by two such reads.  (Padding, not a swizzle: the address of
//    every fragment is the same register plus a constant.)
template <int BM_, int BN_, int NB, bool A_KC, bool B_KC, int WM_, int WN_>
struct SplitCore {
  typedef float T;
  static constexpr int ES = 4;
  static constexpr int BM = BM_, BN = BN_, BK = 32, MT = 16;
  static constexpr int WM = WM_, WN = WN_, NW = WM * WN, NT = 64 * NW;
  static constexpr int TM = BM / WM / MT, TN = BN / WN / MT;
  static constexpr int PLANES = 3;
  template <int ROWS, bool KC> static constexpr int plane() { return BK * (ROWS * 2 + (KC ? 0 : 32)); }
  static constexpr int A_PLANE = plane<BM, A_KC>(), B_PLANE = plane<BN, B_KC>();  // bytes
  static constexpr int B0 = PLANES * A_PLANE;                          // B planes: product by product behind A's
  static constexpr int TILE_BYTES = PLANES * (A_PLANE + NB * B_PLANE);
  static constexpr int STAGE_ROWS = 16;  // of the epilogue, which stages up to three matrices of a dual product, two of a single one
  static constexpr int LDS_BYTES = std::max(TILE_BYTES, NW * (NB == 2 ? 3 : 2) * STAGE_ROWS * TN * MT * 4);
  static constexpr int BLOCKS_PER_CU = 2;
  static constexpr bool REPEATS = false;  // (see w_gemm_block)
  static constexpr uint32_t kNowhere = 0xffffff00u;
  static constexpr int kFew = 8;  // (of one product the split sum is 1.4 times as far off as the rounded product, of four 0.8 times)
  typedef __attribute__((ext_vector_type(8))) __bf16 frag_t;
  static_assert(NW == 4 && BM % (32 * WM) == 0 && BN % (16 * WN) == 0, "four wavefronts, whole blocks of 32 rows each");
  static_assert(A_KC || BM == 64 || BM == 128, "whole loads of row-contiguous tiles");
  static_assert(B_KC || BN == 64 || BN == 128, "whole loads of row-contiguous tiles");
  static_assert(LDS_BYTES <= 80 * 1024, "two blocks per CU");

  // 16-byte loads per thread and operand tile; a K-contiguous tile of 32 rows leaves half of the threads without one
  template <int ROWS, bool KC> static constexpr int loads() { return KC ? 2 * ((ROWS * 4 + NT - 1) / NT) : ROWS * BK / 4 / NT; }
  // three bf16 values each of x and y, in the halves of a register
  __device__ static __forceinline__ void split(float x, float y, uint32_t (&p)[PLANES]) {
    p[0] = f32x2_to_bf16x2(x, y);
    x -= __uint_as_float(p[0] << 16);
    y -= __uint_as_float(p[0] & 0xffff0000u);
    p[1] = f32x2_to_bf16x2(x, y);
    x -= __uint_as_float(p[1] << 16);
    y -= __uint_as_float(p[1] & 0xffff0000u);
    p[2] = f32x2_to_bf16x2(x, y);
  }

  // One operand tile: where its pieces come from and go to.
  template <int ROWS, bool KC>
  struct Loader {
    static constexpr int N = loads<ROWS, KC>();
    static constexpr int NO = KC ? N / 2 : 1;
    uint32_t off[NO], step;   // byte offsets of the loads from the tile's origin: two loads 64 bytes apart (KC), or `step` apart
    u32x4_t v[N];             // fp32 values
    uint32_t s[N][2][PLANES]; // and their parts, two values in a register
    // plain tiles
    __device__ __forceinline__ void start(uint32_t ld) {
      const int t = threadIdx.x;
      step = (uint32_t)(NT / (ROWS / 4)) * ld * 4;
#pragma unroll
      for (int i = 0; i < NO; i++) {
        const int q = t + i * NT;
        if (KC) off[i] = q < ROWS * 4 ? (uint32_t)(q >> 2) * ld * 4 + (q & 3) * 16 : kNowhere;
        else off[i] = (uint32_t)(q / (ROWS / 4)) * ld * 4 + (q % (ROWS / 4)) * 16;
      }
    }
    // rows that a map names
    __device__ __forceinline__ void gather(const RowMap& map, uint32_t ld) {
#pragma unroll
      for (int i = 0; i < NO; i++) {
        const int q = threadIdx.x + i * NT, row = q >> 2;
        off[i] = row < map.rows ? (uint32_t)map(row) * ld * 4 + (q & 3) * 16 : kNowhere;
      }
    }
    // descriptor of the tile; `left`: bytes from its origin to the end of the operand
    __device__ static __forceinline__ __amdgpu_buffer_rsrc_t desc(const char* base, int64_t left) {
      return make_rsrc(base, left <= 0 ? 0u : left > 0xffffffffll ? 0xffffffffu : (uint32_t)left);
    }
    // k_left: valid values of K from the tile's origin on (beyond them a row of a K-contiguous operand goes on with the next one)
    template <int j>
    __device__ __forceinline__ void load(__amdgpu_buffer_rsrc_t r, int k_left) {
      const int k = (threadIdx.x & 3) * 4 + (j & 1) * 16;
      const uint32_t at = KC ? off[KC ? j / 2 : 0] + (j & 1) * 64 : off[0] + j * step;  // (kNowhere and 64 more are nowhere)
      v[j] = __builtin_amdgcn_raw_buffer_load_b128(r, !KC || k < k_left ? at : kNowhere, 0, 0);
    }
    template <int j>
    __device__ __forceinline__ void split_one() {
#pragma unroll
      for (int i = 0; i < 2; i++) split(__uint_as_float(v[j][2 * i]), __uint_as_float(v[j][2 * i + 1]), s[j][i]);
    }
    // to LDS: three planes, `stride` bytes apart
    __device__ __forceinline__ void put(char* lds, int stride) const {
      const int t = threadIdx.x;
#pragma unroll
      for (int j = 0; j < N; j += KC ? 2 : 1) {
        if constexpr (KC) {
          const int q = t + (j >> 1) * NT, row = q >> 2, p = q & 3;
          if (ROWS * 4 < NT && q >= ROWS * 4) break;
          char* to = lds + (row >> 4) * 1024 + p * 256 + ((row & 15) ^ (4 * p)) * 16;
#pragma unroll
          for (int x = 0; x < PLANES; x++)
            *reinterpret_cast<u32x4_t*>(to + x * stride) = u32x4_t{s[j][0][x], s[j][1][x], s[j + 1][0][x], s[j + 1][1][x]};
        } else {
          const int q = t + j * NT, k = q / (ROWS / 4), c = q % (ROWS / 4);
          char* to = lds + k * (ROWS * 2 + 32) + c * 8;
#pragma unroll
          for (int x = 0; x < PLANES; x++) *reinterpret_cast<uint2*>(to + x * stride) = make_uint2(s[j][0][x], s[j][1][x]);
        }
      }
    }
    // the fp32 values themselves, [rows][32] or [32][rows]
    __device__ __forceinline__ void put_exact(char* lds) const {
#pragma unroll
      for (int j = 0; j < N; j++) {
        const int q = threadIdx.x + (KC ? j >> 1 : j) * NT;
        if (!KC) *reinterpret_cast<u32x4_t*>(lds + q * 16) = v[j];
        else if (q < ROWS * 4) *reinterpret_cast<u32x4_t*>(lds + (q >> 2) * 128 + (q & 3) * 16 + (j & 1) * 64) = v[j];
      }
    }
  };

  // fragment of 16 rows (columns) from `row0` on of a plane
  template <int ROWS, bool KC>
  __device__ static __forceinline__ frag_t frag(const char* plane, int row0, int lane) {
    if constexpr (KC) {
      const int p = lane >> 4, r = lane & 15;
      return __builtin_bit_cast(frag_t, *reinterpret_cast<const u32x4_t*>(plane + (row0 >> 4) * 1024 + p * 256 + (r ^ (4 * p)) * 16));
    } else {
      typedef __attribute__((address_space(3))) short4_t* lds_ptr;
      const int s = lane & 15, k = 4 * (lane >> 4) + (s >> 2), col = row0 + 4 * (s & 3);
      const char* at = plane + k * (ROWS * 2 + 32) + col * 2;
      const short4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)at);
      const short4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(at + 16 * (ROWS * 2 + 32)));
      const short8_t both = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
      return __builtin_bit_cast(frag_t, both);
    }
  }

  // All K steps of a tile.  While tile t is multiplied, the values of t + 1 are split in registers, in the shadow of the matrix
  // instructions, and each register that this frees is loaded with its part of t + 2.  LDS holds one tile: the barriers
  // around its stores stall one block while the other one of the CU multiplies.
  template <bool EXACT, class SegFn>
  __device__ static __forceinline__ void k_loop(char* smem, int n_segs, int nk, SegFn& segf, int64_t lda, int64_t ldb, const RowMap& amap,
                                                f32x4_t (&acc)[NB][TM][TN], int lane, int wm0, int wn0) {
#pragma unroll
    for (int nb = 0; nb < NB; nb++)
#pragma unroll
      for (int i = 0; i < TM; i++)
#pragma unroll
        for (int j = 0; j < TN; j++) acc[nb][i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    typedef Loader<BM, A_KC> LoadA;
    typedef Loader<BN, B_KC> LoadB;
    LoadA a;
    LoadB b[NB];
    if (A_KC && amap.gathered()) a.gather(amap, (uint32_t)lda);
    else a.start((uint32_t)lda);
#pragma unroll
    for (int nb = 0; nb < NB; nb++) b[nb].start((uint32_t)ldb);
    const int64_t a_step = A_KC ? BK * ES : (int64_t)BK * ES * lda, b_step = B_KC ? BK * ES : (int64_t)BK * ES * ldb;
    const int n_iters = n_segs * nk;
    if (n_iters == 0) return;
    // the tile to load next; beyond the last one the loads read nothing
    SegSrc<T, NB> g = segf(0);
    int sg = 0, ki = 0, k_left = 0;
    __amdgpu_buffer_rsrc_t ad, bd[NB];
    auto aim = [&]() __attribute__((always_inline)) {
      const bool some = sg < n_segs;
      ad = LoadA::desc((const char*)g.a + ki * a_step, some ? g.a_bytes - ki * a_step : 0);
#pragma unroll
      for (int nb = 0; nb < NB; nb++) bd[nb] = LoadB::desc((const char*)g.b[nb] + ki * b_step, some ? g.b_bytes - ki * b_step : 0);
      k_left = g.k_len - ki * BK;
      if (++ki == nk) {
        ki = 0;
        if (++sg < n_segs) g = segf(sg);
      }
    };
    constexpr int L = LoadA::N + NB * LoadB::N;
    auto load = [&](auto nc) __attribute__((always_inline)) {
      constexpr int n = decltype(nc)::value, m = n - LoadA::N;
      if constexpr (m < 0) a.template load<n>(ad, k_left);
      else b[m / LoadB::N].template load<m % LoadB::N>(bd[m / LoadB::N], k_left);
    };
    auto split_load = [&](auto nc) __attribute__((always_inline)) {
      constexpr int n = decltype(nc)::value, m = n - LoadA::N;
      if constexpr (m < 0) a.template split_one<n>();
      else b[m / LoadB::N].template split_one<m % LoadB::N>();
    };
    aim();
    static_for<L>(load);
    if constexpr (EXACT) {
      for (int it = 0; it < n_iters; it++) {
        __syncthreads();  // every wave is done with the tile before
        a.put_exact(smem);
#pragma unroll
        for (int nb = 0; nb < NB; nb++) b[nb].put_exact(smem + B0 + nb * PLANES * B_PLANE);
        aim();
        static_for<L>(load);
        __syncthreads();
        const float *la = (const float*)smem, *lb = (const float*)(smem + B0);
        const int r = lane & 15;
        for (int k = lane >> 4; k < BK; k += 4) {
          float fa[TM];
#pragma unroll
          for (int i = 0; i < TM; i++) fa[i] = A_KC ? la[(wm0 + i * MT + r) * BK + k] : la[k * BM + wm0 + i * MT + r];
#pragma unroll
          for (int nb = 0; nb < NB; nb++)
#pragma unroll
            for (int j = 0; j < TN; j++) {
              const float* p = lb + nb * (PLANES * B_PLANE / 4);
              const float fb = B_KC ? p[(wn0 + j * MT + r) * BK + k] : p[k * BN + wn0 + j * MT + r];
#pragma unroll
              for (int i = 0; i < TM; i++) acc[nb][i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(fb, fa[i], acc[nb][i][j], 0, 0, 0);
            }
        }
      }
    } else {
      static_for<L>(split_load);
      aim();
      static_for<L>(load);
      constexpr int G = NB * TN, M = 6 * TM;  // groups of MFMAs, by their B fragment
      for (int it = 0; it < n_iters; it++) {
        __syncthreads();  // every wave is done with the tile before
        a.put(smem, A_PLANE);
#pragma unroll
        for (int nb = 0; nb < NB; nb++) b[nb].put(smem + B0 + nb * PLANES * B_PLANE, B_PLANE);
        aim();
        __syncthreads();
        frag_t fa[TM][PLANES], fb[2 + PLANES - 1];  // of B: planes 1 and 2, and plane 0 of the even and of the odd groups
        auto read_b = [&](auto gc, int x) __attribute__((always_inline)) {
          constexpr int q = decltype(gc)::value, nb = q / TN, j = q % TN;
          fb[x > 0 ? 1 + x : q & 1] = frag<BN, B_KC>(smem + B0 + (nb * PLANES + x) * B_PLANE, wn0 + j * MT, lane);
        };
        static_for<PLANES>([&](auto x) __attribute__((always_inline)) {
          read_b(std::integral_constant<int, 0>(), PLANES - 1 - decltype(x)::value);
#pragma unroll
          for (int i = 0; i < TM; i++) fa[i][x] = frag<BM, A_KC>(smem + x * A_PLANE, wm0 + i * MT, lane);
        });
        static_for<G>([&](auto gc) __attribute__((always_inline)) {
          constexpr int q = decltype(gc)::value, nb = q / TN, j = q % TN;
          __builtin_amdgcn_sched_barrier(0);
          constexpr int n0 = q * L / G, n1 = (q + 1) * L / G;
          static_for<n1 - n0>([&](auto n) __attribute__((always_inline)) {
            split_load(std::integral_constant<int, n0 + decltype(n)::value>());
            load(std::integral_constant<int, n0 + decltype(n)::value>());
          });
          auto term = [&](int xb, int xa) __attribute__((always_inline)) {
#pragma unroll
            for (int i = 0; i < TM; i++)
              acc[nb][i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[xb > 0 ? 1 + xb : q & 1], fa[i][xa], acc[nb][i][j], 0, 0, 0);
          };
          // (in an order that lets the next group's fragments take the registers of this one's)
          auto next_b = [&](int x) __attribute__((always_inline)) {
            if constexpr (q + 1 < G) read_b(std::integral_constant<int, q + 1>(), x);
          };
          next_b(0);
          term(2, 0);
          next_b(2);
          term(1, 1);
          term(1, 0);
          next_b(1);
          term(0, 2);
          term(0, 1);
          term(0, 0);
          constexpr int kValu = ((n1 - n0) * 22 + M - 1) / M;  // per MFMA
          static_for<M>([&](auto) __attribute__((always_inline)) {
            __builtin_amdgcn_sched_group_barrier(0x8, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x2, kValu, 0);
          });
        });
      }
    }
  }

  template <class SegFn, class Epi>
  __device__ static __forceinline__ void run(char* smem, int n_segs, int nk, SegFn segf, int64_t lda, int64_t ldb, const Epi& epi,
                                             const RowMap& amap) {
    int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wm0 = (wave / WN) * (BM / WM), wn0 = (wave % WN) * (BN / WN);
    f32x4_t acc[NB][TM][TN];
    // (sums of a few products are rounded least often by the fp32 instruction)
    bool exact = n_segs * nk == 1 && segf(0).k_len <= kFew;
    if (!exact) {
      k_loop<false>(smem, n_segs, nk, segf, lda, ldb, amap, acc, lane, wm0, wn0);
      float bad = 0.f;  // NaN if any value is not finite
#pragma unroll
      for (int nb = 0; nb < NB; nb++)
#pragma unroll
        for (int i = 0; i < TM; i++)
#pragma unroll
          for (int j = 0; j < TN; j++)
#pragma unroll
            for (int r = 0; r < 4; r++) bad = fmaf(acc[nb][i][j][r], 0.f, bad);
      const bool any = __ballot(bad != 0.f) != 0;  // the same in every lane of the wave
      __syncthreads();  // every wave is done with the tiles
      int* found = (int*)smem;
      if (lane == 0) found[wave] = any;
      __syncthreads();
#pragma unroll
      for (int w = 0; w < NW; w++) exact = exact || found[w] != 0;
    }
    // (what comes now forms its addresses itself: shared with the loop above they would have to be kept all through it)
    asm volatile("" : "+v"(lane), "+s"(lda), "+s"(ldb));
    if (exact) k_loop<true>(smem, n_segs, nk, segf, lda, ldb, amap, acc, lane, wm0, wn0);
    __syncthreads();  // every wave is done with the tiles
    TileEpilogue<NB, TM, TN, NW, LDS_BYTES, false, STAGE_ROWS>::run(smem, acc, epi, wave, lane, wm0, wn0);
  }
};

}  // namespace moe
