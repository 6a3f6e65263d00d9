// Tile core of the fp32 products: fp32 operands on the bf16 matrix pipe.
//
// Every fp32 value is the exact sum of three bf16 values, a = a0 + a1 + a2 (each the rounding of what the ones before
// leave; the second is at most 2^-8, the third at most 2^-17 of the first).  Of the nine products of two such sums the six
// that can reach 2^-17 are computed by v_mfma_f32_32x32x16_bf16; of the other three two are at most 2^-25, half a unit in the last place of an
// fp32 product, and are computed where TERMS is 8 (see RouterDx).  Six of those instructions take 192 cycles for 32 x 32 x 16 products, the
// fp32 instruction (v_mfma_f32_32x32x2_f32) 512.
//
// The products a0 b0 have a sum of their own, `hi`, and the others, at most 2^-7 of them, have another, `lo`; the two are added at the
// end.  The instruction rounds its sum after every eight values of K (measured; the fp32 instruction after every value).  The
// roundings of `lo` do not count, those of `hi` are an eighth of the fp32 instruction's in dense sums, and in sums of few products
// most are exact: 16-bit products in a sum of 24 bits.  With all six in one sum, every product that is not zero costs six roundings of
// it.  Errors against 64 bits over those of the fp32 instruction, so and here, router of 64 to 4096 tokens, 8 to 256 experts: dense operands
// 0.49 to 0.84 and 0.31 to 0.61; gradients of the logits that are zero outside the top 1 to 8 experts 1.04 to 1.85 and 0.42 to 1.00; tokens of
// which 3 % are not zero 1.15 to 1.94 and 0.46 to 0.96; sums of one product 1.36 and 1.03.  (One value of K, kFew: the fp32 instruction.)
//
// Infinities, NaNs and sums that overflow come out as NaN or infinity somewhere among the partial products.  Operands below 2^-102 in
// magnitude (2e-31) lose the last bits of their third part to bf16's range, whose end is that of fp32: at most 2^-134 of a value, and all
// of one below 2^-134.  A tile that ends with a value that is not finite, or with one below 2^-76 that is not zero, in any lane
// is computed again with the fp32 instruction, which treats them as fp32 arithmetic does (EXACT below).  So what range loses of a result is
// 2^-134 / 2^-76 of the other operand: below 2^-25 of the result while that is below 2^33 -- except in results whose
// products all have a factor below 2^-134 (5e-41), which are zero.  (A training step of which every tile is computed again: 1500 -> 3240 us with tokens
// of 1e-28, 3790 with NaN.)
//
// Measured, training steps, with the fp32 instruction (on 64 x 128 tiles) and now: T = 2048, d = 1024, 16 experts, top-2, width 2816
// 1940 -> 1445 to 1500 us (144 TFLOP/s of fp32 products); T = 256, d = 128, 8 experts of width 256 92.4 -> 82.
// Also tried, the first of them: all eight products everywhere 1690 us; one sum, K steps of 32 in one tile of LDS with two barriers a step
// 1465; A from memory to the registers of its wavefront, without LDS, B in two tiles of planes with one barrier a step: on
// 256 x 128 tiles, one block per CU, 1575 us (the compiler moves accumulators between the register files), on 128 x 128, two blocks, 1488.
#pragma once

#include "gemm_cores.h"

namespace moe {

// Same interface as MfmaDmaCore.  One block of 4 wavefronts, two blocks per CU.  Operand tiles go from memory to registers (16 bytes per
// lane, two K steps ahead), are split there, once per block, and stored to LDS as three bf16 planes.
// LDS layouts of a plane, 16 values of K; no padding:
//  K-contiguous operand: 1 KB per 32 rows, in the order in which a wave reads them as MFMA fragments: the eight values of K of lane group
//    h of row r at h * 512 + (r ^ 8h) * 16 (the swizzle: a store of eight rows by 32 lanes uses all banks).
//  row-contiguous operand: [16][ROWS], the 64-byte pieces of a row swapped by k (rc_swizzle), so that the 32 lanes of a transposing read
//    (4 rows of K, one piece each) use all banks.
template <int BM_, int BN_, int NB, bool A_KC, bool B_KC, int WM_, int WN_, int TERMS = 6>
struct SplitCore {
  typedef float T;
  static constexpr int ES = 4;
  static constexpr int BM = BM_, BN = BN_, MT = 32;
  static constexpr int WM = WM_, WN = WN_, NW = WM * WN, NT = 64 * NW;
  // Wavefronts of 16 columns of each of two products: one accumulator tile holds both, 16 columns of the first, then 16 of the second.
  static constexpr bool MIX = NB == 2 && BN / WN == 16;
  static constexpr int MB = MIX ? 1 : NB;  // products in accumulator tiles
  static constexpr int TM = BM / WM / MT, TN = MIX ? 1 : BN / WN / MT;
  static constexpr int PLANES = 3;
  static constexpr int kFew = 1;  // values of K for which the fp32 instruction is no further off
  static_assert(TERMS == 6 || TERMS == 8, "without or with the products of the second and third parts");
  // 16 values of K, one MFMA, are a slice.  A K step is one slice of the tall tiles, and two of those with one row of accumulator tiles
  // a wave, whose step is bound by its barrier, its scalar work and LDS latency.  (One slice and two: forward products of T = 16, top-4,
  // d = 2048, 60 experts and four shared of 1408 114 and 76 us, 97 and 65; logits of T = 8192, d = 2048, 64 experts 74 and 62.)  LDS holds two steps.
  static constexpr int SLICES = TM == 1 ? 2 : 1, SK = 16, BK = SK * SLICES;
  static constexpr int A_PLANE = BM * SK * 2, B_PLANE = BN * SK * 2;  // bytes
  static constexpr int B0 = PLANES * A_PLANE;                          // B planes: product by product behind A's
  static constexpr int SLICE_BYTES = PLANES * (A_PLANE + NB * B_PLANE), TILE_BYTES = SLICES * SLICE_BYTES;
  static constexpr int STAGE_ROWS = MT;  // of the epilogue, which stages up to three matrices of a dual product, two of a single one
  static constexpr int LDS_BYTES = std::max(2 * TILE_BYTES, NW * (NB == 2 ? 3 : 2) * STAGE_ROWS * (BN / WN) * 4);
  static constexpr int BLOCKS_PER_CU = 2;
  static constexpr bool REPEATS = false;  // (see w_gemm_block)
  static constexpr uint32_t kNowhere = 0xffffff00u;
  static constexpr uint32_t kTiny = (127u - 76u) << 23;  // the bits of 2^-76
  typedef __attribute__((ext_vector_type(8))) __bf16 frag_t;
  typedef __attribute__((ext_vector_type(16))) float acc_t;  // 32 x 32: a lane has columns 8 * (r / 4) + 4 * (lane / 32) + r % 4 of row lane % 32
  static_assert(NW == 4 && BM % (32 * WM) == 0 && (BN % (32 * WN) == 0 || (MIX && !B_KC)), "four wavefronts, whole tiles of 32 x 32 each");
  static_assert(A_KC || BM == 64 || BM == 128, "whole loads of row-contiguous tiles");
  static_assert(B_KC || BN == 64 || BN == 128, "whole loads of row-contiguous tiles");
  static_assert(LDS_BYTES <= 80 * 1024, "two blocks per CU");

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

  template <int ROWS> __device__ static __forceinline__ int rc_swizzle(int k) { return (ROWS == 128 ? k & 3 : (k >> 1) & 1) * 64; }

  // One operand: where the pieces of its tiles come from and go to.
  template <int ROWS, bool KC>
  struct Loader {
    static constexpr int NS = (ROWS * 4 + NT - 1) / NT;  // 16-byte loads per thread and slice; of 32 rows half of the threads have none
    static constexpr int N = SLICES * NS;
    static constexpr int NO = KC ? NS : 1;
    static constexpr bool ALL = ROWS * 4 >= NT;
    static constexpr int PER_ROW = KC ? 4 : ROWS / 4;  // threads that load a row
    uint32_t off[NO], step;   // byte offsets of the loads from the tile's origin; row-contiguous ones are `step` apart
    uint32_t to;              // LDS bytes from the start of a plane
    u32x4_t v[2][N];          // fp32 values of two tiles
    __device__ __forceinline__ void start(uint32_t ld) {
      const int t = threadIdx.x, row = t / PER_ROW, p = t % PER_ROW;
      step = (uint32_t)(NT / PER_ROW) * ld * 4;
      if constexpr (KC) to = (row >> 5) * 1024 + (p >> 1) * 512 + ((row & 31) ^ (8 * (p >> 1))) * 16 + (p & 1) * 8;
      else to = row * (ROWS * 2) + ((p * 8) ^ rc_swizzle<ROWS>(row));
#pragma unroll
      for (int i = 0; i < NO; i++)
        off[i] = !KC || ALL || row < ROWS ? (uint32_t)(row + i * (NT / PER_ROW)) * ld * 4 + p * 16 : kNowhere;
    }
    // rows that a map names
    __device__ __forceinline__ void gather(const RowMap& map, uint32_t ld) {
#pragma unroll
      for (int i = 0; i < NO; i++) {
        const int row = (threadIdx.x >> 2) + i * (NT / 4);
        off[i] = row < map.rows ? (uint32_t)map(row) * ld * 4 + (threadIdx.x & 3) * 16 : kNowhere;
      }
    }
    // descriptor of the tile; `left`: bytes from its origin to the end of the operand
    __device__ static __forceinline__ __amdgpu_buffer_rsrc_t desc(const char* base, int64_t left) {
      return make_rsrc(base, left <= 0 ? 0u : left > 0xffffffffll ? 0xffffffffu : (uint32_t)left);
    }
    // k_left: valid values of K from the tile's origin on (beyond them a row of a K-contiguous operand goes on with the next one)
    template <int b, int n>
    __device__ __forceinline__ void load(__amdgpu_buffer_rsrc_t r, int k_left) {
      constexpr int slice = n / NS, j = n % NS;
      const int k = slice * SK + (threadIdx.x & 3) * 4;
      const uint32_t at = KC ? off[KC ? j : 0] + slice * (SK * ES) : off[0] + n * step;  // (kNowhere and 64 more are nowhere)
      v[b][n] = __builtin_amdgcn_raw_buffer_load_b128(r, !KC || k < k_left ? at : kNowhere, 0, 0);
    }
    // a load's values, as three planes, to LDS (`lds`: this operand's planes of the first slice)
    template <int b, int n>
    __device__ __forceinline__ void split_put(char* lds) const {
      if (!ALL && (int)threadIdx.x >= ROWS * 4) return;
      uint32_t s[2][PLANES];
#pragma unroll
      for (int i = 0; i < 2; i++) split(__uint_as_float(v[b][n][2 * i]), __uint_as_float(v[b][n][2 * i + 1]), s[i]);
      char* at = lds + to + n / NS * SLICE_BYTES + n % NS * (NT / PER_ROW) * (KC ? 32 : ROWS * 2);
#pragma unroll
      for (int x = 0; x < PLANES; x++) *reinterpret_cast<uint2*>(at + x * (ROWS * SK * 2)) = make_uint2(s[0][x], s[1][x]);
    }
    // the fp32 values themselves, [rows][16] or [16][rows] of a slice
    __device__ __forceinline__ void put_exact(char* lds) const {
#pragma unroll
      for (int n = 0; n < N; n++)
        if (ALL || (int)threadIdx.x < ROWS * 4) *reinterpret_cast<u32x4_t*>(lds + n / NS * SLICE_BYTES + (threadIdx.x + n % NS * NT) * 16) = v[0][n];
    }
  };

  // fragment of 32 rows (columns) from `row0` on of a plane: eight values of K, 8 * (lane / 32) on, of row lane % 32
  template <int ROWS, bool KC>
  __device__ static __forceinline__ frag_t frag(const char* plane, int row0, int lane) {
    if constexpr (KC) {
      const int h = lane >> 5, r = lane & 31;
      return __builtin_bit_cast(frag_t, *reinterpret_cast<const u32x4_t*>(plane + (row0 >> 5) * 1024 + h * 512 + (r ^ (8 * h)) * 16));
    } else {
      return rc_frag<ROWS>(plane, row0 + 16 * ((lane >> 4) & 1), lane);
    }
  }
  // `col`: the lane's group of 16 columns
  template <int ROWS>
  __device__ static __forceinline__ frag_t rc_frag(const char* plane, int col, int lane) {
    typedef __attribute__((address_space(3))) short4_t* lds_ptr;
    const int s = lane & 15, k = 8 * (lane >> 5) + (s >> 2);
    const char* at = plane + k * (ROWS * 2);
    const int c = (col + 4 * (s & 3)) * 2;
    const short4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(at + (c ^ rc_swizzle<ROWS>(k))));
    const short4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(at + 4 * ROWS * 2 + (c ^ rc_swizzle<ROWS>(k + 4))));
    const short8_t both = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    return __builtin_bit_cast(frag_t, both);
  }
  // the same of a fragment that is half of the first product's plane, half of the second's (`plane`: the first one's)
  __device__ static __forceinline__ frag_t mixed_frag(const char* plane, int col0, int lane) {
    const int second = (lane >> 4) & 1;
    return rc_frag<BN>(plane + second * (PLANES * B_PLANE), col0, lane);
  }

  // All K steps of a tile.  While tile t is multiplied, the values of t + 1 are split, in the shadow of the matrix instructions, and stored
  // to the other tile of LDS, and each register that this frees is loaded with its part of t + 3.  One barrier per step.
  // EXACT: the fp32 instruction; the sums are `hi`.
  template <bool EXACT, class SegFn>
  __device__ static __forceinline__ void k_loop(char* smem, int n_segs, int nk, SegFn& segf, int64_t lda, int64_t ldb, const RowMap& amap,
                                                acc_t (&hi)[MB][TM][TN], acc_t (&lo)[MB][TM][TN], int lane, int wm0, int wn0) {
    const acc_t zero = {};
#pragma unroll
    for (int nb = 0; nb < MB; nb++)
#pragma unroll
      for (int i = 0; i < TM; i++)
#pragma unroll
        for (int j = 0; j < TN; j++) {
          hi[nb][i][j] = zero;
          if (!EXACT) lo[nb][i][j] = zero;
        }
    typedef Loader<BM, A_KC> LoadA;
    typedef Loader<BN, B_KC> LoadB;
    LoadA a;
    LoadB b[NB];
    a.start((uint32_t)lda);
    if (A_KC && amap.gathered()) a.gather(amap, (uint32_t)lda);
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
    // the n-th load of a tile, to registers `buf`
    auto load = [&](auto buf, auto nc) __attribute__((always_inline)) {
      constexpr int x = decltype(buf)::value, n = decltype(nc)::value, m = n - LoadA::N;
      if constexpr (m < 0) a.template load<x, n>(ad, k_left);
      else b[m / LoadB::N].template load<x, m % LoadB::N>(bd[m / LoadB::N], k_left);
    };
    auto split_put = [&](auto buf, auto nc, char* lds) __attribute__((always_inline)) {
      constexpr int x = decltype(buf)::value, n = decltype(nc)::value, m = n - LoadA::N;
      if constexpr (m < 0) a.template split_put<x, n>(lds);
      else b[m / LoadB::N].template split_put<x, m % LoadB::N>(lds + B0 + m / LoadB::N * (PLANES * B_PLANE));
    };
    const std::integral_constant<int, 0> buf0;
    const std::integral_constant<int, 1> buf1;
    aim();
    static_for<L>([&](auto n) __attribute__((always_inline)) { load(buf0, n); });
    if constexpr (EXACT) {
      for (int it = 0; it < n_iters; it++) {
        __syncthreads();  // every wave is done with the tile before
        a.put_exact(smem);
#pragma unroll
        for (int nb = 0; nb < NB; nb++) b[nb].put_exact(smem + B0 + nb * PLANES * B_PLANE);
        const int k_here = min(BK, k_left);
        aim();
        static_for<L>([&](auto n) __attribute__((always_inline)) { load(buf0, n); });
        __syncthreads();
        const int r = lane & 31;
        for (int k0 = 0; k0 < k_here; k0 += 2) {
          const char* slice = smem + k0 / SK * SLICE_BYTES;
          const float *la = (const float*)slice, *lb = (const float*)(slice + B0);
          const int k = k0 % SK + (lane >> 5);
          float fa[TM];
#pragma unroll
          for (int i = 0; i < TM; i++) fa[i] = A_KC ? la[(wm0 + i * MT + r) * SK + k] : la[k * BM + wm0 + i * MT + r];
#pragma unroll
          for (int nb = 0; nb < MB; nb++)
#pragma unroll
            for (int j = 0; j < TN; j++) {
              const int product = MIX ? r >> 4 : nb, col = MIX ? wn0 + (r & 15) : wn0 + j * MT + r;
              const float* p = lb + product * (PLANES * B_PLANE / 4);
              const float fb = B_KC ? p[col * SK + k] : p[k * BN + col];
#pragma unroll
              for (int i = 0; i < TM; i++) hi[nb][i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(fb, fa[i], hi[nb][i][j], 0, 0, 0);
            }
        }
      }
    } else {
      aim();
      static_for<L>([&](auto n) __attribute__((always_inline)) { load(buf1, n); });
      aim();
      static_for<L>([&](auto n) __attribute__((always_inline)) {
        split_put(buf0, n, smem);
        load(buf0, n);
      });
      constexpr int PER = MB * TN, G = SLICES * PER, M = TERMS * TM;  // groups of MFMAs, by their B fragment
      // multiplies the tile in half `now` of LDS; the next one goes to the other half
      auto step = [&](auto now_c) __attribute__((always_inline)) {
        constexpr int now = decltype(now_c)::value;
        const std::integral_constant<int, 1 - now> other;
        const char* tile = smem + now * TILE_BYTES;
        char* next = smem + (1 - now) * TILE_BYTES;
        __syncthreads();  // the tile is there, and every wave is done with the one before
        aim();
        frag_t fa[SLICES][TM][PLANES], fb[2 + PLANES - 1];  // of B: planes 1 and 2, and plane 0 of the even and of the odd groups
        auto read_b = [&](auto gc, int x) __attribute__((always_inline)) {
          constexpr int q = decltype(gc)::value, nb = q % PER / TN, j = q % TN;
          const char* from = tile + q / PER * SLICE_BYTES + B0 + (nb * PLANES + x) * B_PLANE;
          frag_t& f = fb[x > 0 ? 1 + x : q & 1];
          if constexpr (MIX) f = mixed_frag(from, wn0, lane);
          else f = frag<BN, B_KC>(from, wn0 + j * MT, lane);
        };
        auto read_a = [&](int slice, int x) __attribute__((always_inline)) {
#pragma unroll
          for (int i = 0; i < TM; i++) fa[slice][i][x] = frag<BM, A_KC>(tile + slice * SLICE_BYTES + x * A_PLANE, wm0 + i * MT, lane);
        };
        static_for<PLANES>([&](auto x) __attribute__((always_inline)) {
          read_b(std::integral_constant<int, 0>(), PLANES - 1 - decltype(x)::value);
          read_a(0, x);
        });
        static_for<G>([&](auto gc) __attribute__((always_inline)) {
          constexpr int q = decltype(gc)::value, slice = q / PER, nb = q % PER / TN, j = q % TN;
          __builtin_amdgcn_sched_barrier(0);
          constexpr int n0 = q * L / G, n1 = (q + 1) * L / G;
          static_for<n1 - n0>([&](auto n) __attribute__((always_inline)) {
            const std::integral_constant<int, n0 + decltype(n)::value> which;
            split_put(other, which, next);
            load(other, which);
          });
          auto term = [&](int xb, int xa) __attribute__((always_inline)) {
#pragma unroll
            for (int i = 0; i < TM; i++) {
              acc_t& sum = xa + xb == 0 ? hi[nb][i][j] : lo[nb][i][j];
              sum = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[xb > 0 ? 1 + xb : q & 1], fa[slice][i][xa], sum, 0, 0, 0);
            }
          };
          // (in an order that lets the next group's fragments take the registers of this one's)
          auto next_b = [&](int x) __attribute__((always_inline)) {
            if constexpr (q + 1 < G) read_b(std::integral_constant<int, q + 1>(), x);
          };
          if constexpr (q + 1 < G && q / PER < (q + 1) / PER) static_for<PLANES>([&](auto x) __attribute__((always_inline)) { read_a(slice + 1, x); });
          next_b(0);
          if (TERMS == 8) term(2, 1);
          term(2, 0);
          next_b(2);
          if (TERMS == 8) term(1, 2);
          term(1, 1);
          term(1, 0);
          next_b(1);
          term(0, 2);
          term(0, 0);
          term(0, 1);
          constexpr int kValu = ((n1 - n0) * 22 + M - 1) / M;  // per MFMA
          static_for<M>([&](auto) __attribute__((always_inline)) {
            __builtin_amdgcn_sched_group_barrier(0x8, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x2, kValu, 0);
          });
        });
      };
      for (int it = 0; it < n_iters; it += 2) {
        step(buf0);
        if (it + 1 < n_iters) step(buf1);
      }
    }
  }

  template <class SegFn, class Epi>
  __device__ static __forceinline__ void run(char* smem, int n_segs, int nk, SegFn segf, int64_t lda, int64_t ldb, const Epi& epi,
                                             const RowMap& amap) {
    int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wm0 = (wave / WN) * (BM / WM), wn0 = (wave % WN) * (BN / WN);
    constexpr int NQ = MIX ? 2 : MT / 8;  // a lane's groups of four columns of a product in an accumulator tile
    f32x4_t acc[NB][TM][TN * NQ];
    auto each = [&](auto f) __attribute__((always_inline)) {  // acc = f(where it is among the sums)
#pragma unroll
      for (int nb = 0; nb < NB; nb++)
#pragma unroll
        for (int i = 0; i < TM; i++)
#pragma unroll
          for (int j = 0; j < TN; j++)
#pragma unroll
            for (int r = 0; r < 4 * NQ; r++) acc[nb][i][j * NQ + r / 4][r % 4] = f(MIX ? 0 : nb, i, j, MIX ? 8 * nb + r : r);
    };
    bool exact = n_segs * nk == 1 && segf(0).k_len <= kFew;
    if (!exact) {
      acc_t hi[MB][TM][TN], lo[MB][TM][TN];
      k_loop<false>(smem, n_segs, nk, segf, lda, ldb, amap, hi, lo, lane, wm0, wn0);
      float bad = 0.f;              // NaN if any value is not finite
      uint32_t least = 0xffffffffu;  // of the magnitudes that are not zero, as bits: twice them less one
      each([&](int nb, int i, int j, int r) __attribute__((always_inline)) {
        const float v = hi[nb][i][j][r] + lo[nb][i][j][r];
        bad = fmaf(v, 0.f, bad);
        least = min(least, 2 * __float_as_uint(v) - 1);
        return v;
      });
      const bool any = __ballot(bad != 0.f || least < 2 * kTiny - 1) != 0;  // the same in every lane of the wave
      __syncthreads();  // every wave is done with the tiles
      int* found = (int*)smem;
      if (lane == 0) found[wave] = any;
      __syncthreads();
#pragma unroll
      for (int w = 0; w < NW; w++) exact = exact || found[w] != 0;
    }
    // (what comes now forms its addresses itself: shared with the loop above they would have to be kept all through it)
    asm volatile("" : "+v"(lane), "+s"(lda), "+s"(ldb));
    if (exact) {
      acc_t sum[MB][TM][TN];
      k_loop<true>(smem, n_segs, nk, segf, lda, ldb, amap, sum, sum, lane, wm0, wn0);
      each([&](int nb, int i, int j, int r) __attribute__((always_inline)) { return sum[nb][i][j][r]; });
    }
    __syncthreads();  // every wave is done with the tiles
    TileEpilogue<NB, TM, TN * NQ, NW, LDS_BYTES, false, STAGE_ROWS, MT, false>::run(smem, acc, epi, wave, lane, wm0, wn0);
  }
};

}  // namespace moe
