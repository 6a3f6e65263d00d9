// Expert and router products whose rows are too long for the tile cores (see wide_rows).
#include "expert_impl.h"

namespace moe {

template <typename T, int NB, int EPI, bool B_KC>
__global__ __launch_bounds__(256) void wide_row_gemm_kernel(RowGemm p, int bm, int blocks_per_tile) {
  typedef Epilogue<T, NB, EPI> Epi;
  constexpr int NA = Epi::NAUX > 0 ? Epi::NAUX : 1;
  const int mt = blockIdx.x / blocks_per_tile, lane = threadIdx.x & 63;
  RowTile t;
  if (p.tiles) {
    if (mt >= *p.n_tiles) return;
    t = p.tiles[mt];
  } else {
    const int per_group = (p.n_rows + bm - 1) / bm;
    t.group = mt / per_group;
    t.row0_in = (mt - t.group * per_group) * bm;
    t.rows = min(bm, p.n_rows - t.row0_in);
    t.row0_out = t.group * p.n_rows + t.row0_in;
  }
  const int n4 = p.N / 4;
  const int64_t items = (int64_t)tile_rows(t) * n4;
  for (int64_t i = (blockIdx.x - mt * blocks_per_tile) * 4 + (threadIdx.x >> 6); i < items; i += 4 * blocks_per_tile) {
    const int m = (int)(i / n4), n = (int)(i - (int64_t)m * n4) * 4;
    const int a_row = (p.a_rows_out ? t.row0_out : t.row0_in) + m;
    const int64_t src = p.a_index ? p.a_index[a_row] / p.a_index_div : a_row;
    float v[NB][4] = {};
    for (int sg = 0; sg < p.n_pairs * p.n_segs; sg++) {
      const int pair = sg >= p.n_segs ? 1 : 0, seg = sg - pair * p.n_segs;
      const T* a = (const T*)p.A[pair] + src * p.lda + seg * p.a_seg;
      const int64_t b_off = t.group * p.b_group + seg * p.b_seg;
      for (int k = lane; k < p.K; k += 64) {
        const float x = Elem<T>::load(a + k);
#pragma unroll
        for (int nb = 0; nb < NB; nb++) {
          const T* b = (const T*)(nb == 0 ? p.B[pair] : p.Bdual) + b_off;
#pragma unroll
          for (int q = 0; q < 4; q++)
            v[nb][q] = fmaf(x, Elem<T>::load(b + (B_KC ? (int64_t)(n + q) * p.ldb + k : (int64_t)k * p.ldb + n + q)), v[nb][q]);
        }
      }
    }
#pragma unroll
    for (int nb = 0; nb < NB; nb++)
#pragma unroll
      for (int q = 0; q < 4; q++) v[nb][q] = wave_sum(v[nb][q]);
    if (lane == 0) {
      const int64_t off = ((int64_t)((p.c_rows_out ? t.row0_out : t.row0_in) + m) * p.ldc + n) * Epi::OES;
      float aux[NA][4], o[Epi::NOUT][4];
#pragma unroll
      for (int x = 0; x < Epi::NAUX; x++)
        Epi::unpack(*reinterpret_cast<const typename Epi::packed_t*>((const char*)(EPI == EPI_ADD ? p.out[0] : p.in[x]) + off), aux[x]);
      Epi epi;
      epi.apply(v, aux, p.c_scale ? p.c_scale[p.a_index[a_row]] : 1.f, o);
#pragma unroll
      for (int x = 0; x < Epi::NOUT; x++) Epi::pack((char*)p.out[x] + off, o[x]);
    }
  }
}

// weight gradients: the items are four columns of a row of every group's product(s)
template <typename T>
__global__ __launch_bounds__(256) void wide_w_gemm_kernel(WGemm p, int n_products) {
  const int lane = threadIdx.x & 63, n4 = p.N / 4;
  if (!p.ginfo && p.active_ids && blockIdx.x == 0)
    for (int i = threadIdx.x; i < p.n_groups; i += 256) {
      p.active_ids[i] = i;
      if (i == 0) *p.n_active = p.n_groups;
    }
  const int64_t per_group = (int64_t)p.M * n4, items = per_group * p.n_groups * n_products;
  for (int64_t i = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6); i < items; i += (int64_t)gridDim.x * 4) {
    const int item = (int)(i / per_group), z = item / p.n_groups, rank = item - z * p.n_groups;
    const int4 gi = p.ginfo ? p.ginfo[rank] : make_int4(rank, p.n_rows, 0, rank);  // {group, rows, first row, slot}
    if (gi.y <= 0) continue;
    const int64_t in_group = i - item * per_group;
    const int m = (int)(in_group / n4), n = (int)(in_group - (int64_t)m * n4) * 4;
    const T* a = (const T*)p.A + (gi.z + (p.a_per_group ? (int64_t)gi.x * p.n_rows : 0)) * p.lda + m;
    const T* b = (const T*)p.B[z] + (gi.z + (p.b_per_group ? (int64_t)gi.x * p.n_rows : 0)) * p.ldb + n;
    float v[4] = {};
    for (int k = lane; k < gi.y; k += 64) {
      const float x = Elem<T>::load(a + k * p.lda);
#pragma unroll
      for (int q = 0; q < 4; q++) v[q] = fmaf(x, Elem<T>::load(b + k * p.ldb + q), v[q]);
    }
#pragma unroll
    for (int q = 0; q < 4; q++) v[q] = wave_sum(v[q]);
    if (lane == 0) Epilogue<T, 1, EPI_STORE>::pack((T*)p.C[z] + (int64_t)gi.w * p.c_slot + (int64_t)m * p.N + n, v);
  }
}

constexpr int kWideBlocks = 8192;  // 4 wavefronts each, 8 per SIMD
template <typename T, int NB, int EPI, bool B_KC>
void launch_wide_row(const char* label, const RowGemm& p, int bm, int max_tiles, hipStream_t st) {
  if (max_tiles == 0) return;
  ProfScope prof(label, st);
  hipLaunchKernelGGL((wide_row_gemm_kernel<T, NB, EPI, B_KC>), dim3((unsigned)max_tiles * std::max(1, kWideBlocks / max_tiles)), dim3(256), 0,
                     st, p, bm, std::max(1, kWideBlocks / max_tiles));
}
template <typename T>
void launch_wide_w(const char* label, const WGemm& p, int n_products, hipStream_t st) {
  ProfScope prof(label, st);
  hipLaunchKernelGGL(wide_w_gemm_kernel<T>, dim3(kWideBlocks), dim3(256), 0, st, p, n_products);
}

#define MOE_WIDE(T)                                                                                        \
  template void launch_wide_w<T>(const char*, const WGemm&, int, hipStream_t);                             \
  MOE_WIDE_ROW(T, 2, EPI_SWIGLU_FWD, false)                                                                \
  MOE_WIDE_ROW(T, 1, EPI_GELU_FWD, false)                                                                  \
  MOE_WIDE_ROW(T, 1, EPI_STORE, false)                                                                     \
  MOE_WIDE_ROW(T, 1, EPI_STORE_F32, false)                                                                 \
  MOE_WIDE_ROW(T, 1, EPI_SWIGLU_BWD, true)                                                                 \
  MOE_WIDE_ROW(T, 1, EPI_GELU_BWD, true)                                                                   \
  MOE_WIDE_ROW(T, 1, EPI_STORE, true)                                                                      \
  MOE_WIDE_ROW(T, 1, EPI_ADD, true)
#define MOE_WIDE_ROW(T, NB, EPI, B_KC) \
  template void launch_wide_row<T, NB, EPI, B_KC>(const char*, const RowGemm&, int, int, hipStream_t);
MOE_WIDE(float)
MOE_WIDE(bf16_t)
}  // namespace moe
