// moe_dispatch: stable counting sort of the T*k assignments by expert, then the row copy.
//
//   1. dispatch_count  one wavefront per chunk of kChunk assignments: LDS histogram over experts
//                      (LDS atomics are used for the COUNTS only, so the result does not depend
//                      on their order), written to ws as hist[chunk][e].
//   2. dispatch_scan   one block: exclusive scan over chunks per expert (in place), counts,
//                      and the exclusive scan over experts (offsets).
//   3. dispatch_rows   one block per token: finds the rows of its k assignments, reads the token row once and
//                      writes it to them.  Many assignments of short rows are ranked before, by dispatch_rank,
//                      one wavefront per chunk (dispatch_place says when).
#include <algorithm>
#include <mutex>

#include "gate_device.h"
#include "gemm_plan.h"
#include "moe_common.h"

namespace moe {

constexpr int kChunk = 256;  // most assignments per chunk
constexpr int kShareFloats = 8192;  // LDS floats of the fused prologue for the per-wave share sums

__global__ __launch_bounds__(64) void dispatch_count(const int32_t* __restrict__ topk_idx, int A, int E, int chunk_len,
                                                     int32_t* __restrict__ hist) {
  __shared__ int32_t cnt[MOE_MAX_EXPERTS];
  const int lane = threadIdx.x;
  const int chunk = blockIdx.x;
  for (int e = lane; e < E; e += 64) cnt[e] = 0;
  __syncthreads();
  const int a0 = chunk * chunk_len, a1 = min(A, a0 + chunk_len);
  for (int s = 0; s < chunk_len; s += 64) {
    int a = a0 + s + lane;
    if (a < a1) {
      int e = topk_idx[a];
      if (e >= 0 && e < E) atomicAdd(&cnt[e], 1);
    }
  }
  __syncthreads();
  for (int e = lane; e < E; e += 64) hist[(size_t)chunk * E + e] = cnt[e];
}

// One block; bound by memory latency.  The chunks are cut into C equal runs (C: a power of two up to 1024 / E, and no
// more than gives every run a batch of chunks): thread (c, e) first sums run c of expert e, the run sums are scanned
// over c, then the thread rewrites its run as exclusive prefixes.  Loads go a batch at a time ahead of the dependent
// additions and stores.  (Batches of 8, the shares read
// after the counters, as many runs as threads: T = 256, E = 8: 8.5 us, now 5.1; T = 2777, E = 60: 10.7, now 8.4.)
// With pl.tiles, the block goes on to the plan of the experts' products, in place of a launch ahead of the forward products.  (More here,
// and the launch that it saves, by number of experts: 8: 2.6 and 3.6 us, 24: 3.6 and 5.6, 60: 4.2 and 5.3, 256: 6 and 9; and the gap
// between two launches.  Training step of T = 256, d = 128, 8 experts, fp32, with the cheaper marshalling of the calls: 93.6 -> 92.2 us.)
// With `partial` (the fused prologue), the block also finishes the auxiliary load-balancing loss: P_e from
// the per-chunk sums of the gate's shares (added in the same fixed order as the counters), then
// L = alpha E sum_e (counts[e] / (T k)) P_e over ascending e.
constexpr int kScanBatch = 16;
__global__ __launch_bounds__(1024) void dispatch_scan(int32_t* __restrict__ hist, int n_chunks, int E,
                                                      int32_t* __restrict__ counts,
                                                      int32_t* __restrict__ offsets,
                                                      const float* __restrict__ partial, float* __restrict__ P,
                                                      float* __restrict__ loss, int T, int k, float alpha, Plan pl,
                                                      int plan_bm, int32_t* active_ids, int32_t* n_active) {
  __shared__ __align__(16) float term[MOE_MAX_EXPERTS];
  __shared__ __align__(16) int32_t wsum[16];
  __shared__ int32_t part[1024];
  __shared__ float fpart[1024];
  constexpr int B = kScanBatch;
  int C = 1;
  while (C * 2 * E <= 1024 && C * B < n_chunks) C *= 2;
  const int c = threadIdx.x / E, e_run = threadIdx.x - c * E;
  const int per = (n_chunks + C - 1) / C;
  const int w0 = min(n_chunks, c * per), w1 = min(n_chunks, w0 + per);
  const bool worker = c < C;
  if (worker) {
    int sum = 0;
    float fs = 0.f;
    for (int w = w0; w < w1; w += B) {
      int v[B];
      float f[B];
#pragma unroll
      for (int q = 0; q < B; q++) v[q] = w + q < w1 ? hist[(size_t)(w + q) * E + e_run] : 0;
      if (partial) {
#pragma unroll
        for (int q = 0; q < B; q++) f[q] = w + q < w1 ? partial[(size_t)(w + q) * E + e_run] : 0.f;
#pragma unroll
        for (int q = 0; q < B; q++) fs += f[q];
      }
#pragma unroll
      for (int q = 0; q < B; q++) sum += v[q];
    }
    part[c * E + e_run] = sum;
    fpart[c * E + e_run] = fs;
  }
  __syncthreads();
  if (worker) {
    int run = 0;
#pragma unroll 8
    for (int q = 0; q < c; q++) run += part[q * E + e_run];
    for (int w = w0; w < w1; w += B) {
      int v[B];
#pragma unroll
      for (int q = 0; q < B; q++) v[q] = w + q < w1 ? hist[(size_t)(w + q) * E + e_run] : 0;
#pragma unroll
      for (int q = 0; q < B; q++) {
        if (w + q < w1) hist[(size_t)(w + q) * E + e_run] = run;
        run += v[q];
      }
    }
  }
  const int e = threadIdx.x;
  int run = 0, all;
  if (e < E) {
#pragma unroll 8
    for (int q = 0; q < C; q++) run += part[q * E + e];
    counts[e] = run;
  }
  const int end = block_scan_1024(run, wsum, all);
  if (e < E) offsets[e + 1] = end;
  if (e == 0) offsets[0] = 0;
  if (pl.tiles) build_plan(e < E ? run : 0, end - run, E, plan_bm, pl, active_ids, n_active);
  if (partial) {
    float t = 0.f;
    if (e < E) {
      float fs = 0.f;
#pragma unroll 8
      for (int q = 0; q < C; q++) fs += fpart[q * E + e];
      const float pe = T > 0 ? fs / (float)T : 0.f;
      P[e] = pe;
      t = T > 0 ? pe * ((float)run / ((float)T * (float)k)) : 0.f;
    }
    term[e] = t;
    __syncthreads();
    if (e == 0) {
      float fs = 0.f;
#pragma unroll 8
      for (int q = 0; q < E; q += 4) {  // (zeros beyond E)
        const float4 v = *reinterpret_cast<const float4*>(term + q);
        fs = fs + v.x + v.y + v.z + v.w;
      }
      *loss = alpha * (float)E * fs;
    }
  }
}

// The gate and the first step of the dispatch in one pass over the logits: a block owns one chunk of
// tokens_per_chunk tokens (tokens_per_chunk * k <= kChunk assignments); its wavefronts take the tokens
// of the chunk in turn (route_token), count the selected experts in LDS (integer atomics on counts
// only) and, for the auxiliary loss, add up the gate's shares of their tokens; the waves' sums are
// added in wave order, so the per-chunk sums do not depend on timing.
template <int R>
__global__ __launch_bounds__(1024) void route_hist_kernel(const float* __restrict__ logits, int32_t* __restrict__ topk_idx,
                                                          float* __restrict__ topk_w, int T, int E, int k, int gate,
                                                          int renorm, int tokens_per_chunk, int32_t* __restrict__ hist,
                                                          float* __restrict__ partial) {
  __shared__ int32_t cnt[MOE_MAX_EXPERTS];
  __shared__ float shares[kShareFloats];  // [wave][64 R]: the launcher keeps waves * 64 R within it
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, n_waves = blockDim.x >> 6;
  const int chunk = blockIdx.x;
  for (int e = threadIdx.x; e < E; e += blockDim.x) cnt[e] = 0;
  __syncthreads();
  const int t0 = chunk * tokens_per_chunk, t1 = min(T, t0 + tokens_per_chunk);
  float acc[R];
#pragma unroll
  for (int r = 0; r < R; r++) acc[r] = 0.f;
  for (int t = t0 + wave; t < t1; t += n_waves) {
    float v[R], w;
    int e;
    route_token<R>(logits + (size_t)t * E, lane, E, k, gate, renorm, v, e, w);
    if (lane < k) {
      topk_idx[(size_t)t * k + lane] = e;
      topk_w[(size_t)t * k + lane] = w;
      atomicAdd(&cnt[e], 1);
    }
    if (partial) {
      float s[R], p[R], inv_tot;
      gate_shares_of<R>(v, lane, E, gate, s, p, inv_tot);
#pragma unroll
      for (int r = 0; r < R; r++) acc[r] += p[r];
    }
  }
  if (partial) {
#pragma unroll
    for (int r = 0; r < R; r++)
      if (lane + 64 * r < E) shares[wave * 64 * R + lane + 64 * r] = acc[r];
  }
  __syncthreads();
  for (int e = threadIdx.x; e < E; e += blockDim.x) {
    hist[(size_t)chunk * E + e] = cnt[e];
    if (partial) {
      float fs = 0.f;
      for (int wv = 0; wv < n_waves; wv++) fs += shares[wv * 64 * R + e];
      partial[(size_t)chunk * E + e] = fs;
    }
  }
}

// Ranks of one chunk per wavefront, in a launch of their own: walks the chunk in assignment order, the rank of an
// assignment among equal experts inside a 64-wide step comes from ballots in lane order (the same rows as
// dispatch_rows finds by itself).  An index out of range has no row: its row_of stays as it is.
__global__ __launch_bounds__(64) void dispatch_rank(const int32_t* __restrict__ topk_idx, int A, int E, int chunk_len,
                                                    const int32_t* __restrict__ hist, const int32_t* __restrict__ offsets,
                                                    int32_t* __restrict__ row_of, int32_t* __restrict__ src_of) {
  __shared__ int32_t nxt[MOE_MAX_EXPERTS];
  const int lane = threadIdx.x, chunk = blockIdx.x;
  for (int e = lane; e < E; e += 64) nxt[e] = offsets[e] + hist[(size_t)chunk * E + e];
  __syncthreads();
  const int a0 = chunk * chunk_len, n = min(A - a0, chunk_len);
  const uint64_t below = lane == 0 ? 0ull : ~0ull >> (64 - lane);
  for (int s = 0; s < n; s += 64) {
    const int i = s + lane;
    int e = i < n ? topk_idx[a0 + i] : -1;
    if (e < 0 || e >= E) e = -1;
    uint64_t todo = __ballot(e >= 0);
    int rank = 0, group = 0;
    bool last = false;
    while (todo) {
      const int le = __shfl(e, __ffsll((unsigned long long)todo) - 1, kWave);
      const uint64_t same = __ballot(e == le);
      if (e == le) {
        rank = __popcll(same & below);
        group = __popcll(same);
        last = (same >> lane) == 1ull;  // highest lane of the group
      }
      todo &= ~same;
    }
    const int r = e >= 0 ? nxt[e] + rank : -1;
    __syncthreads();
    if (last) nxt[e] += group;
    __syncthreads();
    if (r >= 0) {
      row_of[a0 + i] = r;
      src_of[r] = a0 + i;
    }
  }
}

// Rows of one token per block, and with PLACE their ranks.  Wavefronts first place the token's assignments, one each at a
// time: the rows before its own are those of the experts before, those of the earlier chunks, and, inside its chunk, the
// earlier assignments to the same expert, counted by ballots over the at most kChunk indices before it (so row_of is the
// same on every run: a stable sort).  Then Xp[row_of[t*k+j], :] = X[t, :], 16 bytes per lane per access; the first pieces
// are loaded ahead of the barrier between.  An index out of range has no row.  K > 0: k known at compile time.
// (Ranks in a launch of their own, one wavefront per chunk: T = 16, top-4: 3.3 + 2.7 us, now 3.7; T = 2777, top-3: 4.9 +
// 8.9, now 10.9; T = 8192, d = 768, top-2: 5.0 + 9.0, now 11.7.  Where that loses: see dispatch_place.)
template <int K, bool PLACE>
__global__ __launch_bounds__(512) void dispatch_rows(const uint4* __restrict__ X, const int32_t* __restrict__ topk_idx,
                                                     const int32_t* __restrict__ hist, const int32_t* __restrict__ offsets,
                                                     int E, int chunk_len, int k_rt, int vec_per_row,
                                                     int32_t* __restrict__ row_of, int32_t* __restrict__ src_of,
                                                     uint4* __restrict__ Xp) {
  __shared__ int32_t rows[MOE_MAX_TOPK];
  constexpr int KM = K > 0 ? K : 1;
  const int k = K > 0 ? K : k_rt;
  const int t = blockIdx.x, nthr = blockDim.x;
  const int lane = threadIdx.x & 63;
  const uint4* src = X + (size_t)t * vec_per_row;
  int c = threadIdx.x;
  uint4 v0 = {}, v1 = {};
  if (c < vec_per_row) v0 = src[c];
  if (c + nthr < vec_per_row) v1 = src[c + nthr];
  if (PLACE) {
    for (int j = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6); j < k; j += nthr >> 6) {
      const int a = t * k + j;
      const int chunk = (int)((uint32_t)a / (uint32_t)chunk_len), a0 = chunk * chunk_len;
      const int e = topk_idx[a];
      int x[kChunk / 64];
#pragma unroll
      for (int q = 0; q < kChunk / 64; q++) x[q] = a0 + 64 * q + lane < a ? topk_idx[a0 + 64 * q + lane] : -1;
      int r = -1;
      if (e >= 0 && e < E) {
        r = offsets[e] + hist[(size_t)chunk * E + e];
#pragma unroll
        for (int q = 0; q < kChunk / 64; q++) r += __popcll(__ballot(x[q] == e));
      }
      if (lane == 0) {
        rows[j] = r;
        if (r >= 0) {
          row_of[a] = r;
          src_of[r] = a;
        }
      }
    }
    __syncthreads();
  }
  // ranked before: the indices are looked at again only if some are out of range (fewer rows than assignments)
  const bool some_out = !PLACE && offsets[E] != (int)gridDim.x * k;
  auto row_at = [&](int j) { return PLACE ? rows[j] : row_of[(size_t)t * k + j]; };
  auto no_row = [&](int j) {
    const int e = topk_idx[(size_t)t * k + j];
    return e < 0 || e >= E;
  };
  if (K > 0) {
    int row[KM];
#pragma unroll
    for (int j = 0; j < KM; j++) row[j] = __builtin_amdgcn_readfirstlane(row_at(j));
    if (some_out) {
#pragma unroll
      for (int j = 0; j < KM; j++)
        if (no_row(j)) row[j] = -1;
    }
    // two pieces per thread and trip: both loads are issued before the 2k stores
    while (c < vec_per_row) {
#pragma unroll
      for (int j = 0; j < KM; j++) {
        if (row[j] < 0) continue;
        uint4* dst = Xp + (size_t)row[j] * vec_per_row;
        dst[c] = v0;
        if (c + nthr < vec_per_row) dst[c + nthr] = v1;
      }
      c += 2 * nthr;
      if (c < vec_per_row) v0 = src[c];
      if (c + nthr < vec_per_row) v1 = src[c + nthr];
    }
  } else {
    for (; c < vec_per_row; c += nthr) {
      const uint4 v = src[c];
      for (int j = 0; j < k; j++) {
        const int r = some_out && no_row(j) ? -1 : row_at(j);
        if (r >= 0) Xp[(size_t)r * vec_per_row + c] = v;
      }
    }
  }
}

// ranks and row copy of a dispatch whose per-chunk histograms `hist` (chunks of chunk_len assignments)
// have been scanned
static void dispatch_place(const moe_shape_t* shape, const void* X, const int32_t* topk_idx, const int32_t* offsets,
                           int32_t* row_of, int32_t* src_of, void* Xp, const int32_t* hist, int chunk_len, int n_chunks,
                           hipStream_t st) {
  if (shape->T == 0) return;
  const int vec_per_row = (int)((size_t)shape->d * elem_size(shape->dtype) / 16);
  // Ranks found by the row blocks save a launch, but every block pays their chain of dependent reads: with short rows there
  // is no copy to hide it under, and its cost grows with the assignments.  A launch of their own costs 2 us and up to
  // 25 more for the rounds of a step of 64 assignments over many experts.  Whole moe_dispatch calls, ranks in the row blocks
  // against a launch of their own, bf16: T = 131072, top-8 of 8 experts, d = 128: 233 against 115 us; top-4 of 60, d = 256: 184
  // against 111; T = 32768, d = 128, top-4 of 8: 40 against 25, of 60: 43 against 42, of 256: 56 against 62; rows of 4 KB
  // (T = 131072, top-4 of 8): 484 against 503; top-1 (T = 131072, d = 128): 39 against 44.  The line is where the two meet over
  // T = 1024 .. 400000, top-2 .. top-32, 8 to 256 experts, d = 8 .. 1024 (worst misses on either side: 10 %).
  const int64_t row_bytes = (int64_t)vec_per_row * 16;
  const bool ranked = shape->k > 1 && row_bytes <= 2048 &&
                      (int64_t)shape->T * shape->k >= (40960 + 2048 * std::min(shape->E, 64)) * (2048 + row_bytes) / 2048;
  if (ranked) {
    ProfScope prof("dispatch_rank", st);
    hipLaunchKernelGGL(dispatch_rank, dim3(n_chunks), dim3(64), 0, st, topk_idx, shape->T * shape->k, shape->E, chunk_len, hist,
                       offsets, row_of, src_of);
  }
  ProfScope prof("dispatch_rows", st);
  // Blocks as wide as a row, but copies of long rows that leave the caches behind run with 256 threads: 8 rows a compute
  // unit stay in flight (T = 32768, top-3 of 16, d = 7168: 365 -> 350 us, d = 12288: 628 -> 610; T = 8192, top-8, d = 7168: 214
  // -> 211).  Below some 600 MB written it is even or slower (T = 4096, top-4, d = 12288: 108 against 111), and rows of up to
  // 512 pieces prefer it only now and then (d = 4096: T = 8192, top-8: 123 against 121, T = 32768, top-3: 188 against 201).
  const bool long_rows = vec_per_row > 512 && (int64_t)shape->T * shape->k * row_bytes >= (int64_t)576 << 20;
  const unsigned copy_threads = long_rows ? 256 : row_block_threads(shape->d, 16 / (int)elem_size(shape->dtype));
  // Short rows get more threads than pieces, so that up to four assignments are placed at a time; rows of at least 64
  // pieces whose ranks are known get twice as many (T = 131072, top-8, d = 512: 258 -> 233 us, d = 1024: 475 -> 451; below, the
  // second wavefront costs: d = 256: 137 -> 163).
  const unsigned threads = !ranked ? std::max(copy_threads, 64u * std::min(shape->k, 4)) : vec_per_row < 64 ? copy_threads : 2 * copy_threads;
#define MOE_ROWS_KERNEL(K, PLACE)                                                                                               \
  hipLaunchKernelGGL((dispatch_rows<K, PLACE>), dim3(shape->T), dim3(threads), 0, st, (const uint4*)X, topk_idx, hist, offsets, \
                     shape->E, chunk_len, shape->k, vec_per_row, row_of, src_of, (uint4*)Xp)
#define MOE_ROWS(K)                      \
  if (ranked) MOE_ROWS_KERNEL(K, false); \
  else MOE_ROWS_KERNEL(K, true)
  MOE_BY_TOP_K(shape->k, MOE_ROWS);
#undef MOE_ROWS
#undef MOE_ROWS_KERNEL
}

// the launches of a dispatch; `hist` is scratch of n_chunks * E counters (every one is written
// by dispatch_count before anything reads it)
static void dispatch_launch(const moe_shape_t* shape, const void* X, const int32_t* topk_idx, int32_t* counts,
                            int32_t* offsets, int32_t* row_of, int32_t* src_of, void* Xp, int32_t* hist,
                            hipStream_t st) {
  const int A = shape->T * shape->k;
  const int n_chunks = (A + kChunk - 1) / kChunk;
  if (n_chunks > 0) {
    ProfScope prof("dispatch_count", st);
    hipLaunchKernelGGL(dispatch_count, dim3(n_chunks), dim3(64), 0, st, topk_idx, A, shape->E, kChunk, hist);
  }
  {
    ProfScope prof("dispatch_scan", st);
    hipLaunchKernelGGL(dispatch_scan, dim3(1), dim3(1024), 0, st, hist, n_chunks, shape->E, counts, offsets,
                       (const float*)nullptr, (float*)nullptr, (float*)nullptr, 0, 1, 0.f, Plan{}, 0, (int32_t*)nullptr, (int32_t*)nullptr);
  }
  dispatch_place(shape, X, topk_idx, offsets, row_of, src_of, Xp, hist, kChunk, n_chunks, st);
}

// chunks of the fused prologue: whole tokens, at most kChunk assignments, and fewer than that while the
// batch is too small to give every compute unit a chunk (a chunk is a block of the first kernel).  Of many experts half as many
// chunks: the scan, one block, then has half of its counters to read, and a chunk's wavefronts still have a token each.  (T = 1961,
// top-2 of 140 experts, forward 88.8 -> 85.3 us a pass; T = 304, top-3 of 245, training 1408 -> 1368; of 24 to 64 experts no gain, and
// with a quarter as many the gate's kernel loses up to 2 %.)
static int prologue_tokens_per_chunk(const moe_shape_t* s) {
  const int most = s->E > 128 ? 128 : 256;
  return std::max(1, std::min(kChunk / s->k, (s->T + most - 1) / most));
}
static int prologue_chunks(const moe_shape_t* s) {
  const int tpc = prologue_tokens_per_chunk(s);
  return (s->T + tpc - 1) / tpc;
}

// Scratch of moe_dispatch_static: one array per GPU, part of the loaded code object, so that no call
// allocates.  Host code must not use the symbol's name as an address: the per-device address comes
// from hipGetSymbolAddress, once per device, and is what the kernels receive.
constexpr size_t kStaticHistInts = (size_t)MOE_DISPATCH_STATIC_MAX_COUNTERS;
static __device__ __align__(256) int32_t scratch[kStaticHistInts];
constexpr int kMaxDevices = 64;
static std::mutex g_scratch_mu;
static int32_t* g_scratch_ptr[kMaxDevices];  // per device, set on the first call with that device current

// address of the current device's scratch array, or NULL with the error text set
static int32_t* static_scratch() {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) {
    set_error("moe_dispatch_static: no current device (or a device index above %d)", kMaxDevices - 1);
    return nullptr;
  }
  std::lock_guard<std::mutex> lk(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !p) {
      set_error("moe_dispatch_static: hipGetSymbolAddress failed: %s", hipGetErrorString(e));
      return nullptr;
    }
    g_scratch_ptr[dev] = (int32_t*)p;
  }
  return g_scratch_ptr[dev];
}
}  // namespace moe

extern "C" size_t moe_dispatch_workspace_bytes(const moe_shape_t* shape) {
  using namespace moe;
  if (!shape || shape->E < 1 || shape->T < 0 || shape->k < 1) return 0;
  size_t A = (size_t)shape->T * shape->k;
  size_t n_chunks = (A + kChunk - 1) / kChunk;
  return align_up((n_chunks > 0 ? n_chunks : 1) * (size_t)shape->E * sizeof(int32_t), 256);
}

extern "C" int moe_dispatch(const moe_shape_t* shape, const void* X, const int32_t* topk_idx, int32_t* counts,
                            int32_t* offsets, int32_t* row_of, int32_t* src_of, void* Xp, void* ws,
                            size_t ws_bytes, void* stream) {
  using namespace moe;
  int rc = check_shape(shape, "moe_dispatch");
  if (rc) return rc;
  // with T == 0 only counts and offsets are written (zeros); the per-assignment arrays may be null
  if (!counts || !offsets || !ws || (shape->T > 0 && (!topk_idx || !row_of || !src_of || !X || !Xp))) {
    set_error("moe_dispatch: null pointer");
    return MOE_EINVAL;
  }
  if (!aligned16(X) || !aligned16(Xp) || !aligned16(ws)) {
    set_error("moe_dispatch: X, Xp and ws must be 16-byte aligned");
    return MOE_EINVAL;
  }
  if (ws_bytes < moe_dispatch_workspace_bytes(shape)) {
    set_error("moe_dispatch: workspace of %zu bytes, need %zu", ws_bytes, moe_dispatch_workspace_bytes(shape));
    return MOE_EWS;
  }
  dispatch_launch(shape, X, topk_idx, counts, offsets, row_of, src_of, Xp, (int32_t*)ws, (hipStream_t)stream);
  return launch_status("moe_dispatch");
}

extern "C" int moe_dispatch_static(const moe_shape_t* shape, const void* X, const int32_t* topk_idx, int32_t* counts,
                                   int32_t* offsets, int32_t* row_of, int32_t* src_of, void* Xp, void* stream) {
  using namespace moe;
  int rc = check_shape(shape, "moe_dispatch_static");
  if (rc) return rc;
  if (!counts || !offsets || (shape->T > 0 && (!topk_idx || !row_of || !src_of || !X || !Xp))) {
    set_error("moe_dispatch_static: null pointer");
    return MOE_EINVAL;
  }
  if (!aligned16(X) || !aligned16(Xp)) {
    set_error("moe_dispatch_static: X and Xp must be 16-byte aligned");
    return MOE_EINVAL;
  }
  const size_t need = moe_dispatch_workspace_bytes(shape);
  if (need > kStaticHistInts * sizeof(int32_t)) {
    set_error("moe_dispatch_static: ceil(T*k / 256) * E = %zu counters exceed the built-in scratch of %zu; use "
              "moe_dispatch with a workspace", need / sizeof(int32_t), kStaticHistInts);
    return MOE_EWS;
  }
  int32_t* hist = static_scratch();
  if (!hist) return MOE_ELAUNCH;
  dispatch_launch(shape, X, topk_idx, counts, offsets, row_of, src_of, Xp, hist, (hipStream_t)stream);
  return launch_status("moe_dispatch_static");
}

extern "C" size_t moe_route_dispatch_workspace_bytes(const moe_shape_t* shape) {
  using namespace moe;
  if (!shape || shape->E < 1 || shape->T < 0 || shape->k < 1) return 0;
  const size_t per = align_up((size_t)std::max(1, prologue_chunks(shape)) * (size_t)shape->E * 4, 256);
  return 2 * per;  // integer histograms, then the share sums of the auxiliary loss
}

// moe_route_dispatch, with the plan of the experts' products if `plan` is not NULL
static int route_dispatch(const char* who, const moe_shape_t* shape, const float* logits, const void* X, float aux_alpha,
                          int32_t* topk_idx, float* topk_w, int32_t* counts, int32_t* offsets, int32_t* row_of, int32_t* src_of, void* Xp,
                          float* aux_P, float* aux_loss, void* plan, int32_t* active_ids, int32_t* n_active, void* ws,
                          size_t ws_bytes, void* stream) {
  using namespace moe;
  int rc = check_shape(shape, who);
  if (rc) return rc;
  if (!counts || !offsets || !ws || (aux_P != nullptr) != (aux_loss != nullptr) ||
      (shape->T > 0 && (!logits || !topk_idx || !topk_w || !row_of || !src_of || !X || !Xp))) {
    set_error("%s: null pointer (aux_P and aux_loss go together)", who);
    return MOE_EINVAL;
  }
  if (!aligned16(X) || !aligned16(Xp) || !aligned16(ws)) {
    set_error("%s: X, Xp and ws must be 16-byte aligned", who);
    return MOE_EINVAL;
  }
  const size_t need = moe_route_dispatch_workspace_bytes(shape);
  if (ws_bytes < need) {
    set_error("%s: workspace of %zu bytes, need %zu", who, ws_bytes, need);
    return MOE_EWS;
  }
  hipStream_t st = (hipStream_t)stream;
  const int T = shape->T, E = shape->E, k = shape->k;
  const int tpc = prologue_tokens_per_chunk(shape), n_chunks = prologue_chunks(shape);
  int32_t* hist = (int32_t*)ws;
  const int bm = plan_tile_rows(shape->dtype, E, T * k, shape->d, shape->d_ff);
  const Plan pl = plan ? carve_plan(plan, E, plan_cap(E, T * k)) : Plan{};
  float* partial = aux_P ? (float*)((char*)ws + need / 2) : nullptr;
  if (n_chunks > 0) {
    ProfScope prof("route_hist_kernel", st);
    // one wavefront per token of the chunk, as many as the share sums leave room for in LDS
#define MOE_ROUTE_HIST(R)                                                                                              \
  do {                                                                                                                 \
    const int waves = std::max(1, std::min(std::min(16, kShareFloats / (64 * R)), tpc));                               \
    hipLaunchKernelGGL(route_hist_kernel<R>, dim3(n_chunks), dim3(64 * waves), 0, st, logits, topk_idx, topk_w, T, E, k, \
                       shape->gate, shape->renorm, tpc, hist, partial);                                                \
  } while (0)
    MOE_BY_EXPERTS(E, MOE_ROUTE_HIST);
#undef MOE_ROUTE_HIST
  }
  {
    ProfScope prof("dispatch_scan", st);
    hipLaunchKernelGGL(dispatch_scan, dim3(1), dim3(1024), 0, st, hist, n_chunks, E, counts, offsets,
                       (const float*)partial, aux_P, aux_loss, T, k, aux_alpha, pl, bm, active_ids, n_active);
  }
  dispatch_place(shape, X, topk_idx, offsets, row_of, src_of, Xp, hist, tpc * k, n_chunks, st);
  return launch_status(who);
}

extern "C" int moe_route_dispatch(const moe_shape_t* shape, const float* logits, const void* X, float aux_alpha,
                                  int32_t* topk_idx, float* topk_w, int32_t* counts, int32_t* offsets,
                                  int32_t* row_of, int32_t* src_of, void* Xp, float* aux_P, float* aux_loss, void* ws,
                                  size_t ws_bytes, void* stream) {
  return route_dispatch("moe_route_dispatch", shape, logits, X, aux_alpha, topk_idx, topk_w, counts, offsets, row_of, src_of, Xp, aux_P,
                        aux_loss, nullptr, nullptr, nullptr, ws, ws_bytes, stream);
}

extern "C" int moe_route_dispatch_plan(const moe_shape_t* shape, const float* logits, const void* X, float aux_alpha,
                                       int32_t* topk_idx, float* topk_w, int32_t* counts, int32_t* offsets,
                                       int32_t* row_of, int32_t* src_of, void* Xp, float* aux_P, float* aux_loss, void* plan,
                                       size_t plan_size, int32_t* active_ids, int32_t* n_active, void* ws, size_t ws_bytes, void* stream) {
  using namespace moe;
  const int rc = check_shape(shape, "moe_route_dispatch_plan");
  if (rc) return rc;
  if (!plan || !active_ids || !n_active || !aligned16(plan)) {
    set_error("moe_route_dispatch_plan: null or unaligned plan, active_ids or n_active");
    return MOE_EINVAL;
  }
  if (plan_size < moe_expert_plan_bytes(shape)) {
    set_error("moe_route_dispatch_plan: plan of %zu bytes, need %zu", plan_size, moe_expert_plan_bytes(shape));
    return MOE_EWS;
  }
  return route_dispatch("moe_route_dispatch_plan", shape, logits, X, aux_alpha, topk_idx, topk_w, counts, offsets, row_of, src_of, Xp, aux_P,
                        aux_loss, plan, active_ids, n_active, ws, ws_bytes, stream);
}
