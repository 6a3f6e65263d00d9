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
#include "expert_impl.h"

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

void launch_plan(const int32_t* offsets, int n_groups, int n_rows, int BM, const Plan& pl, int32_t* active_ids, int32_t* n_active,
                 hipStream_t st) {
  ProfScope prof("plan_kernel", st);
  hipLaunchKernelGGL(plan_kernel, dim3(1), dim3(1024), 0, st, offsets, n_groups, n_rows, BM, pl, active_ids, n_active);
}

// one translation unit each
#define MOE_CORES(PATH)                                                                                                 \
  extern template void expert_fwd_impl<PATH>(const FwdArgs&, hipStream_t);                                            \
  extern template void expert_bwd_impl<PATH>(const BwdArgs&, hipStream_t);                                            \
  extern template void router_fwd_impl<PATH>(const moe_shape_t*, const void*, const void*, float*, char*, char*,      \
                                             size_t, hipStream_t);                                                     \
  extern template void router_bwd_impl<PATH>(const moe_shape_t*, const void*, const void*, const float*, void*, void*, \
                                             bool, char*, char*, size_t, hipStream_t);
MOE_CORES(PATH_F32)
MOE_CORES(PATH_BF16_TAIL)
MOE_CORES(PATH_BF16)

static int pick_path(const moe_shape_t* s) {
  if (s->dtype == MOE_F32) return PATH_F32;
  return (s->d % 64 == 0 && s->d_ff % 64 == 0) ? PATH_BF16 : PATH_BF16_TAIL;
}

static size_t plan_size_for(int n_groups, int n_rows, bool shared) {
  // sized for the smallest row tile of any path, so the query does not depend on the path taken
  const int bound = shared ? n_groups * (n_rows / 64 + 2) : max_row_tiles(n_groups, n_rows, 64);
  return align_up(plan_bytes(n_groups, bound + 1), 256);
}
// dG and dU: [n_rows, d_ff] each; shared mode keeps them per group
static size_t grad_size_for(const moe_shape_t* s, int n_groups, int n_rows, bool shared) {
  return align_up((size_t)(shared ? n_groups : 1) * (size_t)n_rows * s->d_ff * elem_size(s->dtype), 256);
}
// what a call needs; shared calls use more where it is there (for products summed in parts), and the queries
// below ask for as much as they can use
static size_t fwd_base(const moe_shape_t*, int n_groups, int n_rows, bool shared) { return plan_size_for(n_groups, n_rows, shared); }
static size_t bwd_base(const moe_shape_t* s, int n_groups, int n_rows, bool shared) {
  return plan_size_for(n_groups, n_rows, shared) + 2 * grad_size_for(s, n_groups, n_rows, shared);
}
static size_t shared_parts(const moe_shape_t* s, int n_groups, int n_rows, bool bwd) {
  switch (pick_path(s)) {
    case PATH_F32: return expert_part_bytes<PATH_F32>(s->d, s->d_ff, n_groups, n_rows, bwd);
    case PATH_BF16_TAIL: return expert_part_bytes<PATH_BF16_TAIL>(s->d, s->d_ff, n_groups, n_rows, bwd);
    default: return expert_part_bytes<PATH_BF16>(s->d, s->d_ff, n_groups, n_rows, bwd);
  }
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
  return fwd_base(shape, n_groups, n_rows, shared != 0) + (shared ? shared_parts(shape, n_groups, n_rows, false) : 0);
}

// plan + dG + dU + parts
extern "C" size_t moe_expert_bwd_workspace_bytes(const moe_shape_t* shape, int32_t n_groups, int32_t n_rows,
                                                 int32_t shared) {
  using namespace moe;
  if (!shape || n_groups < 1 || n_rows < 0) return 0;
  return bwd_base(shape, n_groups, n_rows, shared != 0) + (shared ? shared_parts(shape, n_groups, n_rows, true) : 0);
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
  const size_t need = fwd_base(shape, n_groups, n_rows, offsets == nullptr);
  if (ws_bytes < need) {
    set_error("moe_expert_fwd: workspace of %zu bytes, need %zu", ws_bytes, need);
    return MOE_EWS;
  }
  if (n_rows == 0) return MOE_OK;
  FwdArgs a = {shape->d, shape->d_ff, n_groups, n_rows, offsets, Xin, Wg, Wu, Wd, G, U, H, Yout,
               (char*)ws, (char*)ws + need, ws_bytes - need};
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
  const size_t need = bwd_base(shape, n_groups, n_rows, offsets == nullptr);
  if (ws_bytes < need) {
    set_error("moe_expert_bwd: workspace of %zu bytes, need %zu", ws_bytes, need);
    return MOE_EWS;
  }
  char* dG = (char*)ws + plan_size_for(n_groups, n_rows, offsets == nullptr);
  BwdArgs a = {shape->d, shape->d_ff, n_groups, n_rows, offsets, Xin, Wg, Wu, Wd, G, U, H, dYin, dXin,
               active_ids, n_active, dWg_c, dWu_c, dWd_c, (char*)ws, dG,
               dG + grad_size_for(shape, n_groups, n_rows, offsets == nullptr), (char*)ws + need, ws_bytes - need};
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
  FwdArgs a = {shape->d, shape->d_ff, n_groups, n_rows, offsets, X, Wg, Wu, Wd, G, U, H, Yout, (char*)ws, nullptr, 0};
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
  char* dG = (char*)ws + plan_size_for(n_groups, n_rows, false);
  BwdArgs a = {shape->d, shape->d_ff, n_groups, n_rows, offsets, Xp, Wg, Wu, Wd, G, U, H, dYp, dXp,
               active_ids, n_active, dWg_c, dWu_c, dWd_c, (char*)ws, dG, dG + grad_size_for(shape, n_groups, n_rows, false), nullptr, 0};
  a.dY = dY; a.src_of = src_of; a.row_w = topk_w; a.src_div = shape->k; a.src_rows = shape->T;
  switch (pick_path(shape)) {
    case PATH_F32: expert_bwd_impl<PATH_F32>(a, (hipStream_t)stream); break;
    case PATH_BF16_TAIL: expert_bwd_impl<PATH_BF16_TAIL>(a, (hipStream_t)stream); break;
    default: expert_bwd_impl<PATH_BF16>(a, (hipStream_t)stream); break;
  }
  return launch_status("moe_expert_bwd_gather");
}

// ------------------------------------------------------------------------------------ router
namespace moe {

static int router_path(const moe_shape_t* s) {
  if (s->dtype == MOE_F32) return PATH_F32;
  return s->d % 64 == 0 ? PATH_BF16 : PATH_BF16_TAIL;
}
static size_t router_parts(const moe_shape_t* s, bool bwd) {
  switch (router_path(s)) {
    case PATH_F32: return router_part_bytes<PATH_F32>(s, bwd);
    case PATH_BF16_TAIL: return router_part_bytes<PATH_BF16_TAIL>(s, bwd);
    default: return router_part_bytes<PATH_BF16>(s, bwd);
  }
}
static size_t router_fwd_base(const moe_shape_t* shape) {
  const int Ep = padded_experts(shape);
  if (Ep == shape->E) return 256;
  return align_up((size_t)shape->d * Ep * elem_size(shape->dtype), 256) + align_up((size_t)shape->T * Ep * 4, 256);
}
static size_t router_bwd_base(const moe_shape_t* shape) {
  const int Ep = padded_experts(shape);
  const size_t es = elem_size(shape->dtype);
  return align_up((size_t)shape->T * Ep * es, 256) + 2 * align_up((size_t)shape->d * Ep * es, 256);
}

}  // namespace moe

extern "C" size_t moe_router_fwd_workspace_bytes(const moe_shape_t* shape) {
  using namespace moe;
  if (!shape || shape->E < 1 || shape->d < 1 || shape->T < 0) return 0;
  return router_fwd_base(shape) + router_parts(shape, false);
}

extern "C" size_t moe_router_bwd_workspace_bytes(const moe_shape_t* shape) {
  using namespace moe;
  if (!shape || shape->E < 1 || shape->d < 1 || shape->T < 0) return 0;
  return router_bwd_base(shape) + router_parts(shape, true);
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
  const size_t need = router_fwd_base(shape);
  if (ws_bytes < need) {
    set_error("moe_router_fwd: workspace of %zu bytes, need %zu", ws_bytes, need);
    return MOE_EWS;
  }
  switch (router_path(shape)) {
    case PATH_F32: router_fwd_impl<PATH_F32>(shape, X, Wr, logits, (char*)ws, (char*)ws + need, ws_bytes - need, (hipStream_t)stream); break;
    case PATH_BF16_TAIL: router_fwd_impl<PATH_BF16_TAIL>(shape, X, Wr, logits, (char*)ws, (char*)ws + need, ws_bytes - need, (hipStream_t)stream); break;
    default: router_fwd_impl<PATH_BF16>(shape, X, Wr, logits, (char*)ws, (char*)ws + need, ws_bytes - need, (hipStream_t)stream); break;
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
  const size_t need = router_bwd_base(shape);
  if (ws_bytes < need) {
    set_error("moe_router_bwd: workspace of %zu bytes, need %zu", ws_bytes, need);
    return MOE_EWS;
  }
  if (shape->T == 0) {  // no tokens: the weight gradient is zero, there is no dX
    if (shape->dtype == MOE_F32) recolumn<float, float>("router_pad", nullptr, dWr, shape->d, 0, shape->E, (hipStream_t)stream);
    else recolumn<bf16_t, bf16_t>("router_pad", nullptr, dWr, shape->d, 0, shape->E, (hipStream_t)stream);
    return launch_status("moe_router_bwd");
  }
  switch (router_path(shape)) {
    case PATH_F32: router_bwd_impl<PATH_F32>(shape, X, Wr, dlogits, dWr, dX, accumulate != 0, (char*)ws, (char*)ws + need, ws_bytes - need, (hipStream_t)stream); break;
    case PATH_BF16_TAIL: router_bwd_impl<PATH_BF16_TAIL>(shape, X, Wr, dlogits, dWr, dX, accumulate != 0, (char*)ws, (char*)ws + need, ws_bytes - need, (hipStream_t)stream); break;
    default: router_bwd_impl<PATH_BF16>(shape, X, Wr, dlogits, dWr, dX, accumulate != 0, (char*)ws, (char*)ws + need, ws_bytes - need, (hipStream_t)stream); break;
  }
  return launch_status("moe_router_bwd");
}
