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
// For calls that bring no plan (moe_route_dispatch_plan builds one in its own kernels).
// offsets == NULL (a shared call without rows, whose active_ids and n_active are all there is to write): no group has rows.
__global__ __launch_bounds__(1024) void plan_kernel(const int32_t* __restrict__ offsets, int n_groups, int BM, Plan pl,
                                                    int32_t* active_ids, int32_t* n_active) {
  const int e = threadIdx.x;
  int c = 0, st = 0;
  if (e < n_groups && offsets) {
    st = offsets[e];
    c = max(offsets[e + 1] - st, 0);
  }
  build_plan(c, st, n_groups, BM, pl, active_ids, n_active);
}

void launch_plan(const int32_t* offsets, int n_groups, int BM, const Plan& pl, int32_t* active_ids, int32_t* n_active, hipStream_t st) {
  ProfScope prof("plan_kernel", st);
  hipLaunchKernelGGL(plan_kernel, dim3(1), dim3(1024), 0, st, offsets, n_groups, BM, pl, active_ids, n_active);
}

// one translation unit each
#define MOE_CORES(PATH)                                                                                                 \
  extern template void expert_fwd_impl<PATH>(const FwdArgs*, const FwdArgs*, hipStream_t);                                            \
  extern template void expert_bwd_impl<PATH>(const BwdArgs*, const BwdArgs*, hipStream_t);                                            \
  extern template void router_fwd_impl<PATH>(const moe_shape_t*, const void*, const void*, float*, char*, char*,      \
                                             size_t, hipStream_t);                                                     \
  extern template void router_bwd_impl<PATH>(const moe_shape_t*, const void*, const void*, const float*, void*, void*, \
                                             bool, char*, char*, size_t, hipStream_t);
MOE_CORES(PATH_F32)
MOE_CORES(PATH_BF16_TAIL)
MOE_CORES(PATH_BF16)
extern template void expert_fwd_impl<PATH_BF16_SMALL>(const FwdArgs*, const FwdArgs*, hipStream_t);
extern template void expert_bwd_impl<PATH_BF16_SMALL>(const BwdArgs*, const BwdArgs*, hipStream_t);

static int full_path(const moe_shape_t* s) {
  if (s->dtype == MOE_F32) return PATH_F32;
  return (s->d % 64 == 0 && s->d_ff % 64 == 0) ? PATH_BF16 : PATH_BF16_TAIL;
}
static bool small_tiles(const moe_shape_t* s, int n_groups, int n_rows) { return small_tiles(s->dtype, n_groups, n_rows, s->d, s->d_ff); }
static int pick_path(const moe_shape_t* s, int n_groups, int n_rows) { return small_tiles(s, n_groups, n_rows) ? (int)PATH_BF16_SMALL : full_path(s); }

static void run_fwd(int path, const FwdArgs* routed, const FwdArgs* shared, hipStream_t st) {
  switch (path) {
    case PATH_F32: expert_fwd_impl<PATH_F32>(routed, shared, st); break;
    case PATH_BF16_TAIL: expert_fwd_impl<PATH_BF16_TAIL>(routed, shared, st); break;
    case PATH_BF16_SMALL: expert_fwd_impl<PATH_BF16_SMALL>(routed, shared, st); break;
    default: expert_fwd_impl<PATH_BF16>(routed, shared, st); break;
  }
}
static void run_bwd(int path, const BwdArgs* routed, const BwdArgs* shared, hipStream_t st) {
  switch (path) {
    case PATH_F32: expert_bwd_impl<PATH_F32>(routed, shared, st); break;
    case PATH_BF16_TAIL: expert_bwd_impl<PATH_BF16_TAIL>(routed, shared, st); break;
    case PATH_BF16_SMALL: expert_bwd_impl<PATH_BF16_SMALL>(routed, shared, st); break;
    default: expert_bwd_impl<PATH_BF16>(routed, shared, st); break;
  }
}

static size_t plan_size_for(int n_groups, int n_rows, bool shared) {
  // Sized for the smallest row tile of any path, so the query does not depend on the path taken.  A shared call with rows
  // has no plan; it asks for the space all the same, so that it refuses what it always refused.
  const int bound = shared ? n_groups * (n_rows / 64 + 2) : plan_cap(n_groups, n_rows);
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
  if (s->d <= 0 || s->d_ff <= 0) return 0;  // a shape that the calls refuse: there are no products to divide
  if (s->dtype == MOE_F32) return expert_part_bytes<PATH_F32>(s->d, s->d_ff, n_groups, n_rows, bwd);
  // (shared rows may be few where the routed ones beside them are not)
  const size_t full = full_path(s) == PATH_BF16 ? expert_part_bytes<PATH_BF16>(s->d, s->d_ff, n_groups, n_rows, bwd)
                                                : expert_part_bytes<PATH_BF16_TAIL>(s->d, s->d_ff, n_groups, n_rows, bwd);
  return few_rows(s->dtype, n_rows, s->d) ? std::max(full, expert_part_bytes<PATH_BF16_SMALL>(s->d, s->d_ff, n_groups, n_rows, bwd)) : full;
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
  run_fwd(pick_path(shape, n_groups, n_rows), offsets ? &a : nullptr, offsets ? nullptr : &a, (hipStream_t)stream);
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
  run_bwd(pick_path(shape, n_groups, n_rows), offsets ? &a : nullptr, offsets ? nullptr : &a, (hipStream_t)stream);
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
  run_fwd(pick_path(shape, n_groups, n_rows), &a, nullptr, (hipStream_t)stream);
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
  run_bwd(pick_path(shape, n_groups, n_rows), &a, nullptr, (hipStream_t)stream);
  return launch_status("moe_expert_bwd_gather");
}

// Routed and shared experts of one layer: see include/moe_hip.h.
namespace moe {

// the checks of the calls for one set of experts, and their argument block; 0, or the error code
static int check_set(const moe_shape_t* shape, const moe_expert_set_t* x, bool routed, bool bwd, const char* who, moe_shape_t& s,
                     size_t& need) {
  s = *shape;
  s.d_ff = x->d_ff;
  int rc = check_expert_args(&s, x->n_groups, x->n_rows, who);
  if (rc) return rc;
  const bool gather = routed && x->src_of != nullptr;
  bool null = !x->Wg || !x->Wd || !x->ws || (routed ? !x->offsets : x->offsets != nullptr || x->src_of != nullptr);
  if (x->n_rows > 0) null = null || !x->Xin || !x->G || (x->Wu && !x->U) || !x->H;
  if (bwd) {
    null = null || !x->active_ids || !x->n_active || !x->dWg_c || (x->Wu && !x->dWu_c) || !x->dWd_c;
    if (x->n_rows > 0) null = null || !x->dYin || !x->dXin || (gather && (!x->dY || !x->row_w));
  } else if (x->n_rows > 0) {
    null = null || !x->Yout;
  }
  if (null) {
    set_error("%s: null pointer (offsets are the routed experts' alone)", who);
    return MOE_EINVAL;
  }
  const void* fwd_ptrs[] = {x->Xin, x->Wg, x->Wu, x->Wd, x->G, x->U, x->H, x->ws, bwd ? nullptr : x->Yout};
  const void* bwd_ptrs[] = {x->dYin, x->dY, x->dXin, x->dWg_c, x->dWu_c, x->dWd_c};
  bool aligned = true;
  for (const void* p : fwd_ptrs) aligned = aligned && aligned16(p);
  if (bwd)
    for (const void* p : bwd_ptrs) aligned = aligned && aligned16(p);
  if (!aligned || !aligned16(x->plan)) {
    set_error("%s: every tensor must be 16-byte aligned", who);
    return MOE_EINVAL;
  }
  if ((gather || x->plan) && (!routed || x->n_groups != shape->E || x->n_rows != shape->T * shape->k)) {
    set_error("%s: rows read in place, and those of a plan, are those of the shape: E groups, T*k rows", who);
    return MOE_EINVAL;
  }
  if (gather && (int64_t)shape->T * shape->d * (int64_t)elem_size(shape->dtype) >= ((int64_t)1 << 32) - 4096) {
    set_error("%s: rows read in place must take less than 4 GiB (32-bit byte offsets)", who);
    return MOE_EINVAL;
  }
  need = bwd ? bwd_base(&s, x->n_groups, x->n_rows, !routed) : fwd_base(&s, x->n_groups, x->n_rows, !routed);
  if (x->ws_bytes < need) {
    set_error("%s: workspace of %zu bytes, need %zu", who, x->ws_bytes, need);
    return MOE_EWS;
  }
  return MOE_OK;
}
static int check_sets(const moe_shape_t* shape, const moe_expert_set_t* routed, const moe_expert_set_t* shared, bool bwd, const char* who,
                      moe_shape_t (&s)[2], size_t (&need)[2]) {
  if (!shape || !routed) {
    set_error("%s: null pointer", who);
    return MOE_EINVAL;
  }
  const int rc = check_set(shape, routed, true, bwd, who, s[0], need[0]);
  return rc || !shared ? rc : check_set(shape, shared, false, bwd, who, s[1], need[1]);
}
// Common launches need the same kernels for both: one activation, and cores that take both widths.  Anything else (no
// rows on one side, rows beyond the tile cores' offsets) goes one after the other, as the two calls would.  Where only one
// width has a K tail both sets run on the cores that mask it: the masks cost less than launches apart.  (Apart and together,
// us a pass, routed width / shared: 1408 / 4 of 1400, 16 tokens, forward 130 and 113; 1408 / 1000, T = 2048, d = 1024, training 392 and
// 313; 1368 / 2 of 2048, T = 4096 768 and 682; 1408 / 2 of 712, T = 4096, d = 2048 1647 and 1607; 6400 / 3208, T = 8192, d = 4096 8717
// and 8626.)
// The cores of common launches: the small ones if both sets' products are short; PATH_BF16_TAIL where either width needs it (it takes what
// PATH_BF16 takes, with the same results).
static int common_path(const moe_shape_t (&s)[2], const moe_expert_set_t* routed, const moe_expert_set_t* shared) {
  if (small_tiles(&s[0], routed->n_groups, routed->n_rows) && short_product((int64_t)shared->n_groups * shared->n_rows, s[1].d, s[1].d_ff))
    return PATH_BF16_SMALL;
  return std::min(full_path(&s[0]), full_path(&s[1]));
}
static bool can_share(const moe_shape_t (&s)[2], const moe_expert_set_t* routed, const moe_expert_set_t* shared) {
  if (!shared) return false;
  const int64_t ld = std::max({s[0].d, s[0].d_ff, s[1].d_ff});
  return routed->n_rows > 0 && shared->n_rows > 0 && !routed->Wu == !shared->Wu && !wide_rows(ld, elem_size(s[0].dtype));
}

}  // namespace moe

extern "C" size_t moe_expert_plan_bytes(const moe_shape_t* shape) {
  using namespace moe;
  if (!shape || shape->E < 1 || shape->T < 0 || shape->k < 1) return 0;
  return align_up(plan_bytes(shape->E, plan_cap(shape->E, shape->T * shape->k)), 256);
}

extern "C" int moe_experts_fwd(const moe_shape_t* shape, const moe_expert_set_t* routed, const moe_expert_set_t* shared, void* stream) {
  using namespace moe;
  moe_shape_t s[2];
  size_t need[2];
  const int rc = check_sets(shape, routed, shared, false, "moe_experts_fwd", s, need);
  if (rc) return rc;
  const moe_expert_set_t* sets[2] = {routed, shared};
  FwdArgs a[2];
  for (int i = 0; i < (shared ? 2 : 1); i++) {
    const moe_expert_set_t* x = sets[i];
    a[i] = {shape->d, x->d_ff, x->n_groups, x->n_rows, x->offsets, x->Xin, x->Wg, x->Wu, x->Wd, x->G, x->U, x->H, x->Yout,
            (char*)x->ws, (char*)x->ws + need[i], x->ws_bytes - need[i]};
    a[i].plan = x->plan;
    if (x->src_of) { a[i].src_of = x->src_of; a[i].src_div = shape->k; a[i].src_rows = shape->T; }
  }
  const int p0 = pick_path(&s[0], routed->n_groups, routed->n_rows), p1 = shared ? pick_path(&s[1], shared->n_groups, shared->n_rows) : p0;
  hipStream_t st = (hipStream_t)stream;
  if (can_share(s, routed, shared)) {
    run_fwd(common_path(s, routed, shared), &a[0], &a[1], st);
  } else {
    if (routed->n_rows > 0) run_fwd(p0, &a[0], nullptr, st);
    if (shared && shared->n_rows > 0) run_fwd(p1, nullptr, &a[1], st);
  }
  return launch_status("moe_experts_fwd");
}

extern "C" int moe_experts_bwd(const moe_shape_t* shape, const moe_expert_set_t* routed, const moe_expert_set_t* shared, void* stream) {
  using namespace moe;
  moe_shape_t s[2];
  size_t need[2];
  const int rc = check_sets(shape, routed, shared, true, "moe_experts_bwd", s, need);
  if (rc) return rc;
  const moe_expert_set_t* sets[2] = {routed, shared};
  BwdArgs a[2];
  for (int i = 0; i < (shared ? 2 : 1); i++) {
    const moe_expert_set_t* x = sets[i];
    char* dG = (char*)x->ws + plan_size_for(x->n_groups, x->n_rows, i == 1);
    a[i] = {shape->d, x->d_ff, x->n_groups, x->n_rows, x->offsets, x->Xin, x->Wg, x->Wu, x->Wd, x->G, x->U, x->H, x->dYin, x->dXin,
            x->active_ids, x->n_active, x->dWg_c, x->dWu_c, x->dWd_c, (char*)x->ws, dG,
            dG + grad_size_for(&s[i], x->n_groups, x->n_rows, i == 1), (char*)x->ws + need[i], x->ws_bytes - need[i]};
    a[i].plan = x->plan;
    if (x->src_of) {
      a[i].dY = x->dY; a[i].src_of = x->src_of; a[i].row_w = x->row_w; a[i].src_div = shape->k; a[i].src_rows = shape->T;
    }
  }
  const int p0 = pick_path(&s[0], routed->n_groups, routed->n_rows), p1 = shared ? pick_path(&s[1], shared->n_groups, shared->n_rows) : p0;
  hipStream_t st = (hipStream_t)stream;
  if (can_share(s, routed, shared)) {
    run_bwd(common_path(s, routed, shared), &a[0], &a[1], st);
  } else {
    run_bwd(p0, &a[0], nullptr, st);
    if (shared) run_bwd(p1, nullptr, &a[1], st);
  }
  return launch_status("moe_experts_bwd");
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
