// Expert and router GEMMs: fp32.
#include "expert_impl.h"

namespace moe {
template void expert_fwd_impl<PATH_F32>(const FwdArgs*, const FwdArgs*, hipStream_t);
template void expert_bwd_impl<PATH_F32>(const BwdArgs*, const BwdArgs*, hipStream_t);
template void router_fwd_impl<PATH_F32>(const moe_shape_t*, const void*, const void*, float*, char*, char*, size_t, hipStream_t);
template void router_bwd_impl<PATH_F32>(const moe_shape_t*, const void*, const void*, const float*, void*, void*, bool, char*, char*,
                                     size_t, hipStream_t);
}  // namespace moe

MOE_TRACE_DEFINE_READER(moe_trace_read_f32)
