// Expert GEMMs: bf16, calls of few rows.
#include "expert_impl.h"

namespace moe {
template void expert_fwd_impl<PATH_BF16_SMALL>(const FwdArgs*, const FwdArgs*, hipStream_t);
template void expert_bwd_impl<PATH_BF16_SMALL>(const BwdArgs*, const BwdArgs*, hipStream_t);
}  // namespace moe

MOE_TRACE_DEFINE_READER(moe_trace_read_small)
