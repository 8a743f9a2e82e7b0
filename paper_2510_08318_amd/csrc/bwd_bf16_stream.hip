// bf16-I/O backward with dq and dv stored non-temporally (see bwd_bf16.hip).
#include "bwd_bf16.h"

namespace linattn {

hipError_t launch_bwd_bf16_stream(const BwdArgs& a, const Plan& p, hipStream_t s) { return run_bwd<true>(a, p, s); }

}  // namespace linattn
