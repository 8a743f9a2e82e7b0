// bf16-I/O backward with dq and dv stored through the caches, and the choice between the two forms (stream_gradients).  The form with
// non-temporal stores is a file of its own: with both in one code object, of 1.6 MB instead of 0.8, a launch starts later.  A step with dW~,
// us: 12 heads x 2000 x 128 69.1 / 68.2 in two, 12 x 32760 332.6 / 329.3.
#include "bwd_bf16.h"

namespace linattn {

hipError_t launch_bwd_bf16(const BwdArgs& a, const Plan& p, hipStream_t s) {
  return stream_gradients(p) ? launch_bwd_bf16_stream(a, p, s) : run_bwd<false>(a, p, s);
}

}  // namespace linattn
