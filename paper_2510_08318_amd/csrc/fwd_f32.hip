// fp32-arithmetic forward path, on fp32 tensors (no bf16 rounding anywhere; the 1e-5 accuracy contract) or on bf16
// tensors (LINATTN_BF16_F32MATH: bf16 storage with none of the fp16 operands of the LINATTN_BF16 path): every product is
// the sum of exact bf16 piece products on the matrix cores, see f32_split.h.
#include "kernels.h"
#include "f32_split.h"
#include "f32_state.h"
#include "f32_apply.h"

namespace linattn {
namespace {

using namespace f32;

template <typename T>
hipError_t state_any(const void* k, const void* v, const void* wk, float* partials, const Plan& p, hipStream_t s) {
  if (p.kind == kPhiRelu)
    return p.d == 128 ? run_state_pass<128, kPhiRelu, T, false>(k, v, wk, nullptr, partials, p, s)
                      : run_state_pass<64, kPhiRelu, T, false>(k, v, wk, nullptr, partials, p, s);
  return p.d == 128 ? run_state_pass<128, kPhiHedgehog, T, false>(k, v, wk, nullptr, partials, p, s)
                    : run_state_pass<64, kPhiHedgehog, T, false>(k, v, wk, nullptr, partials, p, s);
}
template <typename T>
hipError_t apply_any(const void* q, const void* wq, const float* state, void* out,
                     const void* blend_in, const float* blend_r, const Plan& p, hipStream_t s) {
  if (p.kind == kPhiRelu)      // the descriptor check has refused a blend with this map
    return p.d == 128 ? run_apply_pass<128, kPhiRelu, T, false>(q, wq, state, out, nullptr, nullptr, p, s)
                      : run_apply_pass<64, kPhiRelu, T, false>(q, wq, state, out, nullptr, nullptr, p, s);
  if (blend_in)
    return p.d == 128 ? run_apply_pass<128, kPhiHedgehog, T, true>(q, wq, state, out, blend_in, blend_r, p, s)
                      : run_apply_pass<64, kPhiHedgehog, T, true>(q, wq, state, out, blend_in, blend_r, p, s);
  return p.d == 128 ? run_apply_pass<128, kPhiHedgehog, T, false>(q, wq, state, out, nullptr, nullptr, p, s)
                    : run_apply_pass<64, kPhiHedgehog, T, false>(q, wq, state, out, nullptr, nullptr, p, s);
}

}  // namespace

hipError_t launch_state_partials_f32(const void* k, const void* v, const void* wk, float* partials,
                                     const Plan& p, hipStream_t s) {
  return p.bf16_storage ? state_any<uint16_t>(k, v, wk, partials, p, s) : state_any<float>(k, v, wk, partials, p, s);
}

hipError_t launch_apply_f32(const void* q, const void* wq, const float* state, void* out,
                            const void* blend_in, const float* blend_r, const Plan& p, hipStream_t s) {
  return p.bf16_storage ? apply_any<uint16_t>(q, wq, state, out, blend_in, blend_r, p, s)
                        : apply_any<float>(q, wq, state, out, blend_in, blend_r, p, s);
}

}  // namespace linattn
