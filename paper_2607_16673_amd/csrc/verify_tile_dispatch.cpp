// verify_tile_dispatch.cpp -- which unit of the tree-masked contraction
// (verify_tile.hip, one translation unit per head size, form of the step and
// activation type) takes a verification.
#include "kernels.hpp"
#include "sla.h"

namespace sla {

bool parallel_supported(int dk, int dv, int n, int dtype) {
  // bf16 activations: bf16 matrix cores (q and k exact in bf16, the fp32
  // operands split hi + lo); fp32 activations: fp32 matrix cores.  A draft
  // whose stage exceeds the LDS is refused at launch
  // (hipErrorInvalidConfiguration).
  return (dtype == SLA_DTYPE_BF16 || dtype == SLA_DTYPE_F32) && (dk == 64 || dk == 128 || dk == 256) &&
         dv % 16 == 0 && n >= 1 && n <= SLA_MAX_NODES;
}

template <bool GATES, bool F32>
static hipError_t launch_form(const VerifyArgs &a, hipStream_t s) {
  switch (a.dk) {
    case 64: return launch_tile<64, GATES, F32>(a, s);
    case 128: return launch_tile<128, GATES, F32>(a, s);
    case 256: return launch_tile<256, GATES, F32>(a, s);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_verify_parallel(const VerifyArgs &a, int dtype, hipStream_t s) {
  const bool gates = a.family == SLA_FAMILY_GLA;
  if (dtype == SLA_DTYPE_BF16) return gates ? launch_form<true, false>(a, s) : launch_form<false, false>(a, s);
  if (dtype == SLA_DTYPE_F32) return gates ? launch_form<true, true>(a, s) : launch_form<false, true>(a, s);
  return hipErrorInvalidConfiguration;
}

}  // namespace sla
