#include "mjh_step_reg.h"

namespace mjh {

StepRegKernel step_reg_kernel_small(RegShape r, bool rk4) {
  if (r.nb != 16) return nullptr;
  if (r.team == 16) return rk4 ? mjh_step_reg_kernel<16, 16, true> : mjh_step_reg_kernel<16, 16, false>;
  if (r.team == 32) return rk4 ? mjh_step_reg_kernel<32, 16, true> : mjh_step_reg_kernel<32, 16, false>;
  return nullptr;
}

}  // namespace mjh
