#include "mjh_step_reg.h"

namespace mjh {

StepRegKernel step_reg_kernel_large(RegShape r, bool rk4) {
  if (r.nb != 28) return nullptr;
  if (r.team == 32) return rk4 ? mjh_step_reg_kernel<32, 28, true> : mjh_step_reg_kernel<32, 28, false>;
  if (r.team == 64) return rk4 ? mjh_step_reg_kernel<64, 28, true> : mjh_step_reg_kernel<64, 28, false>;
  return nullptr;
}

}  // namespace mjh
