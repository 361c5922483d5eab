#include "mjh_step_reg.h"

namespace mjh {

StepRegKernel step_reg_kernel_medium(RegShape r, bool rk4) {
  if (r.nb != 20) return nullptr;
  if (r.team == 32) return rk4 ? mjh_step_reg_kernel<32, 20, true> : mjh_step_reg_kernel<32, 20, false>;
  if (r.team == 64) return rk4 ? mjh_step_reg_kernel<64, 20, true> : mjh_step_reg_kernel<64, 20, false>;
  return nullptr;
}

}  // namespace mjh
