#include "mjh_adjoint_dev.h"

namespace mjh {

RolloutKernels rollout_kernels_64_28() {
  RolloutKernels k;
  k.fwd = rollout_fwd_kernel<64, 28>;
  k.bwd = rollout_bwd_kernel<64, 28>;
  return k;
}

}  // namespace mjh
