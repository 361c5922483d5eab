#include "mjh_adjoint_dev.h"

namespace mjh {

RolloutKernels rollout_kernels_64_20() {
  RolloutKernels k;
  k.fwd = rollout_fwd_kernel<64, 20>;
  k.bwd = rollout_bwd_kernel<64, 20>;
  return k;
}

}  // namespace mjh
