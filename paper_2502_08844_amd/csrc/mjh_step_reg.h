// The step kernels whose solves run in registers, one instantiation per team size T, padded
// row length NB and integrator (RK: fourth-order Runge-Kutta).  They are spread over several
// source files so that the build compiles them in parallel.
#pragma once
#include "mjh_worlds.h"

namespace mjh {

// The team a thread works for, or -1 when its wavefront has no world.  Matrix instructions and
// lane swaps take every lane of the wavefront, so lanes past the last world join that world's
// team: they compute and write the same values (its LDS and outputs included), in step with it.
template <int T>
__device__ __forceinline__ int team_of(int nw) {
  if ((int)(threadIdx.x & ~63u) / T >= nw) return -1;
  return min((int)threadIdx.x / T, nw - 1);
}

// Four waves per SIMD for rows of up to 20 entries (the quadruped's residency), two for longer
// rows, whose worlds fill a CU's LDS at that count.
template <int T, int NB, bool RK>
__global__ void __launch_bounds__(kMaxBlock, NB > 20 ? 2 : 4)
mjh_step_reg_kernel(const DevGroup* __restrict__ groups, const DevTask* __restrict__ tasks,
                    int nstep) {
  extern __shared__ float lds[];
  const DevTask tk = tasks[blockIdx.x];
  const DevGroup& G = groups[tk.group];
  const int team = team_of<T>(tk.nw);
  if (team < 0) return;
  float* W = lds + (size_t)team * G.m.lds_words;
  run_worlds<RK, false, T, NB>(G, W, tk.w0 + team, nstep, threadIdx.x & (T - 1), T, nullptr);
}

using StepRegKernel = void (*)(const DevGroup*, const DevTask*, int);
// the instantiation for a shape, or nullptr
StepRegKernel step_reg_kernel_small(RegShape r, bool rk4);   // rows of 16
StepRegKernel step_reg_kernel_medium(RegShape r, bool rk4);  // rows of 20
StepRegKernel step_reg_kernel_large(RegShape r, bool rk4);   // rows of 28
StepRegKernel step_mix_kernel();                             // several shapes

}  // namespace mjh
