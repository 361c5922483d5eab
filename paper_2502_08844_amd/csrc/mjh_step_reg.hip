// Launchers of the register-resident step and env kernels, and the kernels for batches of
// several shapes and for the env step.
#include "mjh_step_reg.h"

namespace mjh {

// A batch whose groups have different shapes: each work-group takes its group's.
__global__ void __launch_bounds__(kMaxBlock, 2)
mjh_step_mix_kernel(const DevGroup* __restrict__ groups, const DevTask* __restrict__ tasks,
                    int nstep) {
  extern __shared__ float lds[];
  const DevTask tk = tasks[blockIdx.x];
  const DevGroup& G = groups[tk.group];
  const int T = G.team;
  const int team = T == 64 ? team_of<64>(tk.nw) : T == 32 ? team_of<32>(tk.nw) : team_of<16>(tk.nw);
  if (team < 0) return;
  float* W = lds + (size_t)team * G.m.lds_words;
  const int lane = threadIdx.x & (T - 1), world = tk.w0 + team;
  if (T == 64) run_worlds<false, false, 64, 28>(G, W, world, nstep, lane, 64, nullptr);
  else if (T == 32) run_worlds<false, false, 32, 20>(G, W, world, nstep, lane, 32, nullptr);
  else run_worlds<false, false, 16, 16>(G, W, world, nstep, lane, 16, nullptr);
}

// The env step of 32-lane teams with rows of 20 (a free root and 11 to 14 joints); the LDS
// layout is mjh_env_kernel's.
template <bool DR>
__global__ void __launch_bounds__(kMaxBlock, 4)
mjh_env_reg_kernel(const DevGroup* __restrict__ groups, const DevTask* __restrict__ tasks,
                   EnvArgs E, int tab_words, int ap_words) {
  extern __shared__ float lds[];
  const DevTask tk = tasks[blockIdx.x];
  const DevGroup& G = groups[tk.group];
  const int team = team_of<32>(tk.nw);
  if (team < 0) return;
  float* ap = lds + tab_words + team * (G.m.nu + E.ndr);
  float* W = lds + tab_words + ap_words + (size_t)team * G.m.lds_words;
  env_worlds<false, 32, 20>(G, E, W, ap, DR ? ap + G.m.nu : nullptr, tk.w0 + team,
                            threadIdx.x & 31, 32, nullptr);
}

static StepRegKernel step_kernel_for(RegShape r, bool rk4) {
  if (r.team == 0) return rk4 ? nullptr : mjh_step_mix_kernel;
  if (StepRegKernel k = step_reg_kernel_small(r, rk4)) return k;
  if (StepRegKernel k = step_reg_kernel_medium(r, rk4)) return k;
  return step_reg_kernel_large(r, rk4);
}

hipError_t launch_step_reg(const DevGroup* groups, const DevTask* tasks, int ntask, int nstep,
                           int block, size_t lds_bytes, bool rk4, RegShape reg,
                           hipStream_t stream) {
  const StepRegKernel k = step_kernel_for(reg, rk4);
  if (!k) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k, dim3(ntask), dim3(block), lds_bytes, stream, groups, tasks, nstep);
  return hipGetLastError();
}

hipError_t launch_env_reg(const DevGroup* groups, const DevTask* tasks, int ntask,
                          const EnvArgs& E, int block, size_t lds_bytes, int tab_words,
                          int ap_words, hipStream_t stream) {
  if (E.dr)
    hipLaunchKernelGGL((mjh_env_reg_kernel<true>), dim3(ntask), dim3(block), lds_bytes, stream,
                       groups, tasks, E, tab_words, ap_words);
  else
    hipLaunchKernelGGL((mjh_env_reg_kernel<false>), dim3(ntask), dim3(block), lds_bytes, stream,
                       groups, tasks, E, tab_words, ap_words);
  return hipGetLastError();
}

hipError_t allow_env_reg_lds(bool dr, size_t bytes) {
  return hipFuncSetAttribute(
      dr ? (const void*)mjh_env_reg_kernel<true> : (const void*)mjh_env_reg_kernel<false>,
      hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
}

hipError_t allow_step_reg_lds(RegShape reg, bool rk4, size_t bytes) {
  const StepRegKernel k = step_kernel_for(reg, rk4);
  if (!k) return hipErrorInvalidValue;
  return hipFuncSetAttribute((const void*)k, hipFuncAttributeMaxDynamicSharedMemorySize,
                             (int)bytes);
}

}  // namespace mjh
