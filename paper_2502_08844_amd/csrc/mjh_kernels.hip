// Kernels of the batched physics step.
//
// mjh_step_kernel: one work-group per task (a run of worlds of one model); inside it a
// team of T lanes (16, 32 or 64, chosen per model) owns one world.  The world's state
// is loaded from HBM into LDS once, advanced `nstep` steps on chip (only the controls
// are read per step), and written back once.  The same kernel serves a batch of
// several models: each work-group reads its task and its group's model descriptor.
// No work-group barrier is used, so teams beyond a task's world count simply exit.
#include <hip/hip_runtime.h>

#include "mjh_worlds.h"

namespace mjh {

template <bool RK, bool CONE>
__global__ void __launch_bounds__(kMaxBlock, 4)
mjh_step_kernel(const DevGroup* __restrict__ groups, const DevTask* __restrict__ tasks,
                int nstep, int tab_words) {
  extern __shared__ float lds[];
  const DevTask tk = tasks[blockIdx.x];
  const DevGroup& G = groups[tk.group];
  load_pair_table(G.m, (unsigned*)lds);
  const int T = G.team;
  const int team = threadIdx.x / T;
  if (team >= tk.nw) return;
  float* W = lds + tab_words + (size_t)team * G.m.lds_words;
  const int lane = threadIdx.x - team * T;
  const int world = tk.w0 + team;
  run_worlds<RK, CONE>(G, W, world, nstep, lane, T, (const unsigned char*)lds);
}

// LDS: the pair table, then `ap_words` holding each team's previous action and, with
// randomisation, its parameter record (nu + ndr words a team), then the worlds' working
// sets at the usual stride.
template <bool RK, bool DR>
__global__ void __launch_bounds__(kMaxBlock, 4)
mjh_env_kernel(const DevGroup* __restrict__ groups, const DevTask* __restrict__ tasks,
               EnvArgs E, int tab_words, int ap_words) {
  extern __shared__ float lds[];
  const DevTask tk = tasks[blockIdx.x];
  const DevGroup& G = groups[tk.group];
  load_pair_table(G.m, (unsigned*)lds);
  const int T = G.team;
  const int team = threadIdx.x / T;
  if (team >= tk.nw) return;
  float* ap = lds + tab_words + team * (G.m.nu + E.ndr);
  float* W = lds + tab_words + ap_words + (size_t)team * G.m.lds_words;
  env_worlds<RK>(G, E, W, ap, DR ? ap + G.m.nu : nullptr, tk.w0 + team, threadIdx.x - team * T, T,
             (const unsigned char*)lds);
}

// Translational inverse weight of every body at qpos0:
//   w(b) = trace(J_com(b) M^-1 J_com(b)^T) / 3,
// and (M^-1)_kk of every dof k, one work-group of 64 lanes evaluating the model once.
__global__ void __launch_bounds__(64) mjh_invweight_kernel(DevModel m, int tab_words) {
  extern __shared__ float lds[];
  load_pair_table(m, (unsigned*)lds);
  float* W = lds + tab_words;
  const Team t{(int)threadIdx.x, 64, (const unsigned char*)lds};
  world_init(m, W, t);
  for (int i = t.lane; i < m.nq; i += t.T) W[m.o_qpos + i] = m.qpos0[i];
  t.sync();
  forward_sweep(m, W, t);
  backward_and_mass(m, W, t);
  ltdl_factor(m, W, t);
  // scratch: the smooth-force and unconstrained-acceleration vectors, unused here (the
  // Newton vectors share words with the poses read below, and the sweep scratch with
  // the factor in H)
  float* jr = W + m.o_frc;
  float* x = W + m.o_a0;
  const float* cdof = W + m.o_cdof;
  for (int b = 0; b < m.nbody; b++) {
    if (b == 0) {
      if (t.lane == 0) m.body_invweight[0] = 0.f;
      continue;
    }
    float c[3];
    mv3(W + m.o_xmat + 9 * b, m.body_ipos + 3 * b, c);
    for (int k = 0; k < 3; k++) c[k] += W[m.o_xpos + 3 * b + k];
    float tr = 0.f;
    for (int r = 0; r < 3; r++) {
      for (int i = t.lane; i < m.nv; i += t.T) {
        float v = 0.f;
        if (m.body_dofmask[b] >> i & 1ull) {
          float wx[3];
          cross3(cdof + 6 * i, c, wx);
          v = cdof[6 * i + 3 + r] + wx[r];
        }
        jr[i] = v;
      }
      t.sync();
      ltdl_solve(m, W, t, jr, x);
      float part = 0.f;
      for (int i = t.lane; i < m.nv; i += t.T) part += jr[i] * x[i];
      tr += t.sum(part);
      t.sync();
    }
    if (t.lane == 0) m.body_invweight[b] = tr / 3.f;
  }
  // joint-limit and friction-loss rows: (M^-1)_kk of every dof
  for (int k = 0; k < m.nv; k++) {
    for (int i = t.lane; i < m.nv; i += t.T) jr[i] = i == k ? 1.f : 0.f;
    t.sync();
    ltdl_solve(m, W, t, jr, x);
    if (t.lane == 0) m.dof_invweight[k] = x[k];
    t.sync();
  }
}

// ------------------------------------------------------------- host-side launchers
hipError_t launch_step(const DevGroup* groups, const DevTask* tasks, int ntask, int nstep,
                       int block, size_t lds_bytes, int tab_words, bool rk4, bool cone,
                       RegShape reg, hipStream_t stream) {
  if (ntask <= 0) return hipSuccess;
  if (reg.nb)  // (these need no pair table)
    return launch_step_reg(groups, tasks, ntask, nstep, block,
                           lds_bytes - (size_t)tab_words * sizeof(float), rk4, reg, stream);
  if (cone)
    hipLaunchKernelGGL((mjh_step_kernel<true, true>), dim3(ntask), dim3(block), lds_bytes,
                       stream, groups, tasks, nstep, tab_words);
  else if (rk4)
    hipLaunchKernelGGL((mjh_step_kernel<true, false>), dim3(ntask), dim3(block), lds_bytes,
                       stream, groups, tasks, nstep, tab_words);
  else
    hipLaunchKernelGGL((mjh_step_kernel<false, false>), dim3(ntask), dim3(block), lds_bytes,
                       stream, groups, tasks, nstep, tab_words);
  return hipGetLastError();
}

hipError_t set_step_lds_limit(size_t bytes) {
  hipError_t e = hipFuncSetAttribute((const void*)mjh_step_kernel<false, false>,
                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
  if (e == hipSuccess)
    e = hipFuncSetAttribute((const void*)mjh_step_kernel<true, false>,
                            hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
  if (e != hipSuccess) return e;
  return hipFuncSetAttribute((const void*)mjh_step_kernel<true, true>,
                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
}

hipError_t launch_env(const DevGroup* groups, const DevTask* tasks, int ntask, const EnvArgs& E,
                      int block, size_t lds_bytes, int tab_words, int ap_words, bool rk4,
                      RegShape reg, hipStream_t stream) {
  if (ntask <= 0) return hipSuccess;
  if (reg.nb && env_reg_shape(reg, rk4))
    return launch_env_reg(groups, tasks, ntask, E, block, lds_bytes, tab_words, ap_words, stream);
  // one instantiation per case, so that the plain env step carries none of the
  // randomisation's live values; per-world records come with the Euler step only
  if (rk4)
    hipLaunchKernelGGL((mjh_env_kernel<true, false>), dim3(ntask), dim3(block), lds_bytes, stream,
                       groups, tasks, E, tab_words, ap_words);
  else if (E.dr)
    hipLaunchKernelGGL((mjh_env_kernel<false, true>), dim3(ntask), dim3(block), lds_bytes, stream,
                       groups, tasks, E, tab_words, ap_words);
  else
    hipLaunchKernelGGL((mjh_env_kernel<false, false>), dim3(ntask), dim3(block), lds_bytes, stream,
                       groups, tasks, E, tab_words, ap_words);
  return hipGetLastError();
}

hipError_t set_env_lds_limit(size_t bytes) {
  hipError_t e = hipFuncSetAttribute((const void*)mjh_env_kernel<false, false>,
                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
  if (e == hipSuccess)
    e = hipFuncSetAttribute((const void*)mjh_env_kernel<false, true>,
                            hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
  if (e != hipSuccess) return e;
  return hipFuncSetAttribute((const void*)mjh_env_kernel<true, false>,
                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
}

hipError_t launch_invweight(const DevModel& m, hipStream_t stream) {
  const int tab = table_words(m);
  const size_t lds = (size_t)(tab + m.lds_words) * sizeof(float);
  hipError_t e = hipFuncSetAttribute((const void*)mjh_invweight_kernel,
                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(mjh_invweight_kernel, dim3(1), dim3(64), lds, stream, m, tab);
  return hipGetLastError();
}


}  // namespace mjh
