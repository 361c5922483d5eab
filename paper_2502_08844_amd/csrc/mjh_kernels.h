// Kernel entry points shared between the kernel and host translation units.
#pragma once
#include <hip/hip_runtime.h>

#include "mjh_model.h"

namespace mjh {

constexpr int kMaxBlock = 256;  // threads per work-group of the step kernel

// LDS words of a work-group's triangular pair table (16-byte aligned)
__host__ __device__ inline int table_words(const DevModel& m) {
  return ((m.ntri + 3) / 4 + 3) & ~3;
}

// Launch shape of the register-resident solves: team size and padded row length (0: the
// batch takes the solves in LDS; team 0: a batch whose groups have different shapes).
struct RegShape {
  int team = 0, nb = 0;
};
// The shape for worlds of this model on `team` lanes; nb = 0 where the solves stay in LDS: a
// world that does not fit its team (16 lanes, more than 16 dofs) or has more than 28 dofs (two
// matrix rows a lane would not leave the registers of two waves per SIMD), contacts other than
// condim-3 pyramids (the quad-per-contact layout), and at most 16 dofs on 64 lanes, which has no
// instantiation and was not measured (by default those are models of 9 to 16 dofs with more than
// 32 rows).  Where both run, the registers are 1.4 (64 cartpoles: 14.4 against 10.5 us) to 4.2
// times (1999 quadrupeds by Runge-Kutta: 1297 against 312 us) as fast.
inline RegShape reg_shape(const DevModel& m, int team) {
  RegShape r;
  if (!m.jframe || m.cone || m.nv < 1 || m.nv > 28) return r;
  const int nb = m.nv <= 16 ? 16 : m.nv <= 20 ? 20 : 28;
  if (team == 16 ? nb != 16 : team == 64 ? nb == 16 : team != 32) return r;
  r.team = team;
  r.nb = nb;
  return r;
}
// Whether a batch of several shapes has a register-resident kernel for this one: the default
// shapes of the cart-pole, the quadruped, the humanoid and the hand (4096 of the last three x 2
// steps: 753 us with the solves in LDS, 280 with this kernel).  Every shape that the one kernel
// holds runs at the registers of its largest (171 VGPRs, two waves a SIMD).  Other shapes and
// Runge-Kutta were not measured in it; a batch that has one keeps the solves in LDS for all.
inline bool mix_shape(const RegShape& r) {
  return (r.team == 16 && r.nb == 16) || (r.team == 32 && r.nb == 20) ||
         (r.team == 64 && r.nb == 28);
}
// Whether the env step has a register-resident kernel for this shape: quadrupeds on 32 lanes
// (8192 x 4 substeps: 728 us with the solves in LDS, 260 with it).  Other shapes (a quadruped with
// joint limits and friction loss takes 64 lanes) were not measured and keep the solves in LDS.
inline bool env_reg_shape(const RegShape& r, bool rk4) { return r.team == 32 && r.nb == 20 && !rk4; }

// Launch the step kernel: one work-group of `block` threads per task; rk4 selects the
// instantiation that can run fourth-order Runge-Kutta groups, cone the one that can
// also solve elliptic-cone models.
hipError_t launch_step(const DevGroup* groups, const DevTask* tasks, int ntask, int nstep,
                       int block, size_t lds_bytes, int tab_words, bool rk4, bool cone,
                       RegShape reg, hipStream_t stream);
hipError_t launch_step_reg(const DevGroup* groups, const DevTask* tasks, int ntask, int nstep,
                           int block, size_t lds_bytes, bool rk4, RegShape reg,
                           hipStream_t stream);
// Dynamic LDS a kernel may use without asking, and the requests for more (made when a batch's
// launch shape is set, or for its env step, not for every instantiation when a context is
// created: that took 2 ms).  A kernel's limit is shared by all batches: ask for the device's, not
// for one batch's need, which would lower it under another's.
constexpr size_t kDefaultLds = 65536;
hipError_t allow_step_reg_lds(RegShape reg, bool rk4, size_t bytes);
hipError_t allow_env_reg_lds(bool dr, size_t bytes);
// Allow the step kernel `bytes` of dynamic LDS per work-group.
hipError_t set_step_lds_limit(size_t bytes);
// Compute body_invweight of a freshly uploaded model (one work-group).
hipError_t launch_invweight(const DevModel& m, hipStream_t stream);

// Joystick environment steps of a single-group batch (the step kernel's tasks).
struct EnvArgs {
  int nenv, nsub, nobs;
  const float* action;      // [nenv][nworld][nu]
  const float* command;     // [nworld][3]
  const float* reset_qpos;  // [nworld][nq]
  const float* reset_qvel;  // [nworld][nv]
  float* last_action;       // [nworld][nu], read and updated
  float* obs;               // [nenv][nworld][nobs]
  float* reward;            // [nenv][nworld]
  int* done;                // [nenv][nworld]
  int ndr;                  // 8 + 2 nu with per-world parameters, else 0
  const float* dr;          // [nworld][ndr] or nullptr
  const float* noise;       // [nenv][nworld][nobs] or nullptr
};
// ap_words: LDS words after the pair table for the teams' previous actions
hipError_t launch_env(const DevGroup* groups, const DevTask* tasks, int ntask, const EnvArgs& E,
                      int block, size_t lds_bytes, int tab_words, int ap_words, bool rk4,
                      RegShape reg, hipStream_t stream);
hipError_t launch_env_reg(const DevGroup* groups, const DevTask* tasks, int ntask,
                          const EnvArgs& E, int block, size_t lds_bytes, int tab_words,
                          int ap_words, hipStream_t stream);
hipError_t set_env_lds_limit(size_t bytes);

}  // namespace mjh
