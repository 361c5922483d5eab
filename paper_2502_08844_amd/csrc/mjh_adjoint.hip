// Host side of the differentiable rollouts, and the rollout kernels with their solves in LDS.
#include <algorithm>
#include <mutex>

#include "mjh_adjoint_dev.h"

namespace mjh {

// The kernels for this model and team size: register-resident solves where an instantiation
// has them (reg_shape; the unit rows' slots also take 4 nv words of the bodies' scratch).
static RolloutKernels rollout_kernels(const DevModel& m, int team) {
  const RegShape r = reg_shape(m, team);
  if (4 * m.nv <= 24 * m.nbody) {
    if (r.team == 32 && r.nb == 20) return rollout_kernels_32_20();
    if (r.team == 64 && r.nb == 20) return rollout_kernels_64_20();
    if (r.team == 64 && r.nb == 28) return rollout_kernels_64_28();
  }
  RolloutKernels k;
  k.fwd = rollout_fwd_kernel<0, 0>;
  k.bwd = rollout_bwd_kernel<0, 0>;
  return k;
}

// ------------------------------------------------------------------ host side
struct AdjointState {
  RolloutArgs args{};
  float* tape_ckpt = nullptr;
  float* tape_seg = nullptr;
  unsigned* tape_snap = nullptr;
  size_t snap_alloc = 0;  // words
  int* status = nullptr;
  size_t ckpt_words = 0, seg_words = 0, status_words = 0;
  bool have_fwd = false;
  int64_t generation = 0;  // number of forward rollouts so far; the tapes hold the last
};

static int blocks_for(int nworld, int team) {
  const int wpb = kAdjBlock / team;
  return (nworld + wpb - 1) / wpb;
}

mjh_status adjoint_forward(AdjointState** stp, const DevModel& m, int team, int nworld, float* qpos,
                           float* qvel, float* qacc, int horizon, int ckpt, const float* ctrl,
                           int zidx, float ztarget, float wctrl, float* loss, int64_t* generation,
                           hipStream_t stream, std::string& err) {
  if (horizon <= 0 || ckpt <= 0 || (!ctrl && m.nu > 0) || !loss || zidx < 0 || zidx >= m.nq) {
    err = "rollout_fwd: need horizon > 0, ckpt_every > 0, ctrl, loss and 0 <= zidx < nq";
    return MJH_EINVAL;
  }
  if (!qpos || !qvel || !qacc) { err = "rollout_fwd: state not bound"; return MJH_ESTATE; }
  // the reverse sweep differentiates plane-sphere / plane-capsule contact geometry
  team = (team == 16 || team == 32 || team == 64) ? team : 32;
  AdjointState* st = *stp;
  if (!st) {
    st = new (std::nothrow) AdjointState();
    if (!st) { err = "rollout_fwd: out of host memory"; return MJH_ENOMEM; }
    *stp = st;
  }
  const int nseg = (horizon + ckpt - 1) / ckpt;
  const size_t ns = (size_t)m.nq + 2 * m.nv;
  const size_t need_ckpt = (size_t)nseg * nworld * ns;
  const size_t need_seg = (size_t)(std::min(ckpt, horizon) + 1) * nworld * ns;
  if (need_ckpt > st->ckpt_words) {
    if (st->tape_ckpt) (void)hipFree(st->tape_ckpt);
    st->tape_ckpt = nullptr;
    if (hipMalloc(&st->tape_ckpt, need_ckpt * sizeof(float)) != hipSuccess) {
      st->ckpt_words = 0;
      err = "rollout_fwd: out of device memory (checkpoints)";
      return MJH_ENOMEM;
    }
    st->ckpt_words = need_ckpt;
  }
  if (need_seg > st->seg_words) {
    if (st->tape_seg) (void)hipFree(st->tape_seg);
    st->tape_seg = nullptr;
    if (hipMalloc(&st->tape_seg, need_seg * sizeof(float)) != hipSuccess) {
      st->seg_words = 0;
      err = "rollout_fwd: out of device memory (segment tape)";
      return MJH_ENOMEM;
    }
    st->seg_words = need_seg;
  }
  const size_t need_snap =
      (size_t)std::min(ckpt, horizon) * (m.rk4 ? 4 : 1) * nworld * (size_t)m.o_qbi;
  if (need_snap > st->snap_alloc) {
    if (st->tape_snap) (void)hipFree(st->tape_snap);
    st->tape_snap = nullptr;
    if (hipMalloc(&st->tape_snap, need_snap * sizeof(unsigned)) != hipSuccess) {
      st->snap_alloc = 0;
      err = "rollout_fwd: out of device memory (on-chip images of a segment)";
      return MJH_ENOMEM;
    }
    st->snap_alloc = need_snap;
  }
  if ((size_t)nworld > st->status_words) {
    if (st->status) (void)hipFree(st->status);
    st->status = nullptr;
    if (hipMalloc(&st->status, sizeof(int) * (size_t)nworld) != hipSuccess) {
      st->status_words = 0;
      err = "rollout_fwd: out of device memory";
      return MJH_ENOMEM;
    }
    st->status_words = (size_t)nworld;
  }
  RolloutArgs& A = st->args;
  A.m = m;
  A.nworld = nworld; A.horizon = horizon; A.ckpt = ckpt; A.zidx = zidx; A.team = team;
  A.nseg = nseg; A.ztarget = ztarget; A.wctrl = wctrl;
  A.qpos = qpos; A.qvel = qvel; A.qacc = qacc; A.ctrl = ctrl;
  A.tape_ckpt = st->tape_ckpt; A.tape_seg = st->tape_seg; A.loss = loss; A.status = st->status;
  A.tape_snap = st->tape_snap; A.snap_words = m.o_qbi;
  st->have_fwd = false;
  // the tapes are about to be overwritten: an earlier rollout can no longer be reversed
  st->generation++;
  if (generation) *generation = st->generation;
  if (nworld == 0) { st->have_fwd = true; return MJH_OK; }
  const size_t lds =
      ((size_t)table_words(m) + (size_t)(kAdjBlock / team) * m.lds_words) * sizeof(float);
  const RolloutKernels k = rollout_kernels(m, team);
  hipError_t e = hipFuncSetAttribute((const void*)k.fwd,
                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (e == hipSuccess)
    e = hipFuncSetAttribute((const void*)k.bwd,
                            hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (e != hipSuccess) { err = std::string("rollout_fwd: ") + hipGetErrorString(e); return MJH_EHIP; }
  hipLaunchKernelGGL(k.fwd, dim3(blocks_for(nworld, team)), dim3(kAdjBlock), lds,
                     stream, A);
  e = hipGetLastError();
  if (e != hipSuccess) { err = std::string("rollout_fwd: ") + hipGetErrorString(e); return MJH_EHIP; }
  st->have_fwd = true;
  return MJH_OK;
}

mjh_status adjoint_backward(AdjointState* st, int64_t generation, const float* dloss,
                            float* grad_qvel0, float* grad_ctrl, hipStream_t stream,
                            std::string& err) {
  if (!st || !st->have_fwd) { err = "rollout_bwd: call rollout_fwd first"; return MJH_ESTATE; }
  if (generation != st->generation) {
    err = "rollout_bwd: the tapes hold rollout " + std::to_string(st->generation) +
          ", not rollout " + std::to_string(generation) + " (a later rollout_fwd replaced it)";
    return MJH_ESTATE;
  }
  if (!dloss || !grad_qvel0 || (!grad_ctrl && st->args.m.nu > 0)) {
    err = "rollout_bwd: NULL argument";
    return MJH_EINVAL;
  }
  RolloutArgs A = st->args;
  A.dloss = dloss;
  A.grad_qvel0 = grad_qvel0;
  A.grad_ctrl = grad_ctrl;
  if (A.nworld == 0) return MJH_OK;
  const size_t lds =
      ((size_t)table_words(A.m) + (size_t)(kAdjBlock / A.team) * A.m.lds_words) * sizeof(float);
  hipLaunchKernelGGL(rollout_kernels(A.m, A.team).bwd, dim3(blocks_for(A.nworld, A.team)), dim3(kAdjBlock), lds,
                     stream, A);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) { err = std::string("rollout_bwd: ") + hipGetErrorString(e); return MJH_EHIP; }
  return MJH_OK;
}

// ------------------------------------------------------------------ no-alloc rollouts
// Tapes of mjh_rollout_noalloc: one rollout's checkpoints, segment states and per-step
// on-chip images.  A file-scope device array: every device the library runs on holds its
// own copy from the module's load until the process ends, and every call on that device
// shares it (calls that overlap on one device race).  Host code never passes the array's
// name to a kernel: it is a host-side stand-in, not a device address.  The address comes
// from hipGetSymbolAddress, once per device, in noalloc_scratch_init.
static __device__ __align__(256) unsigned char scratch[kNoAllocScratchBytes];

constexpr int kMaxDevices = 64;
static std::mutex g_scratch_mu;
static unsigned char* g_scratch_ptr[kMaxDevices] = {};

hipError_t noalloc_scratch_init(int device) {
  if (device < 0 || device >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (g_scratch_ptr[device]) return hipSuccess;
  void* p = nullptr;
  const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
  if (e != hipSuccess) return e;
  g_scratch_ptr[device] = static_cast<unsigned char*>(p);
  return hipSuccess;
}

static size_t round256(size_t bytes) { return (bytes + 255) & ~size_t(255); }

size_t noalloc_tape_bytes(const DevModel& m, int nworld, int horizon, int ckpt) {
  const size_t nseg = (size_t)((horizon + ckpt - 1) / ckpt);
  const size_t seglen = (size_t)std::min(ckpt, horizon);
  const size_t ns = (size_t)m.nq + 2 * (size_t)m.nv;
  return round256(nseg * nworld * ns * sizeof(float)) +
         round256((seglen + 1) * nworld * ns * sizeof(float)) +
         round256(seglen * (m.rk4 ? 4 : 1) * nworld * (size_t)m.o_qbi * sizeof(unsigned));
}

mjh_status adjoint_noalloc(int device, const DevModel& m, int team, int nworld, float* qpos,
                           float* qvel, float* qacc, int horizon, int ckpt, const float* ctrl,
                           int zidx, float ztarget, float wctrl, const float* dloss, float* loss,
                           float* grad_qvel0, float* grad_ctrl, hipStream_t stream,
                           std::string& err) {
  if (horizon <= 0 || ckpt <= 0 || (!ctrl && m.nu > 0) || !loss || !dloss || !grad_qvel0 ||
      (!grad_ctrl && m.nu > 0) ||
      zidx < 0 || zidx >= m.nq) {
    err = "rollout_noalloc: need horizon > 0, ckpt_every > 0, ctrl, dloss, loss, gradients "
          "and 0 <= zidx < nq";
    return MJH_EINVAL;
  }
  if (!qpos || !qvel || !qacc) { err = "rollout_noalloc: state not bound"; return MJH_ESTATE; }
  if (nworld < 0) { err = "rollout_noalloc: negative world count"; return MJH_EINVAL; }
  const size_t need = noalloc_tape_bytes(m, nworld, horizon, ckpt);
  if (need > kNoAllocScratchBytes) {
    err = "rollout_noalloc: " + std::to_string(nworld) + " worlds over " +
          std::to_string(horizon) + " steps with a checkpoint every " + std::to_string(ckpt) +
          " need " + std::to_string(need) + " bytes of tape, more than the library's " +
          std::to_string(kNoAllocScratchBytes) + "-byte scratch";
    return MJH_EINVAL;
  }
  unsigned char* base = (device >= 0 && device < kMaxDevices) ? g_scratch_ptr[device] : nullptr;
  if (!base) { err = "rollout_noalloc: device scratch not initialised"; return MJH_ESTATE; }
  if (nworld == 0) return MJH_OK;
  team = (team == 16 || team == 32 || team == 64) ? team : 32;
  RolloutArgs A{};
  A.m = m;
  A.nworld = nworld; A.horizon = horizon; A.ckpt = ckpt; A.zidx = zidx; A.team = team;
  A.nseg = (horizon + ckpt - 1) / ckpt; A.ztarget = ztarget; A.wctrl = wctrl;
  A.qpos = qpos; A.qvel = qvel; A.qacc = qacc; A.ctrl = ctrl;
  const size_t ns = (size_t)m.nq + 2 * (size_t)m.nv;
  const size_t seglen = (size_t)std::min(ckpt, horizon);
  size_t off = 0;
  A.tape_ckpt = reinterpret_cast<float*>(base + off);
  off += round256((size_t)A.nseg * nworld * ns * sizeof(float));
  A.tape_seg = reinterpret_cast<float*>(base + off);
  off += round256((seglen + 1) * nworld * ns * sizeof(float));
  A.tape_snap = reinterpret_cast<unsigned*>(base + off);
  A.snap_words = m.o_qbi;
  A.status = nullptr;  // the rollouts' per-world status is not reported
  A.loss = loss; A.dloss = dloss; A.grad_qvel0 = grad_qvel0; A.grad_ctrl = grad_ctrl;
  const size_t lds =
      ((size_t)table_words(m) + (size_t)(kAdjBlock / team) * m.lds_words) * sizeof(float);
  const RolloutKernels k = rollout_kernels(m, team);
  hipError_t e = hipFuncSetAttribute((const void*)k.fwd,
                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (e == hipSuccess)
    e = hipFuncSetAttribute((const void*)k.bwd,
                            hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (e != hipSuccess) { err = std::string("rollout_noalloc: ") + hipGetErrorString(e); return MJH_EHIP; }
  // forward, then reverse: stream order keeps the reverse sweep behind the tapes' writes
  hipLaunchKernelGGL(k.fwd, dim3(blocks_for(nworld, team)), dim3(kAdjBlock), lds,
                     stream, A);
  e = hipGetLastError();
  if (e == hipSuccess) {
    hipLaunchKernelGGL(k.bwd, dim3(blocks_for(nworld, team)), dim3(kAdjBlock), lds,
                       stream, A);
    e = hipGetLastError();
  }
  if (e != hipSuccess) { err = std::string("rollout_noalloc: ") + hipGetErrorString(e); return MJH_EHIP; }
  return MJH_OK;
}

void adjoint_free(AdjointState* st) {
  if (!st) return;
  if (st->tape_ckpt) (void)hipFree(st->tape_ckpt);
  if (st->tape_seg) (void)hipFree(st->tape_seg);
  if (st->tape_snap) (void)hipFree(st->tape_snap);
  if (st->status) (void)hipFree(st->status);
  delete st;
}

}  // namespace mjh
