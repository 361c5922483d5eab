"""A kernel's dynamic LDS limit is shared by every batch that launches it: a batch with a
smaller need must not lower it under one with a larger need that launches later."""
import ctypes as C

import numpy as np
import pytest
import torch

from paper_2502_08844_amd.synth import inputs, robots
from tests.gpu_util import gpu_ctx

pytestmark = pytest.mark.gpu


class FuncAttributes(C.Structure):  # hipFuncAttributes
    _fields_ = [("binary", C.c_int), ("cache", C.c_int), ("const_bytes", C.c_size_t),
                ("local_bytes", C.c_size_t), ("max_dynamic", C.c_int), ("max_threads", C.c_int),
                ("regs", C.c_int), ("carveout", C.c_int), ("ptx", C.c_int),
                ("shared_bytes", C.c_size_t)]


@pytest.fixture(scope="module")
def lib():
    return gpu_ctx()


def _limit(mjh, kernel):
    a = FuncAttributes()
    handle = C.c_char.in_dll(mjh._lib, kernel)
    assert mjh._lib.hipFuncGetAttributes(C.byref(a), C.c_void_p(C.addressof(handle))) == 0
    return a.max_dynamic


def _world(mjh, ctx, m, nw, team, block):
    qp, qv = inputs.initial_state(m.name.split("_")[0], m, nw, seed=1)
    w = mjh.World(ctx, m, nw, qpos=qp, qvel=qv)
    w.batch.set_launch(0, team, block)
    return w


def test_step_limit_never_falls(lib):
    mjh, ctx = lib
    kernel = "_ZN3mjh19mjh_step_reg_kernelILi64ELi28ELb0EEEvPKNS_8DevGroupEPKNS_7DevTaskEi"
    big, small = robots.humanoid(), robots.hand()
    worlds = []
    for m in (big, small):  # four worlds a work-group, over 64 KB in both
        print(f"[gpu] {m.name} in work-groups of 256", flush=True)
        w = _world(mjh, ctx, m, 9, 64, 256)
        u = torch.tensor(inputs.controls(m.name, m, 9, 1, seed=1), dtype=torch.float32,
                         device="cuda")
        w.step(u)
        worlds.append((w, u))
    need = [4 * w.model.dims.lds_bytes for w, _ in worlds]
    assert need[0] > need[1] > 65536
    assert _limit(mjh, kernel) >= need[0]
    w, u = worlds[0]
    w.step(u)
    torch.cuda.synchronize()
    assert torch.isfinite(w.qpos).all()


def test_env_limit_never_falls(lib):
    mjh, ctx = lib
    kernel = ("_ZN3mjh18mjh_env_reg_kernelILb0EEEvPKNS_8DevGroupEPKNS_7DevTaskENS_7EnvArgsEii")
    nw, need = 9, []
    for ncon in (40, 30):  # eight worlds a work-group
        m = robots.quadruped()
        m.opt.nconmax = ncon
        print(f"[gpu] env step with room for {ncon} contacts", flush=True)
        w = _world(mjh, ctx, m, nw, 32, 256)
        z = lambda *s: torch.zeros(*s, device="cuda")  # noqa: E731
        w.batch.env_step(1, z(1, nw, m.nu), z(nw, 3), w.qpos.clone(), w.qvel.clone(),
                         z(nw, m.nu), z(1, nw, 12 + 3 * m.nu), z(1, nw),
                         torch.zeros(1, nw, dtype=torch.int32, device="cuda"))
        torch.cuda.synchronize()
        assert np.isfinite(w.qpos.cpu().numpy()).all()
        need.append(8 * w.model.dims.lds_bytes)
    assert need[0] > need[1] > 65536
    assert _limit(mjh, kernel) >= need[0]
