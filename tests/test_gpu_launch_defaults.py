"""Default launch shapes: the env step's LDS words still fit beside a work-group's worlds, and
models on the solves in LDS keep the shapes that were measured for them."""
import numpy as np
import pytest
import torch

from paper_2502_08844_amd.synth import robots
from paper_2502_08844_amd.synth.model import (ACT_PD, GEOM_BOX, GEOM_PLANE, GEOM_SPHERE, JNT_FREE,
                                              JNT_HINGE, Actuator, Options)
from tests.gpu_util import gpu_ctx

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lib():
    return gpu_ctx()


def _many_legs(n, ncon, fixed=0):
    """A free box with n one-hinge legs with position actuators, ncon of them with a foot, and
    `fixed` bodies without joints."""
    b = robots._Builder("many_legs")
    floor = b.geom(0, GEOM_PLANE, (0, 0, 0))
    root = b.body(0, pos=(0, 0, 1))
    b.joint(root, JNT_FREE)
    b.geom(root, GEOM_BOX, (0.1, 0.1, 0.1), mass=5.0)
    hinges, feet = [], []
    for i in range(n):
        leg = b.body(root, pos=(0.1, 0.05 * i, 0))
        hinges.append(b.joint(leg, JNT_HINGE, axis=(0, 1, 0)))
        feet.append(b.geom(leg, GEOM_SPHERE, (0.05,), pos=(0, 0, -0.2), mass=0.3))
    for i in range(fixed):
        b.geom(b.body(root, pos=(-0.1, 0, 0.01 * i)), GEOM_BOX, (0.01, 0.01, 0.01), mass=0.01)
    m = b.finish()
    m.actuators = [Actuator(type=ACT_PD, joint=j, gear=1.0, kp=20.0, kd=0.5, ctrlrange=(-1.0, 1.0),
                            qdefault=0.0) for j in hinges]
    m.pairs = [(floor, f, 1.0, 3, 0, 0) for f in feet[:ncon]]
    m.opt = Options(timestep=0.004, iterations=4, ls_iterations=8, nconmax=ncon, integrator=0)
    m.qpos0 = np.zeros(m.nq)
    m.qpos0[2] = m.qpos0[3] = 1.0
    return m


@pytest.mark.parametrize("legs,ncon,randomised", [(46, 6, False), (43, 8, True), (48, 8, True)])
def test_env_step_fits_beside_the_default_worlds(lib, legs, ncon, randomised):
    """Worlds of 20 to 23 KB: as many as 256 threads hold fill the LDS to the last few hundred
    bytes, and the env step needs words of its own."""
    _env_step(*lib, _many_legs(legs, ncon), randomised)


def test_env_step_fits_on_the_register_solves(lib):
    """20 dofs and 97 bodies without joints: eight worlds of 20,300 bytes fit in 160 KB, but not
    with the words that randomised worlds need in the env step."""
    mjh, ctx = lib
    m = _many_legs(14, 6, 97)
    d = ctx.model_upload(m).dims
    room = 160 * 1024 - (d.nv * (d.nv + 1) // 2 + 15) // 16 * 16 - 8 * d.lds_bytes
    assert 0 <= room < 4 * 8 * (3 * m.nu + 8)
    _env_step(mjh, ctx, m, True)


def _env_step(mjh, ctx, m, randomised):
    nw = 17
    print(f"[gpu] env step, {m.nu} legs, randomised {randomised}", flush=True)
    w = mjh.World(ctx, m, nw, qpos=np.tile(m.qpos0, (nw, 1)))
    z = lambda *s: torch.zeros(*s, device="cuda")  # noqa: E731
    params = None
    if randomised:
        params = z(nw, 8 + 2 * m.nu)
        params[:, 0] = 1.0
        params[:, 5:7] = 1.0
    obs = z(1, nw, 12 + 3 * m.nu)
    w.batch.env_step(1, z(1, nw, m.nu), z(nw, 3), w.qpos.clone(), w.qvel.clone(), z(nw, m.nu),
                     obs, z(1, nw), torch.zeros(1, nw, dtype=torch.int32, device="cuda"),
                     params=params)
    torch.cuda.synchronize()
    assert torch.isfinite(obs).all()
    assert torch.allclose(w.qvel[:, 2], torch.full((nw,), -9.81 * 0.004, device="cuda"), atol=1e-4)


@pytest.mark.parametrize("kind", ["quadruped_elliptic", "quadruped_frictionless",
                                  "quadruped_rolling"])
def test_solves_in_lds_keep_their_launch_shape(lib, kind):
    mjh, ctx = lib
    m = robots.WORKLOADS[kind]()
    b = ctx.world_alloc([ctx.model_upload(m)], [64])
    team, block = b.get_launch(0)
    assert block == (64 if team == 64 else 128)
    mix = ctx.world_alloc([ctx.model_upload(robots.quadruped()), ctx.model_upload(m)], [64, 64])
    assert mix.get_launch(0) == (32, 128)  # (the whole batch takes the solves in LDS)
