"""The tree sweeps with one body per lane, against the FP64 reference: trees of one body less
than a team's lanes, exactly as many and one more (which take the loops over tables), with
bodies of no, one and three joints, slides, a free joint that is not the first, turned body
frames, joints off their bodies' origins and a body of many children.

One step without constraints is qacc = M^-1 (tau - c).  FP32 rounds every product of a chain of
depth d once or twice, so M and the forces carry a relative error of a few d eps, which the solve
amplifies by M's condition number.  Elimination without pivots does not see a scaling of the
dofs, so both are taken after scaling M to a unit diagonal: the gate is 16 n eps cond, n =
max(nv, bodies), of |D qacc| with D = diag(M)^(1/2).
"""
import numpy as np
import pytest

import oracle
from paper_2502_08844_amd.synth import inputs, robots
from tests.gpu_util import gpu_ctx, run_gpu

pytestmark = pytest.mark.gpu

EPS32 = 2.0 ** -24


@pytest.fixture(scope="module")
def lib():
    return gpu_ctx()


def _tree(nbody, ndof, plain, seed):
    """`nbody` bodies (the world left out) under at most `ndof` dofs; `plain`: no turned frames
    and no joint off its origin."""
    r = inputs.rng(seed, 31)
    bld = robots._Builder(f"tree{nbody}_{ndof}")
    left = ndof
    free_at = 2 if nbody > 2 and left >= 10 else -1
    for k in range(1, nbody + 1):
        # a star around body 1 (more children than a record holds), then chains
        parent = 0 if k in (1, free_at) else 1 if k < 9 else int(r.integers(k - 6, k))
        quat = (1, 0, 0, 0)
        if not plain and k != free_at:
            quat = robots.axis_angle_quat(r.normal(size=3) / 2, float(r.uniform(-1, 1)))
            quat = tuple(np.asarray(quat) / np.linalg.norm(quat))
        b = bld.body(parent, pos=0.1 * r.normal(size=3), quat=quat)
        if k == free_at:
            bld.joint(b, robots.JNT_FREE)
            left -= 6
        else:
            for t in range(min((1, 3, 0, 1)[k % 4], left - (6 if k < free_at else 0))):
                ax = r.normal(size=3)
                bld.joint(b, robots.JNT_SLIDE if (k + t) % 5 == 0 else robots.JNT_HINGE,
                          axis=ax / np.linalg.norm(ax), damping=0.05, armature=1.0,
                          pos=(0, 0, 0) if plain else 0.05 * r.normal(size=3))
                left -= 1
        bld.geom(b, robots.GEOM_BOX, 0.15 + 0.1 * r.uniform(size=3), pos=0.05 * r.normal(size=3),
                 mass=float(r.uniform(0.5, 1.5)) * 8 / nbody)
    m = bld.finish()
    m.opt = robots.Options(timestep=1e-3, iterations=1, nconmax=0)
    m.qpos0 = np.zeros(m.nq)
    m.qpos0[[a + 3 for j, a in zip(m.joints, m.jnt_qposadr()) if j.type == robots.JNT_FREE]] = 1
    return m


@pytest.mark.parametrize("plain", [False, True])
@pytest.mark.parametrize("team,ndof", [(16, 10), (16, 16), (32, 20), (64, 28)])
@pytest.mark.parametrize("over", [-1, 0, 1])
def test_bodies_around_the_lane_count(lib, team, ndof, over, plain):
    mjh, ctx = lib
    m = _tree(team + over, ndof, plain, seed=team + over)
    nw = 5
    r = inputs.rng(ndof, 32)
    qp = np.tile(m.qpos0, (nw, 1))
    for j, a in zip(m.joints, m.jnt_qposadr()):
        qp[:, a] += r.uniform(-0.5, 0.5, nw)
    qp = inputs.f32(qp)
    qv = inputs.f32(r.normal(0.0, 0.5, (nw, m.nv)))
    o = oracle.Oracle(m)
    ref = o.step(qp.copy(), qv.copy(), None, None, nstep=1)
    print(f"[gpu] {m.nbody - 1} bodies, {m.nv} dofs on {team} lanes", flush=True)
    g = run_gpu(ctx, mjh, m, qp, qv, None, None, 1, team=team, block=64, contacts=False)
    n = max(m.nv, m.nbody)
    for w in range(nw):
        M = o.forward(qp[w], qv[w], np.zeros(m.nv), None)["M"]
        D = np.sqrt(np.diag(M))
        cond = np.linalg.cond(M / D[:, None] / D)
        err = np.abs(D * (g["qacc"][w] - ref["qacc"][w])).max() / np.abs(D * ref["qacc"][w]).max()
        assert err <= 16 * n * EPS32 * max(cond, 10.0), (w, err, cond)
