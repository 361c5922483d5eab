"""The plane-box search by eight lanes a pair against the FP64 reference: which of a box's corners
are kept, over all the ways they can be ranked (ties, four of eight, none), several boxes to a team
and more than it has half rows, mixed with pairs of other searches."""
import numpy as np
import pytest

import oracle
from paper_2502_08844_amd.synth import inputs, robots
from tests.gpu_util import gpu_ctx, run_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lib():
    return gpu_ctx()


def _boxes(n):
    """`n` free boxes and a free sphere over a plane; every pair of the plane, in mixed order."""
    bld = robots._Builder(f"boxes{n}")
    pl = bld.geom(0, robots.GEOM_PLANE, (0, 0, 0))
    gs = []
    for k in range(n + 1):
        b = bld.body(0, pos=(2.0 * k, 0, 1))
        bld.joint(b, robots.JNT_FREE)
        gs.append(bld.geom(b, robots.GEOM_SPHERE, (0.1,), mass=1.0) if k == n else
                  bld.geom(b, robots.GEOM_BOX, (0.1, 0.15, 0.2), mass=1.0))
    m = bld.finish()
    m.pairs = [(pl, g, 1.0, 3, 0.0, 0.0) for g in [gs[-1]] + gs[:-1]]
    m.opt = robots.Options(timestep=1e-3, iterations=10, nconmax=4 * n + 1)
    m.qpos0 = np.tile([0, 0, 1.0, 1, 0, 0, 0], n + 1).astype(float)
    return m


@pytest.mark.parametrize("team", [16, 32, 64])
@pytest.mark.parametrize("n", [1, 3, 9])
def test_plane_box_corners(lib, n, team):
    """Positions within 4 eps of the lengths involved (about 2 m): distances are sums of a few
    products of them."""
    mjh, ctx = lib
    m = _boxes(n)
    nw = 7
    r = inputs.rng(n, 16)
    qp = np.tile(m.qpos0, (nw, 1)).reshape(nw, n + 1, 7)
    qp[:, :, 0] = 0.25 * np.arange(n + 1)
    for w in range(nw):
        for k in range(n + 1):
            ang = (0.0, 0.0, 0.01, 0.5, 0.3, 0.0, 1.0)[(w + k) % 7]
            ax = r.normal(size=3)
            qp[w, k, 3:7] = robots.axis_angle_quat(ax / np.linalg.norm(ax), ang)
            # flat and tied, eight corners under, above, ...
            qp[w, k, 2] = (0.199, -0.3, 0.195, 0.15, 0.05, 0.5, -0.1)[(w + k) % 7]
    qp = inputs.f32(qp.reshape(nw, -1))
    qv = np.zeros((nw, m.nv))
    ref = oracle.Oracle(m).step(qp.copy(), qv.copy(), None, None, nstep=1)
    print(f"[gpu] {n} boxes on a plane, {team} lanes", flush=True)
    g = run_gpu(ctx, mjh, m, qp, qv, None, None, 1, team=team, block=64)
    assert np.array_equal(g["ncon"], ref["ncon"])
    assert ref["ncon"].max() >= 3 * n  # (of the reference: the inputs do reach full boxes)
    for w in range(nw):
        a, b = g["contacts"][w, :ref["ncon"][w]], ref["contacts"][w, :ref["ncon"][w]]
        assert np.array_equal(a[:, 16:18], b[:, 16:18]), w  # the pairs and their corners
        assert np.abs(a[:, :4] - b[:, :4]).max() < 4 * 2.0 * 2.0 ** -23, w
