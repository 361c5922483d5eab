"""Status bits of worlds that are not finite: WORLD_NONFINITE alone where the Newton Hessian,
which depends on the pose, still has its factor; and their wavefront neighbours are untouched."""
import numpy as np
import pytest
import torch

from paper_2502_08844_amd.synth import inputs, robots
from tests.gpu_util import gpu_ctx

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lib():
    return gpu_ctx()


@pytest.mark.parametrize("kind,team", [("quadruped", 32), ("quadruped", 64), ("quadruped", 16),
                                       ("quadruped_limits", 32), ("humanoid", 64), ("hand", 64)])
def test_infinite_velocity_is_no_failed_factor(lib, kind, team):
    mjh, ctx = lib
    m = robots.WORKLOADS[kind]()
    nw = 21
    base = kind.split("_")[0]
    qp, qv = inputs.initial_state(base, m, nw, seed=7)
    qp[:, 18 if base == "hand" else 2] -= 0.002
    u = torch.tensor(inputs.controls(base, m, nw, 2, seed=7), dtype=torch.float32, device="cuda")
    bad = np.arange(nw) % 3 == 1
    qbad = qv.copy()
    qbad[bad, 0] = np.inf
    out = []
    for v in (qv, qbad):
        print(f"[gpu] {kind} on {team} lanes, infinite {np.isinf(v).any()}", flush=True)
        w = mjh.World(ctx, m, nw, qpos=qp, qvel=v)
        w.batch.set_launch(0, team, 64)
        w.step(u)
        torch.cuda.synchronize()
        out.append((w.status.cpu().numpy(), w.qacc_ws.cpu().numpy(), w.qvel.cpu().numpy()))
    (s0, a0, v0), (s1, a1, v1) = out
    assert np.all(s1[bad] == mjh.WORLD_NONFINITE), s1
    for x, y in ((s0, s1), (a0, a1), (v0, v1)):
        assert np.array_equal(x[~bad], y[~bad])
