"""Friction-loss bounds from far below to far above the forces in play, against the FP64
reference: the line search evaluates each row's clamped force as it stands, so no digits go
where a bound is large (a bound of 1e8 N m is a locked joint).  256 quadrupeds, ten Newton
iterations, the tolerances of the other parity tests (qacc 1e-4, contact forces 1e-3).  Up to 28
rows on 32 lanes and 40 on 64 hold a row a lane; 40 on 32 are walked in LDS."""
import numpy as np
import pytest

import oracle
from paper_2502_08844_amd.synth import inputs, robots
from tests.gpu_util import compare_step, gpu_ctx, run_gpu, summarize

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lib():
    return gpu_ctx()


@pytest.mark.parametrize("team,limits", [(32, False), (64, True), (32, True)])
@pytest.mark.parametrize("bound", [0.1, 30.0, 1e4, 3e5, 1e7, 1e8])
def test_friction_bounds(lib, bound, team, limits):
    mjh, ctx = lib
    m = robots.quadruped(iterations=10, frictionloss=bound, limits=limits)
    nw = 256
    qp, qv = inputs.initial_state("quadruped", m, nw, seed=31)
    qp[:, 2] -= 0.003
    qp = inputs.f32(qp)
    qv = inputs.f32(qv + inputs.rng(31, 16).normal(0.0, 0.3, qv.shape))
    u = inputs.controls("quadruped", m, nw, 1, seed=31)
    ws = np.zeros((nw, m.nv))
    print(f"[gpu] friction bound {bound:g} on {team} lanes, limits {limits}", flush=True)
    g = run_gpu(ctx, mjh, m, qp, qv, ws, u, 1, team=team, block=64)
    cmp = compare_step(m, oracle.Oracle(m), (qp, qv, ws), u, g)
    cmp["t"], cmp["ncon"] = 0, g["ncon"]
    ea, ef, nflag, ntot = summarize(f"friction bound {bound:g}", [cmp])
    assert ea.max() <= 1e-4
    assert ef.max() <= 1e-3
    assert nflag <= 0.02 * ntot
