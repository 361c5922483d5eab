"""The register-resident solves (one dof per lane, matrix rows in registers) at the edges of
their row lengths and team sizes, against the FP64 reference.

Rows are padded to 16, 20 or 28 entries; 29 dofs and 17 dofs on 16 lanes take the solves in
LDS.  Hinge chains cover every edge of the elimination of M (their inertias spread over the
chain make it ill conditioned, so the gate scales with the condition number: FP32 elimination
of an SPD matrix is backward stable, error <= c n eps cond).  Contact worlds cover wavefronts
with one, two and four worlds whose contact counts differ, down to none.
"""
import numpy as np
import pytest
import torch

import oracle
from paper_2502_08844_amd.synth import inputs, robots
from tests.gpu_util import gpu_ctx, run_gpu

pytestmark = pytest.mark.gpu

EPS32 = 2.0 ** -24


@pytest.fixture(scope="module")
def lib():
    return gpu_ctx()


@pytest.mark.parametrize("team", [16, 32, 64])
@pytest.mark.parametrize("n", [1, 15, 16, 17, 20, 21, 28, 29])
def test_chain_lengths(lib, n, team):
    mjh, ctx = lib
    m = robots.hinge_chain(n, damping=0.05)
    nw = 5
    r = inputs.rng(n, 11)
    qp = inputs.f32(r.uniform(-0.6, 0.6, (nw, m.nq)))
    qv = inputs.f32(r.normal(0.0, 0.5, (nw, m.nv)))
    o = oracle.Oracle(m)
    ref = o.step(qp.copy(), qv.copy(), None, None, nstep=1)
    print(f"[gpu] chain of {n} on {team} lanes", flush=True)
    g = run_gpu(ctx, mjh, m, qp, qv, None, None, 1, team=team, block=64, contacts=False)
    for w in range(nw):
        cond = np.linalg.cond(o.forward(qp[w], qv[w], np.zeros(m.nv), None)["M"])
        err = np.abs(g["qacc"][w] - ref["qacc"][w]).max() / max(np.abs(ref["qacc"][w]).max(), 9.81)
        assert err <= 8 * max(n, 4) * EPS32 * max(cond, 10.0), (w, err, cond)


@pytest.mark.parametrize("team,block", [(16, 64), (32, 64), (32, 128), (64, 64)])
@pytest.mark.parametrize("nw", [1, 3, 8])
def test_wavefront_worlds_with_different_contacts(lib, nw, team, block):
    """Worlds of one wavefront on the ground, tilted and in the air: each one's accelerations
    and forces match the reference, and equal those of the world alone bit for bit."""
    mjh, ctx = lib
    m = robots.quadruped()
    qp = np.tile(robots.quadruped_standing_qpos(m), (nw, 1))
    for w in range(nw):
        qp[w, 2] += (-0.002, 0.2, 0.001)[w % 3]
        qp[w, 7:] += inputs.rng(w, 12).uniform(-0.05, 0.05, 12) * (w % 3 > 0)
    qp = inputs.f32(qp)
    qv = inputs.f32(inputs.rng(5, 13).normal(0.0, 0.1, (nw, m.nv)))
    u = inputs.controls("quadruped", m, nw, 1, seed=3)
    o = oracle.Oracle(m)
    ref = o.step(qp.copy(), qv.copy(), None, u, nstep=1)
    print(f"[gpu] {nw} quadrupeds, {team} lanes, work-group {block}", flush=True)
    g = run_gpu(ctx, mjh, m, qp, qv, None, u, 1, team=team, block=block)
    assert np.array_equal(g["ncon"], ref["ncon"])
    err = np.abs(g["qacc"] - ref["qacc"]).max(1) / np.maximum(np.abs(ref["qacc"]).max(1), 9.81)
    assert err.max() < 1e-4, err
    weight = m.total_mass() * 9.81
    df = np.abs(g["contacts"][:, :, 13:16] - ref["contacts"][:, :, 13:16]).max() / weight
    assert df < 1e-3, df
    for w in range(nw):
        one = run_gpu(ctx, mjh, m, qp[w:w + 1], qv[w:w + 1], None, u[:, w:w + 1], 1, team=team,
                      block=block)
        assert np.array_equal(one["qacc"][0], g["qacc"][w]), w


def test_registers_agree_with_lds_solves(lib):
    """The same quadruped through the register-resident solves (32 lanes) and the solves in
    LDS (16 lanes, fewer than its dofs)."""
    mjh, ctx = lib
    m = robots.quadruped()
    nw = 33
    qp, qv = inputs.initial_state("quadruped", m, nw, seed=21)
    qp[:, 2] -= 0.004
    u = inputs.controls("quadruped", m, nw, 1, seed=21)
    a = run_gpu(ctx, mjh, m, inputs.f32(qp), qv, None, u, 1, team=32, block=128)
    b = run_gpu(ctx, mjh, m, inputs.f32(qp), qv, None, u, 1, team=16, block=64)
    err = np.abs(a["qacc"] - b["qacc"]).max(1) / np.maximum(np.abs(b["qacc"]).max(1), 9.81)
    assert err.max() < 2e-4, err.max()  # both are held to 1e-4 of the reference
    torch.cuda.synchronize()


@pytest.mark.parametrize("kind,team", [("quadruped", 32), ("quadruped", 64), ("humanoid", 64)])
def test_rollout_gradients_of_partial_wavefronts(lib, kind, team):
    """Three worlds (an odd count: the last wavefront's spare lanes shadow its world) against
    the same worlds one at a time, bit for bit, and against directional derivatives of the
    reference (central differences; the gate is the adjoint's, 1e-3 of |grad| |d|)."""
    mjh, ctx = lib
    m = robots.WORKLOADS[kind]()
    H, nw = 6, 3
    qp, qv = inputs.initial_state(kind, m, nw, seed=8)
    qp[:, 2] -= 0.003
    qp = inputs.f32(qp)
    u = inputs.controls(kind, m, nw, H, seed=8)

    def grads(ws):
        w = mjh.World(ctx, m, len(ws), qpos=qp[ws])
        w.batch.set_launch(0, team, 64)
        v = torch.tensor(qv[ws], dtype=torch.float32, device="cuda", requires_grad=True)
        c = torch.tensor(u[:, ws], dtype=torch.float32, device="cuda", requires_grad=True)
        mjh.Rollout.apply(v, c, w, H, 4).sum().backward()
        return v.grad.cpu().numpy(), c.grad.cpu().numpy()

    print(f"[gpu] rollout gradients, {nw} x {kind} on {team} lanes", flush=True)
    gv, gc = grads([0, 1, 2])
    for w in range(nw):
        v1, c1 = grads([w])
        assert np.array_equal(v1[0], gv[w]) and np.array_equal(c1[:, 0], gc[:, w]), w
    o = oracle.Oracle(m)
    r = inputs.rng(8, 21)
    for _ in range(3):
        dv, dc = r.normal(size=gv.shape), r.normal(size=gc.shape)
        h = 1e-6
        up = o.rollout_loss(qp, qv + h * dv, u + h * dc, mode=oracle.MODE_CONVERGED)
        dn = o.rollout_loss(qp, qv - h * dv, u - h * dc, mode=oracle.MODE_CONVERGED)
        want = (up - dn) / (2 * h)
        got = (gv * dv).sum(1) + (gc * dc).sum((0, 2))
        scale = np.sqrt((gv ** 2).sum(1) + (gc ** 2).sum((0, 2))) * np.sqrt(
            (dv ** 2).sum(1) + (dc ** 2).sum((0, 2)))
        assert np.all(np.abs(got - want) <= 1e-3 * scale), (got, want, scale)


@pytest.mark.parametrize("team", [32, 64])
@pytest.mark.parametrize("power,mid", [(1.0, 0.5), (2.0, 0.3), (2.0, 0.5), (3.0, 0.7)])
def test_impedance_curves(lib, power, mid, team):
    """The impedance's products (power 2) and powers, on both sides of the middle: feet from
    just touching to deeper than the impedance width, four and no contacts in one wavefront."""
    mjh, ctx = lib
    m = robots.quadruped()
    m.opt.solimp = (0.6, 0.9, 0.004, mid, power)
    nw = 9
    qp = np.tile(robots.quadruped_standing_qpos(m), (nw, 1))
    qp[:, 2] -= np.linspace(-0.0005, 0.006, nw)
    qp[nw // 2, 2] += 0.2
    qp = inputs.f32(qp)
    qv = inputs.f32(inputs.rng(7, 14).normal(0.0, 0.1, (nw, m.nv)))
    u = inputs.controls("quadruped", m, nw, 1, seed=5)
    ref = oracle.Oracle(m).step(qp.copy(), qv.copy(), None, u, nstep=1)
    print(f"[gpu] impedance of power {power}, middle {mid} on {team} lanes", flush=True)
    g = run_gpu(ctx, mjh, m, qp, qv, None, u, 1, team=team, block=64)
    assert np.array_equal(g["ncon"], ref["ncon"])
    err = np.abs(g["qacc"] - ref["qacc"]).max(1) / np.maximum(np.abs(ref["qacc"]).max(1), 9.81)
    assert err.max() < 1e-4, err


@pytest.mark.parametrize("team", [16, 32, 64])
@pytest.mark.parametrize("n", [1, 4, 15, 16, 17, 20, 21, 28])
def test_newton_at_row_lengths(lib, n, team):
    """Newton's elimination (on the matrix cores for 32 and 64 lanes) at every edge of the padded
    rows, on unit rows: chains with friction loss on every joint, of which some are past their
    limits.  A limit's D is imp / (1 - imp) <= 19 of its dof's diagonal entry, so cond(H) <= 20
    cond(M) with M scaled to a unit diagonal (which elimination does not see), and the gate is
    that of the chains above with it."""
    mjh, ctx = lib
    m = robots.hinge_chain(n, damping=0.05, limit=0.3, frictionloss=0.02)
    for j in m.joints:
        j.armature = 1000.0
    m.opt.iterations = 10
    nw = 5
    r = inputs.rng(n, 15)
    qp = inputs.f32(r.uniform(-0.35, 0.35, (nw, m.nq)))
    qp[1] *= 0.5  # (no limit reached)
    qp = inputs.f32(qp)
    qv = inputs.f32(r.normal(0.0, 0.2, (nw, m.nv)))
    o = oracle.Oracle(m)
    ref = o.step(qp.copy(), qv.copy(), None, None, nstep=1)
    print(f"[gpu] limited chain of {n} on {team} lanes", flush=True)
    g = run_gpu(ctx, mjh, m, qp, qv, None, None, 1, team=team, block=64, contacts=False)
    for w in range(nw):
        M = o.forward(qp[w], qv[w], np.zeros(m.nv), None)["M"]
        D = np.sqrt(np.diag(M))
        cond = 20 * np.linalg.cond(M / D[:, None] / D)
        err = np.abs(D * (g["qacc"][w] - ref["qacc"][w])).max() / np.abs(D * ref["qacc"][w]).max()
        assert err <= 8 * max(n, 4) * EPS32 * cond, (w, err, cond)
