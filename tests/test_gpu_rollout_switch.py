"""Rollout gradients of worlds with a contact row on the switch between its pieces.

A row's residual e = J a - aref decides by its sign whether the row is in the Hessian that the
gradient is taken with.  In each of these worlds one row of one step ends with |e| between
1e-8 and 2e-6 of the terms that it is the difference of (in 64 bits), so FP32 rounding picks
the side, and the gradients of the two sides differ by 0.25 to 4 % of the world's gradient.  The
rollouts keep the arithmetic of the solves in LDS so that the side, once given, stays: the
expected values are theirs (quadruped, 4 steps, a checkpoint every 2, 32 lanes).  The gate is
twenty times the FP32 error of a rollout without such a row (1e-6) and a hundredth of the
smallest jump between the sides.
"""
import json
import os

import numpy as np
import pytest
import torch

from paper_2502_08844_amd.synth import robots
from tests.gpu_util import gpu_ctx

pytestmark = pytest.mark.gpu

GOLDEN = os.path.join(os.path.dirname(__file__), "golden", "rollout_switch.json")


def test_gradients_at_a_row_switch_stay():
    mjh, ctx = gpu_ctx()
    m = robots.quadruped()
    with open(GOLDEN) as f:
        worlds = json.load(f)
    nw, H = len(worlds), len(worlds[0]["ctrl"]) // m.nu
    arr = lambda k, *s: np.stack([np.array(w[k], np.float32).reshape(s) for w in worlds])  # noqa: E731
    print(f"[gpu] rollout gradients of {nw} quadrupeds at a row switch", flush=True)
    w = mjh.World(ctx, m, nw, qpos=arr("qpos", m.nq))
    w.batch.set_launch(0, 32, 128)
    v = torch.tensor(arr("qvel", m.nv), device="cuda", requires_grad=True)
    u = torch.tensor(arr("ctrl", H, m.nu).transpose(1, 0, 2).copy(), device="cuda",
                     requires_grad=True)
    loss = mjh.Rollout.apply(v, u, w, H, 2)
    gv, gu = torch.autograd.grad(loss, (v, u), torch.tensor(arr("dloss"), device="cuda"))
    for k, x in enumerate(worlds):
        for name, got in (("loss", loss[k]), ("dqvel", gv[k]), ("dctrl", gu[:, k])):
            want = np.array(x[name], np.float32).ravel()
            err = np.linalg.norm(got.detach().cpu().numpy().ravel() - want) / np.linalg.norm(want)
            assert err <= 2e-5, (k, name, err)
