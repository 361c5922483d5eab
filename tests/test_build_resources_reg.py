"""Register and scratch budget of the kernels that the default shapes launch: the
register-resident step and env kernels, the mixed-batch kernel and the rollouts, from the
compiler's resource-usage report of the last build (no GPU).

Rows of up to 20 entries run four waves per SIMD at 128 VGPRs and spill a few registers; rows
of 28 run two waves and spill none.  The env kernel keeps its observation and reward terms over
the physics steps and spills 53 (61 with randomised dynamics) VGPRs, the reverse rollout 91.
The bounds are today's figures: more is a regression to look at.
"""
import pytest

from paper_2502_08844_amd import build

STEP = "_ZN3mjh19mjh_step_reg_kernelILi{}ELi{}ELb{}EEEvPKNS_8DevGroupEPKNS_7DevTaskEi"
ENV = "_ZN3mjh18mjh_env_reg_kernelILb{}EEEvPKNS_8DevGroupEPKNS_7DevTaskENS_7EnvArgsEii"
MIX = "_ZN3mjh19mjh_step_mix_kernelEPKNS_8DevGroupEPKNS_7DevTaskEi"
FWD = "_ZN3mjh18rollout_fwd_kernelENS_11RolloutArgsE"
BWD = "_ZN3mjh18rollout_bwd_kernelENS_11RolloutArgsE"

# kernel: waves per SIMD, scratch bytes a lane, spilled VGPRs (lanes, row length, Runge-Kutta)
BUDGET = {
    STEP.format(16, 16, 0): (4, 32, 5), STEP.format(16, 16, 1): (4, 36, 6),
    STEP.format(32, 16, 0): (4, 40, 7), STEP.format(32, 16, 1): (4, 36, 6),
    STEP.format(32, 20, 0): (4, 72, 18), STEP.format(32, 20, 1): (4, 72, 17),
    STEP.format(64, 20, 0): (4, 60, 14), STEP.format(64, 20, 1): (4, 64, 14),
    STEP.format(32, 28, 0): (3, 12, 0), STEP.format(32, 28, 1): (3, 12, 0),
    STEP.format(64, 28, 0): (2, 12, 0), STEP.format(64, 28, 1): (2, 12, 0),
    MIX: (2, 12, 0),
    ENV.format(0): (4, 204, 53), ENV.format(1): (4, 236, 61),
    FWD: (2, 156, 0), BWD: (1, 560, 91),
}


@pytest.fixture(scope="module")
def usage():
    u = build.resource_usage()
    if u is None:
        pytest.skip("no build report yet (run the build first)")
    return u


@pytest.mark.parametrize("kernel", BUDGET)
def test_launched_kernels_stay_within_budget(usage, kernel):
    waves, scratch, spills = BUDGET[kernel]
    k = usage[kernel]
    assert k["Occupancy"] >= waves, k
    assert k["ScratchSize"] <= scratch, k
    assert k["VGPRsSpill"] <= spills, k


def test_every_register_kernel_has_a_budget(usage):
    for kernel in usage:
        if "_reg_kernel" in kernel or "_mix_kernel" in kernel or "rollout_" in kernel:
            assert kernel in BUDGET, kernel
