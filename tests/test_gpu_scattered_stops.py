"""Rollouts whose lanes stop far apart inside a wavefront, and lanes whose speed
does not only fall: the block ladder runs past stops inside a block and finds
them by replay where a lane's speed can only fall, and steps with every test
elsewhere.  FP64 with host-drawn parameters equals the reference bit for bit."""
import numpy as np
import pytest

from paper_2604_27193_amd import workloads as W
from test_gpu_parity import check_fp32c, check_fp64, plain, to_np, upload

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    import torch
    assert torch.cuda.is_available()
    from paper_2604_27193_amd import binding
    binding.lib()
    return binding


# speeds from below zero to 50 m/s and frictions from ice up: the stops of one
# wavefront spread over the whole run
WIDE = {"v0": ("normal", 20.0, 12.0), "mu": ("uniform", 0.08, 1.2), "gap": ("normal", 30.0, 25.0)}
VARIANTS = {
    "wide": WIDE,
    "wide_exit": dict(WIDE, impact_exit=True),
    "wide_none": dict(WIDE, obstacle="none"),
    "wide_unfused": dict(WIDE, nofma=True),
    "wide_lead": dict(WIDE, obstacle="lead", lead_decel=("normal", 3.0, 1.0)),
    # downhill beyond what the brake holds: speeds that rise, or fall and never stop
    "downhill": dict(WIDE, grade=("normal", -0.2, 0.15), a_cmd=-2.0),
    # stops in the dead time (uphill) and speeds that rise through it (downhill)
    "late_command": dict(WIDE, grade=("normal", 0.0, 0.2), dead_time=2.5,
                         v0=("normal", 4.0, 3.0)),
    # a command that pulls forward
    "pushing": dict(WIDE, a_cmd=0.5),
    "short_horizon": dict(WIDE, horizon=1.237),
    "rk4": dict(WIDE, integrator="rk4"),
    "rk4_exit": dict(WIDE, integrator="rk4", impact_exit=True),
    # a step of several actuator time constants: outside the falling rule
    "rk4_stiff": dict(WIDE, integrator="rk4", dt=5e-3, tau=("uniform", 0.002, 0.02)),
    "control": dict(WIDE, gap=("normal", 60.0, 30.0), ctl_period=0.05, ttc_warn=3.0,
                    ttc_brake=2.0, a_warn=-3.0, noise_gap=0.5, noise_v=0.3),
    "perception": dict(WIDE, latency=("uniform", 0.0, 1.0)),
}


@pytest.mark.parametrize("n", [1, 63, 65, 1031])
@pytest.mark.parametrize("name", sorted(VARIANTS))
def test_scattered_stops_fp64(B, orc, name, n):
    d = W.single(n, seed=11, scenario_id=n, **VARIANTS[name])
    assert B.validate(d) == 0
    check_fp64(to_np(plain(B, d)), orc.run(d), exact=True)


@pytest.mark.parametrize("seed", range(4))
def test_stiff_rk4_forms(B, orc, seed):
    """Steps of up to 2.5 actuator time constants: an RK4 stage may leave the
    range between the brake and its command, so neither the never-limited nor
    the limited-for-good form holds, whatever lanes share a wavefront."""
    d = W.single(1031, seed=seed, **VARIANTS["rk4_stiff"])
    check_fp64(to_np(plain(B, d)), orc.run(d), exact=True)


def test_stop_and_crossing_in_one_block(B, orc):
    """Obstacles placed at the samples' own stopping distances, so that a lane
    passes the obstacle in the block it stops in, or just fails to."""
    d = W.single(2048, seed=5, **dict(WIDE, v0=("uniform", 1.0, 40.0)))
    cols = B.sample_params(d, device=False)
    free = orc.run(dict(d, obstacle="none"))
    cols["gap"][:] = free["dist"] + np.linspace(-0.02, 0.001, d["n_samples"])
    ref = orc.rollout_given(d, cols)
    hit = (ref["status"] & 4) != 0
    assert hit.any() and (~hit).any()
    for over in ({}, {"impact_exit": True}):
        d2 = dict(d, **over)
        check_fp64(to_np(B.rollout(d2, params=upload(cols))), orc.rollout_given(d2, cols),
                   exact=True)


@pytest.mark.parametrize("n", [65, 1031])
@pytest.mark.parametrize("name", ["wide", "wide_exit", "wide_none"])
def test_scattered_stops_fp32c(B, orc, name, n):
    """The compensated form on the same scattered stops, speeds split into base
    and increment (long rollouts) and whole in one wavefront."""
    d = W.single(n, seed=11, scenario_id=n, **VARIANTS[name])
    check_fp32c(to_np(B.rollout(d, precision="fp32c")), orc.run(d))


@pytest.mark.parametrize("name", ["wide", "wide_exit", "wide_none", "downhill", "late_command",
                                  "short_horizon", "perception"])
def test_grouping_does_not_change_bits_fp32c(B, name):
    """A sample's result does not depend on its wavefront: every sample of a
    launch equals the same sample in a launch of its own 64."""
    d = W.single(1031, seed=12, **VARIANTS[name])
    cols = B.sample_params(d, device=False)
    whole = to_np(B.rollout(d, params=upload(cols), precision="fp32c"))
    for a in range(0, 1031, 64):
        part = {k: v[a:a + 64] for k, v in cols.items()}
        got = to_np(B.rollout(dict(d, n_samples=len(part["v0"])), params=upload(part),
                              precision="fp32c"))
        for k in got:
            assert np.array_equal(got[k], whole[k][a:a + 64]), (k, a)
