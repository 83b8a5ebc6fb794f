"""Lead-vehicle rollouts around the point where the integration stops carrying
the lead (the ego slower, braking harder, the clearance past its minimum): FP64
with host-drawn parameters equals the reference bit for bit, the compensated form
gives each sample the same bits whatever wavefront it is in."""
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


BASE = {"obstacle": "lead", "gap": ("normal", 40.0, 3.0), "lead_decel": ("normal", 3.0, 0.5)}
VARIANTS = {
    "usual": BASE,
    # the two decelerations nearly equal: gains of either sign and near zero
    "even": dict(BASE, mu=("uniform", 0.30, 0.36), lead_decel=("normal", 3.2, 0.3)),
    # the lead stands before the ego, which then closes again
    "hard_lead": dict(BASE, lead_decel=("uniform", 5.0, 9.0), gap=("uniform", 2.0, 60.0)),
    # a lead that speeds up, or keeps its speed
    "fleeing": dict(BASE, lead_decel=("uniform", -1.0, 0.2)),
    # touching at the start
    "touching": dict(BASE, gap=("normal", 0.0, 0.5)),
    "late": dict(BASE, dead_time=1.7),
    "perception": dict(BASE, latency=("uniform", 0.0, 1.5)),
    "short": dict(BASE, horizon=1.4),
    "fast": dict(BASE, v0=("uniform", 500.0, 1500.0), horizon=3.0),
    "far": dict(BASE, gap=("uniform", 5e4, 2e5)),
    "fine_step": dict(BASE, dt=1e-4, horizon=2.0, tau=("uniform", 0.05, 0.1)),
    "unfused": dict(BASE, nofma=True),
    "hill": dict(BASE, grade=("normal", 0.0, 0.2)),
}


@pytest.mark.parametrize("n", [1, 65, 1031])
@pytest.mark.parametrize("name", sorted(VARIANTS))
def test_lead_fp64(B, orc, name, n):
    d = W.single(n, seed=21, scenario_id=n, **VARIANTS[name])
    ref = orc.run(d)
    got = to_np(plain(B, d))
    check_fp64(got, ref, exact=True)
    assert np.array_equal(got["margin"].view(np.uint64), ref["margin"].view(np.uint64))


@pytest.mark.parametrize("name", sorted(VARIANTS))
def test_lead_grouping_fp32c(B, name):
    d = W.single(1031, seed=22, **VARIANTS[name])
    cols = B.sample_params(d, device=False)
    whole = to_np(B.rollout(d, params=upload(cols), precision="fp32c"))
    for a in range(0, 1031, 64):
        part = {k: v[a:a + 64] for k, v in cols.items()}
        got = to_np(B.rollout(dict(d, n_samples=len(part["v0"])), params=upload(part),
                              precision="fp32c"))
        for k in got:
            assert np.array_equal(got[k], whole[k][a:a + 64]), (k, a)


@pytest.mark.parametrize("name", ["usual", "hard_lead", "late"])
def test_lead_fp32c(B, orc, name):
    d = W.single(4097, seed=23, **VARIANTS[name])
    check_fp32c(to_np(B.rollout(d, precision="fp32c")), orc.run(d))
