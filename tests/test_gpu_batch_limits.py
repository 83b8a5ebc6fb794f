"""Batched launches whose wavefronts hold friction-limited and never-limited
samples up to a limit: horizons on both remainders of two blocks, command
switches and steps that differ between scenarios, perception.  Every scenario
equals its launch alone bit for bit and takes no step past its horizon, through
the batched call, a recorded batch and a recorded mix."""
import numpy as np
import pytest

from paper_2604_27193_amd import workloads as W
from test_gpu_parity import to_np

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    import torch
    assert torch.cuda.is_available()
    from paper_2604_27193_amd import binding
    binding.lib()
    return binding


# both friction classes, and too short for split speeds
MIXED = {"mu": ("uniform", 0.35, 1.0), "v0": ("trunc_normal", 18.0, 1.0, 15.0, 21.0)}
SIZES = (32, 65, 129, 200, 1031)


def scns(base, overs):
    return [dict(base(SIZES[j % len(SIZES)], seed=21, scenario_id=j), **{**MIXED, **o})
            for j, o in enumerate(overs)]


BATCHES = {
    "horizons": scns(W.single, [{"horizon": (1300 + 64 * j) * 1e-3} for j in range(8)]),
    "one_horizon_odd": scns(W.single, [{"horizon": 1.5}] * 5),
    "one_horizon_even": scns(W.single, [{"horizon": 1.564}] * 5),
    "commands": scns(W.single, [{"dead_time": t} for t in (0.05, 0.26, 0.34, 0.46, 0.6, 0.75)]),
    "steps": scns(W.single, [{"dt": t, "horizon": 1.5} for t in (0.5e-3, 1e-3, 2e-3)]),
    "perception": scns(W.perception, [{}] * 4),
    "downhill": scns(W.single, [{"horizon": (1500 + 64 * j) * 1e-3, "a_cmd": -2.0,
                                 "mu": ("const", m), "grade": ("const", -0.3)}
                                for j in range(2) for m in (0.15, 0.85)]),
}
OBSTACLES = {"none": {"obstacle": "none"}, "stationary": {}, "exit": {"impact_exit": True},
             "lead": {"obstacle": "lead", "gap": ("normal", 40.0, 3.0),
                      "lead_decel": ("normal", 3.0, 0.5)}}


@pytest.mark.parametrize("prec", ["fp32c", "fp64"])
@pytest.mark.parametrize("obstacle", sorted(OBSTACLES))
@pytest.mark.parametrize("name", sorted(BATCHES))
def test_limits_in_a_batch(B, name, obstacle, prec):
    import torch
    batch = [dict(d, **OBSTACLES[obstacle]) for d in BATCHES[name]]
    got = {"call": [to_np(o) for o in B.batch_rollout(batch, precision=prec)]}
    g = B.Graph(batch, precision=prec, stats=False, batch=True)
    g.launch()
    g.finish()
    got["graph"] = [to_np(o) for o in g.out]
    m = B.MixGraph(batch[0], precision=prec, max_scn=len(batch), max_samples=1 << 13,
                   stats=False)
    outs = m.launch(batch)
    m.finish()
    torch.cuda.synchronize()
    got["mix"] = [to_np(o) for o in outs]
    for j, d in enumerate(batch):
        alone = to_np(B.rollout(d, precision=prec))
        assert int(alone["steps"].max()) <= round(d["horizon"] / d["dt"])
        for route, sets in got.items():
            for k in alone:
                assert np.array_equal(sets[j][k], alone[k]), (route, j, k)
