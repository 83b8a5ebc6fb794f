"""RK4 with one actuator time constant for all samples: launches of 98,304
samples and more that draw their parameters read the actuator from a table
filled once.  The same samples from columns, which may hold any time constant,
take the plain form: both give the same bits."""
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


N = 98_304
VARIANTS = {
    "preset": {},
    "dead_time": {"dead_time": 0.0537},
    "stationary": {"obstacle": "stationary", "gap": ("normal", 75.0, 10.0)},
    "exit": {"obstacle": "stationary", "gap": ("normal", 75.0, 10.0), "impact_exit": True},
    # stands still after about 330 steps
    "fast_actuator": {"tau": ("const", 0.01)},
    # never stands still: the table runs to the horizon
    "slow_actuator": {"tau": ("const", 2.5), "horizon": 4.003},
    # a step of 2.5 time constants
    "stiff": {"tau": ("const", 0.002), "dt": 5e-3},
    # the command comes at or after the last step
    "late": {"dead_time": 2.0, "horizon": 2.0},
    "never": {"dead_time": 3.0, "horizon": 2.0},
    "weights": {"proposal": {"v0": ("normal", 34.0, 2.0)}},
}


CASES = [(v, N) for v in sorted(VARIANTS)]
CASES += [(v, n) for v in ("preset", "exit") for n in (N - 1, N + 4099)]


@pytest.mark.parametrize("name,n", CASES)
def test_table_equals_plain(B, name, n):
    d = W.paper_preset(n, seed=3, **VARIANTS[name])
    cols = B.sample_params(d, device=True)
    plain = to_np(B.rollout(d, params=cols))
    drawn = to_np(B.rollout(d))
    for k in drawn:
        assert np.array_equal(drawn[k], plain[k], equal_nan=True), k


def test_table_in_graph(B):
    """A recorded launch refills its table at every replay."""
    d = W.paper_preset(N, seed=4)
    eager = to_np(B.rollout(d))
    g = B.Graph(d, stats=False)
    for _ in range(3):
        g.launch()
        g.finish()
        got = to_np(g.out)
        for k in eager:
            assert np.array_equal(got[k], eager[k]), k
