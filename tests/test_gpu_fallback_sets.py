"""The radix-select fallback over several sets of one batch: more sets than one
launch sequence takes, of uneven sizes, censored distances among them, each
against the reference's sort-based statistics."""
import numpy as np
import pytest

from test_gpu_parity import compare_stats, upload
from test_gpu_reduce_batch import tied

pytestmark = pytest.mark.gpu

RISK = (0.5, 0.2, 0.01)
MQ = (0.02, 0.5)
GRID = (20.0, 100.0, 33)


@pytest.fixture(scope="module")
def B():
    import torch
    assert torch.cuda.is_available()
    from paper_2604_27193_amd import binding
    binding.lib()
    return binding


def many(j):
    """Set j: a crowded value bin, ties at the margin's low end for every third
    set (collisions share one margin), some distances censored."""
    rng = np.random.default_rng(100 + j)
    n = int(rng.integers(20_000, 60_000))
    s = tied(n, 9_000 + 500 * j, seed=j)
    if j % 3 == 0:
        s["margin"] = np.where(rng.uniform(size=n) < 0.6, -0.001 * rng.uniform(size=n),
                               rng.uniform(0.0, 50.0, n))
    s["status"] = np.where(rng.uniform(size=n) < 0.05, 3, s["status"]).astype(np.uint8)
    return s


@pytest.mark.parametrize("count", [1, 16, 17, 35])
def test_many_fallback_sets(B, orc, count):
    sets = [many(j) for j in range(count)]
    devs = [upload(s) for s in sets]
    small = upload(tied(5_000, 10, seed=3))  # takes none
    before = B.reduce_fallbacks()
    got = B.batch_reduce(devs[:1] + [small] + devs[1:], risk=RISK, margin_q=MQ, grid=GRID)
    assert B.reduce_fallbacks() == before + count
    for s, g in zip(sets, got[:1] + got[2:]):
        compare_stats(g, orc.reduce(s, risk=RISK, margin_q=MQ, grid=GRID))
