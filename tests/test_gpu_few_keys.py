"""Small launches of few sort keys, whose lanes are counted together: parameters
that do not vary, a horizon that ends every sample (one key per friction class),
and columns that begin constant and go on varying.  FP64 equals the reference bit
for bit, so every sample is placed once."""
import numpy as np
import pytest

from paper_2604_27193_amd import workloads as W
from test_gpu_parity import check_fp64, to_np, upload

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    import torch
    assert torch.cuda.is_available()
    from paper_2604_27193_amd import binding
    binding.lib()
    return binding


def columns(B, d, kind):
    cols = B.sample_params(d, device=False)
    n = d["n_samples"]
    if kind == "one":
        alike = np.arange(n)
    elif kind == "begins_alike":  # the wavefronts' first samples, and every other run of 100
        alike = np.flatnonzero((np.arange(n) < 1024) | (np.arange(n) // 100 % 2 == 0))
    else:
        return cols
    for k in cols:
        cols[k][alike] = cols[k][0]
    return cols


@pytest.mark.parametrize("n", [1, 65, 1000, 1025, 8192, 8193, 20011, 32768])
@pytest.mark.parametrize("kind", ["one", "two", "begins_alike"])
def test_few_keys(B, orc, kind, n):
    d = W.single(n, seed=41, scenario_id=n, horizon=0.6 if kind == "two" else 1.5,
                 v0=("normal", 8.0, 2.0))
    cols = columns(B, d, kind)
    check_fp64(to_np(B.rollout(d, params=upload(cols))), orc.rollout_given(d, cols), exact=True)
