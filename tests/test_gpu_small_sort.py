"""Launch sizes around the one-workgroup sort (up to 32,768 keys, 1,024 at a
time, 8 or 32 a thread, placed 16,384 or 32,768 at a time): FP64 with host-drawn parameters equals the reference bit for bit, drawn
samples equal the same samples given as columns, a batch equals its scenarios one
by one."""
import numpy as np
import pytest

from paper_2604_27193_amd import workloads as W
from test_gpu_parity import check_fp64, plain, to_np, upload

pytestmark = pytest.mark.gpu

SIZES = [1, 63, 1023, 1024, 1025, 8192, 8193, 16384, 16385, 32767, 32768, 32769]


@pytest.fixture(scope="module")
def B():
    import torch
    assert torch.cuda.is_available()
    from paper_2604_27193_amd import binding
    binding.lib()
    return binding


def same(a, b):
    for k in a:
        assert np.array_equal(a[k], b[k], equal_nan=a[k].dtype.kind == "f"), k


@pytest.mark.parametrize("n", SIZES)
def test_given_columns(B, orc, n):
    d = W.single(n, seed=31, scenario_id=n, horizon=1.5)
    check_fp64(to_np(plain(B, d)), orc.run(d), exact=True)


@pytest.mark.parametrize("n", SIZES)
@pytest.mark.parametrize("make", [W.single, W.closed_loop])
def test_drawn(B, make, n):
    d = make(n, seed=31, scenario_id=n, horizon=2.5)
    same(to_np(B.rollout(d)), to_np(B.rollout(d, params=B.sample_params(d))))


@pytest.mark.parametrize("total", [1024, 32767, 32768, 32769])
def test_batch(B, total):
    ds = [W.single(m, seed=32, scenario_id=j, horizon=1.5)
          for j, m in enumerate([1, 700, total - 701])]
    for d, o in zip(ds, B.batch_rollout(ds)):
        same(to_np(o), to_np(B.rollout(d)))
