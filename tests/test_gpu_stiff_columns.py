"""Columns whose actuator time constants lie on both sides of the step (the draws
of an explicit-Euler scenario keep to one): every kernel gives a sample the same
result whatever samples share its wavefront, and FP64 the reference's."""
import numpy as np
import pytest

from paper_2604_27193_amd import workloads as W
from test_gpu_parity import check_fp64, to_np, upload

pytestmark = pytest.mark.gpu
N = 517


@pytest.fixture(scope="module")
def B():
    import torch
    assert torch.cuda.is_available()
    from paper_2604_27193_amd import binding
    binding.lib()
    return binding


def columns(B, obstacle):
    d = W.single(N, seed=31, horizon=3.0, v0=("uniform", 1.0, 12.0), mu=("uniform", 0.3, 1.0),
                 gap=("uniform", 0.5, 15.0), obstacle=obstacle, lead_decel=("normal", 3.0, 0.5))
    cols = B.sample_params(d, device=False)
    cols["tau"][:] = np.random.default_rng(3).uniform(0.52e-3, 4e-3, N)  # up to 1.9 steps
    return d, cols


@pytest.mark.parametrize("obstacle", ["none", "stationary", "lead"])
@pytest.mark.parametrize("form", ["fp64", "fp64_two_samples", "fp32c"])
def test_stiff_columns(B, orc, form, obstacle):
    if form == "fp64_two_samples" and obstacle == "lead":
        pytest.skip("two samples per lane: no lead vehicle")
    d, cols = columns(B, obstacle)
    prec = "fp32c" if form == "fp32c" else "fp64"
    old = B.tune_get(prec, obstacle)
    try:
        if form == "fp64_two_samples":
            B.tune_set(prec, obstacle, 64, 64, 0, 2)
        whole = to_np(B.rollout(d, params=upload(cols), precision=prec))
        for a in range(0, N, 17):
            part = {k: v[a:a + 17] for k, v in cols.items()}
            got = to_np(B.rollout(dict(d, n_samples=len(part["v0"])), params=upload(part),
                                  precision=prec))
            for k in got:
                assert np.array_equal(got[k], whole[k][a:a + 17]), (k, a)
    finally:
        B.tune_set(prec, obstacle, *old)
    if prec == "fp64":
        check_fp64(whole, orc.rollout_given(d, cols), exact=True)
