"""The blocking a fresh plan starts with (GPU): float plans of up to 8-cell kernels take the matrix-core
gridder, wider ones and double plans the vector gridder.  The two do the same sums with one kernel and one
deapodization, so every entry point agrees with the vector blocking set explicitly to FP32
rounding (2e-6 of the norm: a few 2^-24 per operation of sums that add in quadrature)."""
import numpy as np
import pytest
import torch

import oracle
import synth
from paper_2609_17636_amd import Plan

pytestmark = pytest.mark.gpu


def _rel(a, b):
    return float((a.double() - b.double()).norm() / b.double().norm())


@pytest.fixture(scope="module")
def mini():
    return oracle.synthesize(synth.config_c3_mini())


@pytest.mark.parametrize("width", [4, 5, 6, 7, 8, 9])
def test_default_blocking_agrees_with_the_vector_gridder(mini, width):
    p = mini
    default = Plan.from_problem(p, precision="f32", kernel_width=width)
    vector = Plan.from_problem(p, precision="f32", kernel_width=width)
    vector.set_blocking(16, 2, 96, 16, 2)
    info = default.info()
    assert (info["lanes"] == 64) == (info["kernel_width"] <= 8)
    if info["lanes"] == 64:
        assert info["tile"] + info["kernel_width"] == 17
    rng = np.random.default_rng(width)
    x = torch.tensor(rng.uniform(0, 5, p.x_true.shape), dtype=torch.float32, device="cuda")
    out = []
    for plan in (default, vector):
        plan.set_problem_data(p)
        terms, grad = plan.objective_grad(x)
        model = plan.forward(x)
        out.append((terms, grad, model, plan.adjoint(model)))
    (t0, *a), (t1, *b) = out
    assert np.allclose(t0, t1, rtol=2e-6, atol=0)
    for u, v in zip(a, b):
        assert _rel(u, v) <= 2e-6


def test_double_plans_start_with_the_vector_gridder(mini):
    assert Plan.from_problem(mini, precision="f64").info()["lanes"] == 16
