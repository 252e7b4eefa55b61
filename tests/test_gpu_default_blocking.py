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


@pytest.mark.parametrize("w", [False, True])
def test_a_plan_that_small_tiles_do_not_fit_starts_with_larger_ones(w):
    """The card is filled, in pieces smaller than what the default takes beyond 16-cell tiles, until the default
    does not fit any more."""
    n_sub, points, per = 64, 24, 200000
    rng = np.random.default_rng(1)
    grid = np.stack(np.meshgrid(np.arange(n_sub), np.arange(n_sub), indexing="ij"), axis=-1)
    arr = dict(uv=rng.uniform(-1e4, 1e4, (points * per, 2)), vis=rng.standard_normal((points * per, 2)),
               weight=np.ones(points * per), beams=np.ones((points, n_sub, n_sub)),
               interp=np.broadcast_to(grid, (points, n_sub, n_sub, 2)))
    arr = {k: torch.tensor(np.ascontiguousarray(v, dtype=np.float32), device="cuda") for k, v in arr.items()}
    uvw = torch.tensor(rng.uniform(0, 10, points * per), dtype=torch.float32, device="cuda") if w else None
    x = torch.tensor(rng.uniform(0, 1, (1, n_sub, n_sub)), dtype=torch.float32, device="cuda")

    def plan(blocking=None):
        p = Plan(1, n_sub, 5e-5, points, n_sub, per * np.arange(points + 1), [1.0], kernel_width=8, fine_size=2048)
        if blocking:
            p.set_blocking(*blocking)
        p.set_data(**arr)
        if w:
            p.set_w(uvw)
        return p

    p = plan((16, 4, 256, 16, 2))
    need, want = p.info()["device_bytes"], p.objective_grad(x)
    p.close()
    p = plan()
    more = p.info()["device_bytes"] - need
    assert p.info()["lanes"] == 64 and more > 2 ** 28
    p.close()
    torch.cuda.empty_cache()
    fill = [torch.empty(torch.cuda.mem_get_info()[0] - need - more, dtype=torch.uint8, device="cuda")]
    for _ in range(64):  # (some more than is reported as free can be allocated)
        p = plan()
        if p.info()["lanes"] != 64:
            break
        p.close()
        fill.append(torch.empty(more // 3, dtype=torch.uint8, device="cuda"))
    assert p.info()["lanes"] == 16 and p.info()["device_bytes"] == need
    terms, grad = p.objective_grad(x)
    del fill
    torch.cuda.empty_cache()
    assert np.array_equal(terms, want[0]) and torch.equal(grad, want[1])
