"""Work items of the matrix-core gridder that run over several of its batches of 32 records: every sample lies in one
tile, half of them mirrored into it, so an item holds exactly the records that the test counts (GPU).  Value,
gradient, model and adjoint, coplanar and with w planes.  Kernels of 8 cells against the FP64 oracle at
the float build's bound for one evaluation (1e-5).  Narrower ones, whose own error is 2.7e-6 and more (the probe says so),
against the vector gridder, which does the same sums with the same kernel: FP32 rounding, 2e-6 of the norm."""
import numpy as np
import pytest
import torch

import oracle
import synth
from paper_2609_17636_amd import Plan, nufft_probe

pytestmark = pytest.mark.gpu
TOL = 1e-5


def _rel(a, b):
    return float(np.linalg.norm(np.asarray(a) - b) / np.linalg.norm(b))


def _tile_problem(count, w):
    """All footprints start at one cell: fine-grid coordinates in (20, 21) of 64."""
    p = synth.single_pointing("tile", 7, 32, 20.0, max(1, -(-count // 630)), count, "points", 1e-3, ("abs", 0.01), w_term=w)
    rng = np.random.default_rng(count)
    sign = rng.choice([-1.0, 1.0], (count, 1))
    p.uv = (sign * (20.0 + rng.uniform(0.05, 0.95, (count, 2))) / (64 * p.pixel_rad)).astype(np.float32)
    if w:  # in the order of the records: an item is sorted by w
        p.w = np.linspace(1.0, 3.0, count).astype(np.float32)
        p.uv = np.abs(p.uv)
    return oracle.synthesize(p)


def _plan(p, width, blocking):
    plan = Plan.from_problem(p, precision="f32", kernel_width=width, fine_size=64)
    plan.set_blocking(*blocking)
    plan.set_problem_data(p)
    if getattr(p, "w", None) is not None:
        plan.set_w(p.w)
    return plan


def _run(plan, x, y):
    sky = torch.tensor(x, dtype=torch.float32, device="cuda")
    terms, grad = plan.objective_grad(sky)
    v = plan.forward(sky).double().cpu().numpy()
    a = plan.adjoint(torch.tensor(y, device="cuda"))
    return terms[0], grad.double().cpu().numpy(), v[:, 0] + 1j * v[:, 1], a.double().cpu().numpy()


def _check(p, width, blocking, items):
    rng = np.random.default_rng(1)
    x = rng.uniform(0, 1, (1, 32, 32))
    y = (rng.standard_normal((p.n_vis, 2)) * (1 + np.arange(p.n_vis) // 32 % 5)[:, None]).astype(np.float32)
    plan = _plan(p, width, blocking)
    assert plan.info()["n_work_items"] == items and plan.info()["lanes"] == 64
    q, *got = _run(plan, x, y)
    if nufft_probe(32, 64, width) < 0.1 * TOL:
        tol, (terms, g) = TOL, oracle.objective_grad(p, x)
        want_q, want = terms["Q_tot"], [g, oracle.model_vis(p, x), oracle.adjoint_image(p, y[:, 0] + 1j * y[:, 1])]
    else:
        tol, (want_q, *want) = 2e-6, _run(_plan(p, width, (16, 2, 2048, 16, 2)), x, y)
    assert abs(q - want_q) <= tol * abs(want_q)
    for u, v in zip(got, want):
        assert _rel(u, v) <= tol
    return want[1]


@pytest.mark.parametrize("w", [False, True])
@pytest.mark.parametrize("count", [1, 31, 32, 33, 63, 64, 65, 97, 1000])
def test_batches_of_one_item(count, w):
    p = _tile_problem(count, w)
    _check(p, 8, (9, 1, 2048, 64, 1), 1)
    _check(p, 5, (12, 1, 33, 64, 1), -(-count // 33))


@pytest.mark.parametrize("w", [False, True])
@pytest.mark.parametrize("width", [4, 7, 8])
def test_rising_residuals(width, w):
    """Weights rise thirtyfold from batch to batch and fall again: the item's scale is lowered twice, with the window
    accumulated so far, of which the earlier batches are 1e-3 and 3e-2."""
    p = _tile_problem(128, w)
    p.weight = (p.weight * np.repeat([1.0, 30.0, 900.0, 1.0], 32)).astype(np.float32)
    model = _check(p, width, (17 - width, 1, 2048, 64, 1), 1)
    top = np.abs((model - p.vis) * p.weight).reshape(4, 32).max(axis=1)
    assert top[1] > 8 * top[0] and top[2] > 8 * top[1]
