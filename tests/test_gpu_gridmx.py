"""The matrix-core gridder at the sizes where it can go wrong: work items of one visibility and
around its batches of 32, and data whose magnitudes span many powers of two (its factors are
split into half-precision parts under scales chosen per window and per work item)."""
import numpy as np
import pytest
import torch

import oracle
import synth
from paper_2609_17636_amd import Plan

pytestmark = pytest.mark.gpu
# relative bounds of the float build (single evaluations against the FP64 oracle)
TOL = 1e-5


def _rel(a, b):
    return float(np.linalg.norm(np.asarray(a) - b) / np.linalg.norm(b))


def _problem(count, seed=7):
    p = synth.single_pointing("gridmx", seed, 32, 20.0, max(1, -(-count // 630)), count, "points", 1e-3, ("abs", 0.01))
    return oracle.synthesize(p)


def _check(p, x, blocking):
    plan = Plan.from_problem(p, precision="f32")
    plan.set_blocking(*blocking)
    plan.set_problem_data(p)
    want_t, want_g = oracle.objective_grad(p, x)
    terms, grad = plan.objective_grad(torch.tensor(x, dtype=torch.float32, device="cuda"))
    g = grad.double().cpu().numpy()
    assert abs(terms[0] - want_t["Q_tot"]) <= TOL * want_t["Q_tot"]
    assert _rel(g, want_g) <= TOL
    v = plan.forward(torch.tensor(x, dtype=torch.float32, device="cuda")).double().cpu().numpy()
    mv = oracle.model_vis(p, x)
    assert _rel(v[:, 0] + 1j * v[:, 1], mv) <= TOL


@pytest.mark.parametrize("count", [1, 2, 31, 32, 33, 63, 64, 65, 1000])
def test_batch_remainders(count):
    """Work items of one visibility up to several batches, chunks that end within a batch."""
    x = np.random.default_rng(1).uniform(0, 1, (1, 32, 32))
    p = _problem(count)
    for chunk in (16, 33, 512):
        _check(p, x, (9, 1, chunk, 64, 1))


@pytest.mark.parametrize("sky,weight", [(1e-12, 1.0), (1e12, 1e-20), (1e-3, 1e25), (1.0, 1e-30)])
def test_scales(sky, weight):
    """Skies, data and weights far from one: every scale is a power of two and exact."""
    rng = np.random.default_rng(2)
    p = _problem(700)
    x = np.abs(rng.standard_normal((1, 32, 32))) * sky
    p.vis = (p.vis * sky).astype(np.complex64)
    p.weight = (p.weight * weight).astype(np.float32)
    p.lambda_r = float(1e-3 * p.weight[0])
    _check(p, x, (9, 1, 256, 64, 1))


def test_mixed_weights():
    """Weights over eight decades in shuffled order: the work item's scale is set by its early
    records and lowered, with the accumulated window, when a later batch exceeds it."""
    rng = np.random.default_rng(3)
    p = _problem(2000)
    p.weight = (10.0 ** rng.uniform(-4, 4, p.n_vis)).astype(np.float32)
    p.weight[:64] = 1e-6
    x = np.abs(rng.standard_normal((1, 32, 32)))
    _check(p, x, (9, 1, 2048, 64, 1))


def test_zero_residual_and_zero_sky():
    """Nothing to spread: a zero sky with zero data gives a zero gradient and a zero objective."""
    p = _problem(100)
    p.vis = np.zeros(p.n_vis, np.complex64)
    plan = Plan.from_problem(p, precision="f32")
    plan.set_blocking(9, 1, 64, 64, 1)
    plan.set_problem_data(p)
    terms, grad = plan.objective_grad(torch.zeros((1, 32, 32), dtype=torch.float32, device="cuda"))
    assert terms[0] == 0.0 and float(grad.abs().max()) == 0.0


def test_more_records_in_a_tile_than_32_bit_offsets_reach():
    """2^29 + 100,000 visibilities of one tile under a chunk that would take them all: the last ones are their own."""
    n, count, pix = 16, (1 << 29) + 100000, 1e-4
    g = torch.Generator(device="cuda").manual_seed(1)
    uv = torch.rand((count, 2), generator=g, device="cuda").mul_(2.0).add_(1000.0)
    plan = Plan(1, n, pix, 1, n, [0, count], [1.0], kernel_width=8, fine_size=64)
    plan.set_blocking(9, 1, 1 << 30, 64, 1)
    i = torch.arange(n, device="cuda", dtype=torch.float32)
    grid = torch.stack(torch.meshgrid(i, i, indexing="ij"), dim=-1)[None]
    vis, weight = torch.zeros((count, 2), device="cuda"), torch.ones(count, device="cuda")
    plan.set_data(uv, vis, weight, torch.ones((1, n, n), device="cuda"), grid)
    del vis, weight
    torch.cuda.empty_cache()
    assert plan.info()["n_work_items"] == 3
    x = torch.zeros((1, n, n), device="cuda")
    x[0, 2, 3] = 1.0  # direction cosines (3 - 8, 2 - 8) pix
    v = plan.forward(x)
    for s in (slice(0, 100000), slice(count - 100000, count)):
        ph = -2.0 * np.pi * pix * (uv[s].double() @ torch.tensor([-5.0, -6.0], dtype=torch.float64, device="cuda"))
        want = torch.stack([torch.cos(ph), torch.sin(ph)], dim=1)
        assert float((v[s].double() - want).abs().max()) <= TOL * 10  # (of single values, not of a norm)


def test_occupancy_setting_keeps_the_captured_evaluation():
    """One build serves every setting: nothing of the plan changes with it."""
    p = _problem(500)
    plan = Plan.from_problem(p, precision="f32")
    plan.set_problem_data(p)
    x = torch.rand((1, 32, 32), device="cuda")
    grad = torch.empty_like(x)
    terms, _ = plan.objective_grad(x, grad=grad)
    want, nodes = grad.clone(), plan.info()["graph_nodes"]
    assert nodes > 0
    for waves in (6, 7, 0):
        plan.set_gridder_occupancy(waves)
        assert plan.info()["graph_nodes"] == nodes
        assert np.array_equal(plan.objective_grad(x, grad=grad)[0], terms) and torch.equal(grad, want)
