"""The adjoint's extended grid from the per-tile windows (GPU): one slot a tile and many, tiles of both gridders, grids
whose rows and columns end within a wave or a tile.  The fused fold sums the same windows in the same
order inside the column pass, so the two gradients agree to the rounding of the passes around them."""
import numpy as np
import pytest
import torch

import oracle
import synth
from paper_2609_17636_amd import Plan

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_sub,width,blocking", [
    (32, 4, (13, 1, 4096, 64, 1)), (32, 8, (9, 1, 16, 64, 1)), (90, 7, (10, 1, 512, 64, 1)), (90, 6, (11, 1, 32, 64, 1)),
    (90, 8, (24, 2, 64, 16, 2)), (400, 7, (10, 1, 512, 64, 1)), (400, 8, (16, 2, 16, 16, 2))])
def test_fold(n_sub, width, blocking):
    p = oracle.synthesize(synth.single_pointing("fold", 5, n_sub, 20.0, 3, 1800, "points", 1e-3, ("abs", 0.01)))
    plan = Plan.from_problem(p, precision="f32", kernel_width=width)
    plan.set_blocking(*blocking)
    plan.set_problem_data(p)
    x = torch.tensor(np.random.default_rng(1).uniform(0, 1, p.x_true.shape), dtype=torch.float32, device="cuda")
    out = []
    for fused in (0, 2):
        plan.set_fused_fold(fused)
        out.append(plan.objective_grad(x)[1].double())
    assert float((out[0] - out[1]).norm()) <= 1e-6 * float(out[1].norm())
