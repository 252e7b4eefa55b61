"""Value and gradient over the fine-grid sizes at which the row and column passes take one or the other form
of the in-LDS transform (GPU, both builds, fold inside and outside the column pass), against the FP64
oracle at the single-evaluation bounds of each build: 1e-5 and 1e-10."""
import numpy as np
import pytest
import torch

import oracle
import synth
from paper_2609_17636_amd import Plan

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_sub", [32, 60, 128, 250, 500, 1000])
def test_transform_sizes(n_sub):
    p = oracle.synthesize(synth.single_pointing("fft", 3, n_sub, 20.0, 1, 200, "points", 1e-3, ("abs", 0.01)))
    x = np.random.default_rng(1).uniform(0, 1, p.x_true.shape)
    want, g = oracle.objective_grad(p, x)
    for precision, tol in (("f32", 1e-5), ("f64", 1e-10)):
        plan = Plan.from_problem(p, precision=precision)
        plan.set_problem_data(p)
        for fused in (0, 2):
            plan.set_fused_fold(fused)
            terms, grad = plan.objective_grad(torch.tensor(x, dtype=plan.torch_dtype, device="cuda"))
            assert abs(terms[0] - want["Q_tot"]) <= tol * want["Q_tot"]
            assert np.linalg.norm(grad.double().cpu().numpy() - g) <= tol * np.linalg.norm(g)
        plan.close()
