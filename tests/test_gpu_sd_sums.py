"""The single-dish beam sums at the edges of their split over lanes (GPU): sample counts that are not multiples of
a block's, beams shorter than the split, longer than the image, and cut off by its border.  Against
the FP64 oracle at the float build's bound for one evaluation (1e-5)."""
import numpy as np
import pytest
import torch

import oracle
import synth
from paper_2609_17636_amd import Plan

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_sd,stride,fwhm_pix", [(1, 32, 3.0), (3, 9, 0.5), (5, 6, 2.0), (16, 2, 4.0), (7, 4, 40.0),
                                                  (32, 1, 12.0)])
@pytest.mark.parametrize("precision", ["f32", "f64"])
def test_sd_sums(n_sd, stride, fwhm_pix, precision):
    p = oracle.synthesize(synth.single_pointing("sd", 3, 32, 20.0, 1, 300, "points", 1e-3, ("abs", 0.01)))
    rng = np.random.default_rng(n_sd)
    p.sd_n, p.sd_stride, p.sd_offset = n_sd, stride, min(1, 31 - (n_sd - 1) * stride)
    p.sd_fwhm_rad = fwhm_pix * p.pixel_rad
    p.sd_sigma, p.lambda_s = 0.5, 2.0
    p.sd_map = rng.uniform(0, 1, (p.n_chan, n_sd, n_sd)).astype(np.float32)
    x = rng.uniform(0, 1, (1, 32, 32))
    want_t, want_g = oracle.objective_grad(p, x)
    plan = Plan.from_problem(p, precision=precision)
    plan.set_problem_data(p)
    terms, grad = plan.objective_grad(torch.tensor(x, dtype=plan.torch_dtype, device="cuda"))
    tol = 1e-5 if precision == "f32" else 1e-9
    assert abs(terms[0] - want_t["Q_tot"]) <= tol * want_t["Q_tot"]
    assert np.linalg.norm(grad.double().cpu().numpy() - want_g) <= tol * np.linalg.norm(want_g)


@pytest.mark.parametrize("n_sky,n_sd,stride", [(600, 600, 1), (560, 280, 2)])
def test_sd_sums_of_large_maps(n_sky, n_sd, stride):
    """More samples than the blocks of a launch take at once, one lane a sample and eight."""
    p = oracle.synthesize(synth.single_pointing("sd", 3, n_sky, 20.0, 1, 50, "points", 1e-3, ("abs", 0.01)))
    rng = np.random.default_rng(n_sd)
    p.sd_n, p.sd_stride, p.sd_offset = n_sd, stride, 0
    p.sd_fwhm_rad = 6.0 * p.pixel_rad
    p.sd_sigma, p.lambda_s = 0.5, 2.0
    p.sd_map = rng.uniform(0, 1, (p.n_chan, n_sd, n_sd)).astype(np.float32)
    x = rng.uniform(0, 1, (1, n_sky, n_sky))
    want_t, want_g = oracle.objective_grad(p, x)
    for precision, tol in (("f32", 1e-5), ("f64", 1e-9)):
        plan = Plan.from_problem(p, precision=precision)
        plan.set_problem_data(p)
        terms, grad = plan.objective_grad(torch.tensor(x, dtype=plan.torch_dtype, device="cuda"))
        assert abs(terms[0] - want_t["Q_tot"]) <= tol * want_t["Q_tot"]
        assert np.linalg.norm(grad.double().cpu().numpy() - want_g) <= tol * np.linalg.norm(want_g)
