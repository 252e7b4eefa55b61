"""The mosaic combination at the edges of its loads (GPU) against the oracle: pointing and channel counts
around the groups that are loaded together, positions on and beside every edge of the sub-image, NaN
positions (outside, as any other), and image pixels of no weight that hold NaN.

All data are positive and exact in FP32, so the error is relative: at most about 10 roundings a sample and one
an addition, (P + 16) 2^-23 for the quotient.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import dataproc as D  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("P,C,n,N", [(1, 1, 4, 8), (3, 3, 5, 16), (4, 4, 16, 24), (5, 17, 7, 16), (9, 8, 33, 40)])
@pytest.mark.parametrize("precision", ["f32", "f64"])
def test_linear_mosaic_edges(P, C, n, N, precision):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2609_17636_amd import dataproc as G

    dt = torch.float32 if precision == "f32" else torch.float64
    rng = np.random.default_rng(P * 100 + C)
    pos = rng.uniform(-2, n + 1, (P, N, N, 2))
    edges = np.array([-1.0, -0.75, -0.5, 0.0, 0.5, n - 2.0, n - 1.5, n - 1.0, n - 0.5, n - 0.25, n])
    pick = rng.random(pos.shape) < 0.5
    pos[pick] = rng.choice(edges, size=int(pick.sum()))
    pos = pos.astype(np.float32).astype(np.float64)
    sub = rng.uniform(1, 2, (P, C, n, n)).astype(np.float32).astype(np.float64)
    beams = rng.uniform(0.25, 1, (P, n, n)).astype(np.float32).astype(np.float64)
    lost = rng.random((P, N, N)) < 0.1
    gone, at = pos.copy(), pos.copy()
    gone[lost], at[lost] = -10.0, np.nan
    want, peff = D.linear_mosaic(sub, beams, gone, pb_min=0.3)
    # a pixel that no position gives weight to may hold anything
    used = np.zeros((P, n + 2, n + 2), bool)
    for k in range(P):
        r, c = gone[k, ..., 0].ravel(), gone[k, ..., 1].ravel()
        in_ = (r > -1) & (r < n) & (c > -1) & (c < n)
        i, j = np.floor(r[in_]).astype(int) + 1, np.floor(c[in_]).astype(int) + 1
        for di in (0, 1):
            for dj in (0, 1):
                used[k, i + di, j + dj] = True
    sub[np.broadcast_to(~used[:, None, 1:-1, 1:-1], sub.shape)] = np.nan
    t = [torch.tensor(a, dtype=dt, device="cuda") for a in (sub, beams, at)]
    img, pb = G.linear_mosaic(*t, pb_min=0.3)
    # (a quotient within rounding of pb_min may fall on either side)
    clear = np.abs(peff - 0.3) > 1e-5
    tol = (P + 16) * (2.0 ** -23 if precision == "f32" else 2.0 ** -52)
    np.testing.assert_allclose(img.double().cpu().numpy()[:, clear], want[:, clear], rtol=tol, atol=0)
    np.testing.assert_allclose(pb.double().cpu().numpy(), peff, rtol=tol, atol=0)
