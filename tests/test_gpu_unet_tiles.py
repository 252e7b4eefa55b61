"""Convolution kernels of the warm-start network at the edges of their tiles (GPU), against the FP64 layer
oracle: images smaller than a tile and with ragged last tiles, channel counts on both sides of each
choice of kernel, networks whose decoder reads two sources and whose weights are kept by steps.

Single layers: bf16 operands are exact on both sides, so the difference is the FP32 summation error,
at most K u sum|terms| with K = 9 cin products and u = 2^-24.  Networks: an activation within FP32 error
of a bf16 rounding boundary may round the other way (2^-8 of that operand), so relative L2 differences
of 1e-2 forward and 2e-2 per parameter block of the gradient, far below the O(1) of a wrong index.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import unet as U  # noqa: E402

pytestmark = pytest.mark.gpu

U24 = 2.0 ** -24


@pytest.fixture(scope="module")
def nn():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2609_17636_amd import unet

    return unet


def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).cuda()


@pytest.mark.parametrize("n,h,w,cin,cout", [
    (1, 1, 1, 8, 16), (2, 3, 5, 24, 48), (1, 5, 17, 40, 64),          # a 32-wide step spans taps
    (1, 1, 1, 32, 32), (2, 7, 33, 32, 96), (1, 9, 31, 96, 32),        # 32 channels a block, few rows
    (1, 3, 65, 160, 128), (3, 2, 2, 64, 64),                          # 64 channels a block
    (1, 4, 5, 608, 64), (1, 3, 4, 608, 16),                           # more channels than a patch holds
    (1, 257, 259, 32, 32), (1, 255, 263, 32, 64), (1, 181, 183, 32, 128)])  # large tiles, ragged
def test_conv3x3_tiles(nn, n, h, w, cin, cout):
    rng = np.random.default_rng(7 * cin + cout + h)
    x = rng.standard_normal((n, h, w, cin)).astype(np.float32)
    wt = (rng.standard_normal((cout, 3, 3, cin)) * 0.3).astype(np.float32)
    b = rng.standard_normal(cout).astype(np.float32)
    wb = nn.to_bf16(_dev(wt))
    y = nn.conv3x3(_dev(x), wb, bias=_dev(b))
    qx, qw = U.bf16(x), U.bf16(wt)
    want = U.conv3x3(qx, qw, b, relu=False)
    bound = 9 * cin * U24 * (U.conv3x3(np.abs(qx), np.abs(qw)) + np.abs(b)) + 1e-30
    assert np.all(np.abs(y.cpu().numpy() - want) <= bound)
    # operands that start at odd elements: the same bits
    xo = torch.empty(x.size + 1, device="cuda")[1:].view(x.shape).copy_(_dev(x))
    wo = torch.empty(wt.size + 1, dtype=wb.dtype, device="cuda")[1:].view(wb.shape).copy_(wb)
    assert torch.equal(nn.conv3x3(xo, wo, bias=_dev(b)), y)


@pytest.mark.parametrize("levels,base,batch,h,w", [(1, 16, 1, 5, 7), (2, 64, 1, 22, 38), (3, 32, 3, 20, 68),
                                                   (2, 48, 2, 34, 18)])
def test_network_tiles(nn, levels, base, batch, h, w):
    net = nn.UNet(levels=levels, base=base, max_batch=batch, height=h, width=w, seed=3)
    rng = np.random.default_rng(levels + base)
    p = net.get_params()
    p += (rng.standard_normal(p.size) * 0.01).astype(p.dtype)  # (the biases start at zero)
    net.set_params(p)
    x, t = rng.random((2, batch, h, w)).astype(np.float32)
    x4 = np.zeros((batch, h, w, 4))
    x4[..., 0] = x
    want, _ = U.unet_forward(x4, U.unpack(p.astype(np.float64), levels, base, 4), levels, round_bf16=True)
    y = net.forward(_dev(x)).cpu().numpy()
    assert np.linalg.norm(y - want) <= 1e-2 * np.linalg.norm(want)
    _, g = net.loss_grad(_dev(x), _dev(t))
    _, wg = U.unet_loss_grad(x4, t, p.astype(np.float64), levels, base, 4, round_bf16=True)
    o = 0
    for name, shp in U.unet_param_shapes(levels, base, 4):
        k = int(np.prod(shp)) if shp else 1
        assert np.linalg.norm(g[o:o + k] - wg[o:o + k]) <= 2e-2 * np.linalg.norm(wg[o:o + k]), name
        o += k


@pytest.mark.parametrize("n,h,w,cin,cout", [(1, 1, 1, 40, 64), (2, 5, 17, 64, 64), (1, 9, 31, 72, 128), (3, 4, 16, 40, 96),
                                            (1, 13, 19, 32, 64), (2, 6, 7, 8, 24)])
def test_conv3x3_grad_weight_tiles(nn, n, h, w, cin, cout):
    rng = np.random.default_rng(cin + cout + h)
    x = rng.standard_normal((n, h, w, cin)).astype(np.float32)
    dy = rng.standard_normal((n, h, w, cout)).astype(np.float32)
    dw, db = nn.conv3x3_grad_weight(_dev(x), _dev(dy))
    qx, qy = U.bf16(x), U.bf16(dy)
    want = U.conv3x3_grad_weight(qx, qy)[0]
    size = U.conv3x3_grad_weight(np.abs(qx), np.abs(qy))[0]
    P = n * h * w  # products of a weight's sum, and a few additions of partial sums
    assert np.all(np.abs(dw.cpu().numpy() - want) <= (P + 8) * U24 * size + 1e-30)
    s = dy.astype(np.float64).sum(axis=(0, 1, 2))
    assert np.all(np.abs(db.cpu().numpy() - s) <= (P + 8) * U24 * np.abs(dy).sum(axis=(0, 1, 2)))
