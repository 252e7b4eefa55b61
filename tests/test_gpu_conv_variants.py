"""3x3 convolutions at sizes that take each of their kernels' larger tiles (GPU), against the FP64 layer oracle
on bands of rows: pixels of a wave that run over row and image boundaries, steps that span taps, channels staged in
parts, and the FP32 layers that go to the kernels for any channel count.

Operands are exact in bf16 on both sides, so the difference is the FP32 summation error, at most
K u sum|terms| with K = 9 cin + 2 terms and u = 2^-24.  The network: an activation within FP32 error of a bf16
rounding boundary may round the other way (2^-8 of that operand), so relative L2 differences of 1e-2
forward and 2e-2 per parameter block of the gradient.
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


def _rows(x, w, b, r0, r1):
    """Output rows [r0, r1) of the layer."""
    lo, hi = max(r0 - 1, 0), min(r1 + 1, x.shape[1])
    return U.conv3x3(x[:, lo:hi], w, b)[:, r0 - lo:r1 - lo]


@pytest.mark.parametrize("n,h,w,cin,cout", [
    (1, 363, 365, 24, 16), (1, 363, 365, 32, 16), (3, 211, 215, 16, 48),     # one wave 64 pixels x 16 channels
    (1, 363, 365, 40, 64), (1, 363, 365, 40, 96), (1, 129, 127, 40, 96),     # 64 x 64, 64 x 32, 32 x 32
    (1, 9, 35, 608, 64), (1, 11, 67, 640, 96), (1, 148, 150, 288, 96),       # channels of a patch in parts,
    (2, 148, 150, 288, 64), (1, 182, 184, 416, 128),                         # small and large tiles
    (1, 21, 23, 20, 32), (1, 21, 23, 36, 64), (2, 130, 131, 24, 64), (1, 403, 401, 48, 48)])  # any channel count
def test_conv3x3_variants(nn, n, h, w, cin, cout):
    g = torch.Generator(device="cuda").manual_seed(cin + cout + h)
    x, wt, b = (torch.randn(s, generator=g, device="cuda") for s in ((n, h, w, cin), (cout, 3, 3, cin), (cout,)))
    mask, y0 = (torch.randn((n, h, w, cout), generator=g, device="cuda") for _ in range(2))
    y = nn.conv3x3(x, nn.to_bf16(wt), bias=b, relu=True, mask=mask, accumulate=True, out=y0.clone()).cpu().numpy()
    qx, qw, bb = U.bf16(x.cpu().numpy()), U.bf16(wt.cpu().numpy()), b.cpu().numpy().astype(np.float64)
    on, start = mask.cpu().numpy() > 0, y0.cpu().numpy().astype(np.float64)
    for r0 in sorted({0, max(0, h // 2 - 2), max(0, h - 4)}):
        r1 = min(h, r0 + 4)
        want = np.where(on[:, r0:r1], np.maximum(_rows(qx, qw, bb, r0, r1), 0.0), 0.0) + start[:, r0:r1]
        size = _rows(np.abs(qx), np.abs(qw), np.abs(bb), r0, r1) + np.abs(start[:, r0:r1])
        assert np.all(np.abs(y[:, r0:r1] - want) <= (9 * cin + 2) * U24 * size)


def test_network_of_narrow_layers(nn):
    """16 and 48 input channels (steps span taps, two sources, the first at half resolution) on images of more
    than 131,072 pixels together."""
    levels, base, batch, h, w = 2, 16, 3, 212, 216
    net = nn.UNet(levels=levels, base=base, max_batch=batch, height=h, width=w, seed=3)
    rng = np.random.default_rng(5)
    p = net.get_params()
    p += (rng.standard_normal(p.size) * 0.01).astype(p.dtype)
    net.set_params(p)
    x, t = rng.random((2, batch, h, w)).astype(np.float32)
    x4 = np.zeros((batch, h, w, 4))
    x4[..., 0] = x
    want, _ = U.unet_forward(x4, U.unpack(p.astype(np.float64), levels, base, 4), levels, round_bf16=True)
    y = net.forward(torch.from_numpy(x).cuda()).cpu().numpy()
    assert np.linalg.norm(y - want) <= 1e-2 * np.linalg.norm(want)
    _, g = net.loss_grad(torch.from_numpy(x).cuda(), torch.from_numpy(t).cuda())
    _, wg = U.unet_loss_grad(x4, t, p.astype(np.float64), levels, base, 4, round_bf16=True)
    o = 0
    for name, shp in U.unet_param_shapes(levels, base, 4):
        k = int(np.prod(shp)) if shp else 1
        assert np.linalg.norm(g[o:o + k] - wg[o:o + k]) <= 2e-2 * np.linalg.norm(wg[o:o + k]), name
        o += k


@pytest.mark.parametrize("n,h,w,cin,cout", [
    (1, 128, 128, 64, 32), (1, 127, 128, 32, 32), (1, 33, 31, 256, 248), (1, 16, 16, 136, 512),  # around the choice of kernel,
    (512, 8, 8, 40, 64), (250, 8, 8, 72, 32), (700, 5, 4, 32, 64), (1, 2000, 3, 8, 24),  # half and quarter filled patches,
    (1, 23, 24, 320, 320), (1, 70, 66, 8, 16)])  # few and many partial sums
def test_grad_weight_variants(nn, n, h, w, cin, cout):
    g = torch.Generator(device="cuda").manual_seed(cin + cout + h)
    x, dy = (torch.randn(s, generator=g, device="cuda") for s in ((n, h, w, cin), (n, h, w, cout)))
    dw, db = nn.conv3x3_grad_weight(x, dy)
    qx, qy, f = U.bf16(x.cpu().numpy()), U.bf16(dy.cpu().numpy()), dy.cpu().numpy().astype(np.float64)
    want, size = U.conv3x3_grad_weight(qx, qy)[0], U.conv3x3_grad_weight(np.abs(qx), np.abs(qy))[0]
    P = n * h * w  # products of a weight's sum, and a few additions of partial sums
    assert np.all(np.abs(dw.cpu().numpy() - want) <= (P + 8) * U24 * size + 1e-30)
    assert np.all(np.abs(db.cpu().numpy() - f.sum(axis=(0, 1, 2))) <= (P + 8) * U24 * np.abs(f).sum(axis=(0, 1, 2)))


def test_network_on_very_long_rows(nn):
    """Rows of 12,000,000 pixels, of which four are beyond 32-bit offsets: the same as eight images of an eighth of the
    row whose pixels within reach of a seam are zero.  Activations may round the other way where sums differ in their
    order (2^-9 of a few): 1e-3 of the norm."""
    pieces, w, h = 8, 1500000, 4
    g = torch.Generator(device="cuda").manual_seed(1)
    x, t = (torch.rand((pieces, h, w), generator=g, device="cuda") for _ in range(2))
    for a in (x, t):
        a[:, :, :64] = 0.0
        a[:, :, -64:] = 0.0
    out = []
    for batch in (pieces, 1):
        net = nn.UNet(levels=2, base=16, max_batch=batch, height=h, width=pieces * w // batch, seed=3)
        if batch == 1:
            x, t = (a.transpose(0, 1).reshape(1, h, pieces * w).contiguous() for a in (x, t))
        y = net.forward(x)
        if batch > 1:
            y = y.transpose(0, 1).reshape(1, h, pieces * w)
        loss, grads = net.loss_grad(x, t)
        out.append((y.clone(), loss, torch.as_tensor(grads).double().cpu().numpy()))
        net.close()
    (y0, l0, g0), (y1, l1, g1) = out
    assert float((y1 - y0).norm()) <= 1e-3 * float(y0.norm())
    assert abs(l1 - l0) <= 1e-3 * abs(l0)
    assert np.linalg.norm(g1 - g0) <= 1e-3 * np.linalg.norm(g0)


@pytest.mark.parametrize("cin,cout", [(256, 128), (640, 96), (40, 64), (24, 32)])
def test_layers_in_a_captured_graph(nn, cin, cout):
    """Layers whose blocks ask for more than the default LDS among them: every replay gives the eager bits."""
    g = torch.Generator(device="cuda").manual_seed(cin)
    x, wt = torch.randn((2, 40, 36, cin), generator=g, device="cuda"), torch.randn((cout, 3, 3, cin), generator=g, device="cuda")
    wb, y = nn.to_bf16(wt), torch.zeros((2, 40, 36, cout), device="cuda")
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        nn.conv3x3(x, wb, out=y)
    for seed in range(3):
        x.copy_(torch.randn(x.shape, generator=g, device="cuda"))
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(y, nn.conv3x3(x, wb))
