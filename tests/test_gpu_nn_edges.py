"""GPU: the convolution gradients at image sizes around their pixel tiles
(8 x 32 for the weight gradient, 8 x 16 for backward-data) and at every
number of 32-channel slices, layer by layer against the FP64 reference fed
the GPU's own BF16 inputs, weights and output gradients.

Bound: the operands are the same BF16 values and their products are exact in
FP32, so only the FP32 summation differs.  A sum of m terms is off by at most
m 2^-24 of its sum of magnitudes, in practice by about sqrt(m) of that; 1e-4
of the largest value covers the 9 x 256 terms of an input gradient and the
4,000 of a weight gradient used here."""
import numpy as np
import pytest

from oracle import nn_ref as R
from paper_1004_1302_amd import learned as LN

pytestmark = pytest.mark.gpu


def bf16_to_f64(t):
    import torch
    return t.view(torch.bfloat16).to(torch.float64).cpu().numpy()


@pytest.mark.parametrize("levels,n,h,w", [
    ((32,), 1, 1, 1), ((32,), 2, 7, 31), ((32,), 1, 8, 32), ((32,), 1, 9, 33),
    ((32,), 3, 17, 65), ((64,), 1, 9, 15), ((96,), 1, 8, 34), ((128,), 2, 10, 17),
    ((160,), 1, 7, 33), ((256,), 1, 9, 16), ((32, 64), 1, 18, 34), ((64, 96), 1, 16, 66)])
def test_convolution_gradients(levels, n, h, w):
    import torch
    net = LN.UNet(seed=7, levels=levels)
    g = torch.Generator(device="cuda").manual_seed(h * 100 + w)
    x = torch.zeros((n * h * w, LN.CIN), device="cuda")
    x[:, :3] = torch.rand((n * h * w, 3), generator=g, device="cuda")
    gy = torch.randn((n * h * w, LN.CIN), generator=g, device="cuda")
    net.forward(x.reshape(-1), x.to(torch.bfloat16).view(torch.int16).reshape(-1), n, h, w)
    net.backward(gy.reshape(-1))
    torch.cuda.synchronize()
    for k, lay in enumerate(net.layers()):
        inf = net.layer_info(k, n, h, w)
        hh, ww, ci, co = h >> inf.level, w >> inf.level, inf.cin, inf.cout
        P = n * hh * ww
        X = bf16_to_f64(net.tensor(inf.x, P * ci, torch.int16)).reshape(n, hh, ww, ci)
        W = bf16_to_f64(lay.w_bf).reshape(9, ci, co)
        dy = net.tensor(inf.dy, P * co, torch.float32).cpu().numpy().astype(np.float64)
        dy = dy.reshape(n, hh, ww, co)
        if inf.relu:
            y = bf16_to_f64(net.tensor(inf.y, P * co, torch.int16)).reshape(n, hh, ww, co)
            dy = dy * (y > 0)
        dx, dw, _ = R.conv3x3_adjoint(X, W, R.bf16(dy))
        gw = lay.gw.cpu().numpy().astype(np.float64).reshape(9, ci, co)
        gb = lay.gb.cpu().numpy().astype(np.float64)
        assert np.abs(gw - dw).max() <= 1e-4 * np.abs(dw).max(), k
        db = dy.reshape(-1, co).sum(axis=0)
        assert np.abs(gb - db).max() <= 1e-4 * max(np.abs(db).max(), 1e-30), k
        if inf.dx != LN.NONE:
            got = net.tensor(inf.dx, P * ci, torch.float32).cpu().numpy().astype(np.float64)
            assert np.abs(got.reshape(dx.shape) - dx).max() <= 1e-4 * np.abs(dx).max(), k


@pytest.mark.parametrize("ci,co,n,h,w", [
    (32, 32, 57, 33, 65), (32, 64, 30, 31, 63), (32, 96, 24, 16, 97), (64, 32, 35, 33, 65),
    (96, 32, 69, 33, 65), (128, 64, 36, 39, 64), (32, 32, 512, 1, 1)])
@pytest.mark.parametrize("relu,residual", [(True, False), (False, True)])
def test_wide_tiles_equal_small_tiles(ci, co, n, h, w, relu, residual):
    """The convolution in wide pixel tiles (16 x 32, or 8 x 32 for several
    slices) has the sums of the small ones in the same order: outputs that
    are not aligned for the wide kernel's rows take the small one, and both
    give the same bits."""
    import torch
    ops = LN.Ops()
    g = torch.Generator(device="cuda").manual_seed(ci + co + n)
    px = n * h * w

    def bf(*shape):
        return torch.randn(shape, generator=g, device="cuda").to(torch.bfloat16).view(torch.int16)

    x, wf = bf(px, ci), bf(co, 9 * ci)
    bias = torch.randn(co, generator=g, device="cuda")
    res = torch.randn(px * co, generator=g, device="cuda") if residual else None
    got = []
    for shift in (0, 1):
        out_b = torch.zeros(px * co + shift, dtype=torch.int16, device="cuda")[shift:]
        out_f = torch.zeros(px * co + shift, device="cuda")[shift:]
        ops.conv3x3(x, wf, bias, relu, res, out_b, out_f, n, h, w, ci, co)
        got.append((out_b.cpu().numpy(), out_f.cpu().numpy()))
    assert np.array_equal(got[0][0], got[1][0])
    assert np.array_equal(got[0][1], got[1][1])
    assert np.abs(got[0][1]).max() > 0


@pytest.mark.parametrize("h,w,c", [(1, 1, 32), (3, 85, 32), (16, 16, 32), (17, 31, 64), (5, 7, 40),
                                   (5, 7, 12), (5, 7, 3)])
def test_elementwise_kernels_at_ragged_sizes(h, w, c):
    """Tone map, inverse tone map, loss gradient and the pooling adjoint in
    groups of channels equal their definitions in FP32 (elementwise, a few
    roundings each: 1e-6 of the largest value), aligned or not."""
    import torch
    ops = LN.Ops()
    g = torch.Generator(device="cuda").manual_seed(h * w + c)
    img = torch.rand((3, h, w), generator=g, device="cuda") * 5
    for shift in (0, 1):
        def buf(n, dtype=torch.float32):
            return torch.full((n + shift,), 7, dtype=dtype, device="cuda")[shift:]
        f, b = buf(h * w * c), buf(h * w * c, torch.int16)
        ops.tonemap(img, h, w, 0.7, c, f, b)
        ref = torch.zeros((h * w, c), device="cuda")
        ref[:, :3] = torch.log1p(img / 0.7).reshape(3, -1).T
        assert (f.reshape(h * w, c) - ref).abs().max() <= 1e-6 * ref.abs().max()
        assert torch.equal(b, f.to(torch.bfloat16).view(torch.int16))
        back = buf(3 * h * w)
        ops.untonemap(f, h, w, 0.7, c, back)
        assert (back.reshape(3, h, w) - img).abs().max() <= 4e-6 * img.abs().max()
        grad, part = buf(h * w * c), buf(256)
        target = torch.rand(h * w * c + shift, generator=g, device="cuda")[shift:]
        ops.mse(f, target, grad, h * w, c, min(3, c), part, 256)
        d = (f - target).reshape(h * w, c).clone()
        d[:, 3:] = 0
        want = d * (2.0 / (3 * h * w))
        assert (grad.reshape(h * w, c) - want).abs().max() <= 1e-6 * want.abs().max()
        assert abs(float(part.sum()) - float((d * d).sum())) <= 1e-5 * float((d * d).sum())
        small = torch.rand(h * w * c + shift, generator=g, device="cuda")[shift:]
        for acc in (0, 1):
            din = buf(4 * h * w * c)
            ops.pool2_bwd(small, din, 1, 2 * h, 2 * w, c, acc)
            up = small.reshape(h, w, c).repeat_interleave(2, 0).repeat_interleave(2, 1) * 0.25
            assert torch.equal(din, (up + 7 * acc).reshape(-1))


@pytest.mark.parametrize("levels,h,w", [((32,), 512, 512), ((32,), 499, 509), ((32,), 16, 16384),
                                        ((32, 64), 530, 514), ((32,), 16, 16352)])
def test_reconstruction_from_the_last_layer(levels, h, w):
    """The last layer that maps back into the image itself (512 pixel tiles
    and more; the last size has 511) gives the bits of the separate steps,
    which an output that overlaps the decimated image takes; in place and
    with pixels that are negative, infinite or NaN too."""
    import torch
    net = LN.UNet(seed=5, levels=levels)
    ws, nb = net.workspace(1, h, w)

    def reconstruct(src, out):
        assert net.L.splotch_nn_reconstruct(net.h, LN._p(src), h, w, LN._p(out), LN._p(ws), nb,
                                            LN._s()) == 0
        return out.cpu().numpy()

    g = torch.Generator(device="cuda").manual_seed(h + w)
    dec = torch.rand((3, h, w), generator=g, device="cuda") * 3
    for special in (False, True):
        if special:
            dec[0, 5, 7], dec[1, 9, 4], dec[2, 3, 2] = -1.0, float("inf"), float("nan")
        n = dec.numel()
        room = torch.empty(n + 64, device="cuda")
        room[:n] = dec.reshape(-1)
        want = reconstruct(room, room[64:])
        same = dec.reshape(-1).clone()
        for got in (reconstruct(dec, torch.full((n,), 7.0, device="cuda")),
                    reconstruct(same, same)):
            assert np.array_equal(got, want, equal_nan=True)
        assert np.isfinite(want).any()
