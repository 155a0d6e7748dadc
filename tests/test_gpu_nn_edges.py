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
