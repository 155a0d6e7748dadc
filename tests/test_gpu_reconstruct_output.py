"""GPU: a reconstruction leaves the last layer's float32 output where
splotch_nn_layer_info says, on the route that maps back into the image in the
last layer (512 tiles of 16 x 32 pixels and more, the images apart or the same)
as on the separate steps (images that overlap otherwise, fewer tiles): the same
bits, and the network's output for the tone-mapped input."""
import numpy as np
import pytest

from paper_1004_1302_amd import learned as LN

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("levels,cin,h,w", [((32,), 32, 512, 512), ((32,), 32, 499, 509),
                                            ((32,), 64, 512, 514), ((32, 64), 32, 530, 514),
                                            ((32,), 32, 16, 16352)])
def test_reconstruction_writes_the_last_output(levels, cin, h, w):
    import torch
    net = LN.UNet(seed=5, levels=levels, cin=cin)
    ws, nb = net.workspace(1, h, w)
    off = net.layer_info(len(net.layers()) - 1, 1, h, w).y
    y = net.tensor(off, h * w * cin, torch.float32)
    g = torch.Generator(device="cuda").manual_seed(h + w)
    n = 3 * h * w
    room = torch.empty(n + 64, device="cuda")

    def reconstruct(src, out):
        y.fill_(7.0)
        assert net.L.splotch_nn_reconstruct(net.h, LN._p(src), h, w, LN._p(out), LN._p(ws), nb,
                                            LN._s()) == 0
        return y.cpu().numpy().copy(), out.cpu().numpy()

    for seed in range(2):  # another image: nothing of the pass before is left
        dec = torch.rand((n,), generator=g, device="cuda") * 3
        room[:n] = dec
        want, image = reconstruct(room, room[64:])
        # its first three channels are the image's tone map
        scale = float(dec.mean())
        tone = np.log1p(image.reshape(3, -1).T.astype(np.float64) / scale)
        assert np.abs(want.reshape(h * w, cin)[:, :3] - tone).max() <= 1e-5 * np.abs(tone).max()
        same = dec.clone()
        for got, img in (reconstruct(dec, torch.full((n,), 7.0, device="cuda")),
                         reconstruct(same, same)):
            assert np.array_equal(got, want)
            assert np.array_equal(img, image)
