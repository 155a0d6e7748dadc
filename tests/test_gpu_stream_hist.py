"""Depth histogram and copies of the streamed render: particles nearer and
further than a workgroup's 8192 histogram bins reach (a factor of 16 in depth),
subsets around its 16384 keys, no visible particle, and two calls at once.
Against the device-resident render: 2e-5 relative L-infinity, the bound of
the other streamed renders (sums in another order)."""
import threading

import numpy as np
import pytest

from paper_1004_1302_amd import binding as B

from test_gpu_parity import c2_small, check_image, gpu_render
from test_gpu_stream import host_parts, streamed, torch_cuda  # noqa: F401

pytestmark = pytest.mark.gpu


def deep_scene(n, seed, spread):
    """c2_small with its particles moved along their view rays to depths
    spread over a factor `spread` (same screen place, same angular size)."""
    scene = c2_small(n, seed=seed, w=160, h=120)
    cam = scene.camera
    eye = np.asarray(cam.eye, np.float64)
    p = np.stack([scene.x, scene.y, scene.z], 1).astype(np.float64) - eye
    f = np.exp(np.random.default_rng(seed).uniform(-0.5, 0.5, scene.n) * np.log(spread))
    p = eye + p * f[:, None]
    scene.x, scene.y, scene.z = (np.ascontiguousarray(p[:, k], np.float32) for k in range(3))
    scene.h = np.ascontiguousarray(scene.h * f, np.float32)
    return scene


@pytest.mark.parametrize("spread", [1.0, 40.0, 3000.0])
@pytest.mark.parametrize("subset", [16383, 16385, 50_000])
def test_stream_depths_beyond_lds_bins(torch_cuda, spread, subset):  # noqa: F811
    scene = deep_scene(60_000, 71, spread)
    img, st = streamed(torch_cuda, scene, subset=subset, slab=12_000, compensated=True)
    assert st["ordered"] == 1 and st["n_chunks"] >= 2
    check_image(img, gpu_render(scene, compensated=True).astype(np.float64), tol=2e-5)


def test_stream_nothing_visible(torch_cuda):  # noqa: F811
    scene = deep_scene(20_000, 72, 1.0)
    eye = np.asarray(scene.camera.eye, np.float32)
    scene.x, scene.y, scene.z = (np.ascontiguousarray(2 * eye[k] - v, np.float32)
                                 for k, v in enumerate((scene.x, scene.y, scene.z)))
    img, st = streamed(torch_cuda, scene, subset=7_000, slab=9_000)
    dev, dst = gpu_render(scene, stats=True)
    assert st["n_visible"] == dst["n_visible"] == 0
    assert np.array_equal(img, dev)


def test_stream_two_threads(torch_cuda, monkeypatch):  # noqa: F811
    """Two host threads, each with its own stream, workspace and set."""
    torch = torch_cuda
    own = threading.local()

    def workspace(nbytes, device):
        own.ws = torch.empty(nbytes, dtype=torch.uint8, device=device)
        return own.ws

    scenes = [deep_scene(60_000, 73 + k, 40.0) for k in range(2)]
    want = [gpu_render(s, compensated=True).astype(np.float64) for s in scenes]
    parts = [host_parts(torch, s) for s in scenes]
    monkeypatch.setattr(B, "get_workspace", workspace)
    got = [None, None]

    def work(k):
        with torch.cuda.stream(torch.cuda.Stream()):
            _, pal = B.scene_to_device(scenes[k])
            for _ in range(4):
                img = B.render_stream(parts[k], scenes[k].camera, pal, scenes[k].species_params,
                                      subset=5_000, slab=25_000, compensated=True,
                                      **B.scene_options(scenes[k]))
            torch.cuda.current_stream().synchronize()
            got[k] = img.cpu().numpy()

    ts = [threading.Thread(target=work, args=(k,)) for k in range(2)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    for k in range(2):
        check_image(got[k], want[k], tol=2e-5)
