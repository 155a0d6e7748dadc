"""GPU: renders and pair lists in the smallest workspaces they fit, where the
sorts have no room for the short tiles' histograms, equal the ones in roomy
workspaces bit for bit (sorting is stable and exact with either tile size)."""
import ctypes as C

import pytest

from paper_1004_1302_amd import binding as B
from paper_1004_1302_amd import synth

pytestmark = pytest.mark.gpu


def tight_scene(n, tile):
    """Scene and the pairs it has; the workspace for exactly those."""
    import torch
    scene = synth.nfw_halos(n, seed=n, n_halos=9, grid=16, width=150, height=97)
    parts, pal = B.scene_to_device(scene)
    ts, te, pp, total = B.bin_pairs(parts, scene.camera, scene.species_params, tile=tile)
    torch.cuda.synchronize()
    return scene, parts, pal, (ts, te, pp, total)


def workspace(scene, pairs, **kw):
    import torch
    cam = B.camera_struct(scene.camera)
    prm = B.params_struct(scene.species_params, **kw)
    out = C.c_size_t()
    assert B.lib().splotch_workspace_size(scene.n, C.byref(cam), C.byref(prm), pairs,
                                          C.byref(out)) == 0
    return torch.empty(out.value, dtype=torch.uint8, device="cuda")


@pytest.mark.parametrize("tile", [8, 32])
@pytest.mark.parametrize("n", [1, 1024, 1025, 20_000, 150_000])
def test_smallest_workspace(n, tile):
    import torch
    scene, parts, pal, (ts, te, pp, total) = tight_scene(n, tile)
    # one partial image pair only: least room for the sorts
    kw = dict(compensated=True, tile=tile, seg_records=1 << 24)
    want = B.render(parts, scene.camera, pal, scene.species_params, **kw)
    ws = workspace(scene, max(total, 1), tile=tile, seg_records=1 << 24)
    got, st = B.render(parts, scene.camera, pal, scene.species_params, workspace=ws, stats=True,
                       **kw)
    assert st["n_chunks"] == (1 if total else 0)
    assert torch.equal(got, want)
    ws = workspace(scene, max(total, 1), tile=tile)
    ts1, te1, pp1, total1 = B.bin_pairs(parts, scene.camera, scene.species_params, tile=tile,
                                        workspace=ws)
    assert total1 == total
    assert torch.equal(ts1, ts) and torch.equal(te1, te) and torch.equal(pp1, pp)


@pytest.mark.parametrize("tile,width", [(8, 150), (16, 150), (32, 150), (64, 150), (8, 800)])
@pytest.mark.parametrize("n", [300, 20_000, 150_000])
def test_default_segments_where_slots_are_few(n, tile, width):
    """The default segments in workspaces from the one for exactly the pairs,
    whose slots allow only longer segments, to the default one (15,200 tiles
    of 8 pixels: the bookkeeping in four kernels).  An additive set: the
    partial images and their compensated sum round a pixel's positive sum by
    2^-24 a few times, and the terms of a 64-record batch, which begin
    elsewhere in a list with every cut, are added plainly: 2 x 64 x 2^-24 =
    7.7e-6 of a pixel's value."""
    import torch
    scene = synth.plummer_mix(n, seed=n)
    parts, pal = B.scene_to_device(scene)
    cam = synth.ortho_unit_square(width, width * 3 // 4 if width < 800 else 1200)
    kw = dict(compensated=True, tile=tile)
    one, st = B.render(parts, cam, pal, scene.species_params, seg_records=1 << 24, stats=True,
                       max_pairs=20 * n + 200_000, **kw)
    assert st["n_chunks"] == 1
    total = st["n_pairs"]
    scene.camera = cam
    assert float(one.max()) > 0
    for pairs in (total, total + total // 8, 2 * total, 0):
        img, st = B.render(parts, cam, pal, scene.species_params, stats=True,
                           workspace=workspace(scene, pairs, tile=tile), **kw)
        assert st["n_chunks"] == 1 or pairs == 0
        assert float((img - one).abs().max()) <= 1e-5 * float(one.max())
        assert bool(((img - one).abs() <= 1e-5 * one).all())
