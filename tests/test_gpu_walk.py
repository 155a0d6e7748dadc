"""GPU: the row walk's staged distance tables at the list lengths and
positions where a batch, a group of four or eight visits, a scan or a box
edge ends.

Without compensation every splat strategy adds the same terms in the same
order, so the row walk must equal the member-list strategy (which computes
each pixel's distance itself) bit for bit; against the oracle the
repository's image bar of 1e-4 of the largest value holds."""
import numpy as np
import pytest

from paper_1004_1302_amd import binding as B
from paper_1004_1302_amd import synth

pytestmark = pytest.mark.gpu


def crowd(n, ordered, seed, width=37, height=29):
    """n particles over a few 8x8 blocks of a ragged image: sub-pixel to
    whole-image footprints, centres on and off the image edges, two
    log-scaled species with non-positive values among them."""
    rng = np.random.default_rng(seed)
    cam = synth.ortho_unit_square(width, height)
    cam.px_per_unit = 32.0
    x = rng.uniform(0.0, 1.1, n).astype(np.float32)
    y = rng.uniform(0.0, 1.0, n).astype(np.float32)
    # some centres exactly on pixel centres and block borders
    x[::5] = (0.5 + (rng.integers(-18, 20, x[::5].size) + 0.0) / 32.0).astype(np.float32)
    z = rng.uniform(-0.5, 0.5, n).astype(np.float32)
    h = rng.lognormal(np.log(0.06), 0.9, n).astype(np.float32)
    h[::7] = 0.002
    h[::11] = 2.0
    v = rng.lognormal(0.0, 1.0, n).astype(np.float32)
    v[::13] = -1.0
    sp = [synth.Species(log_scale=1, brightness=0.3, absorption=0.3 if ordered else 0.0,
                        mode=synth.ORDERED if ordered else synth.ADDITIVE),
          synth.Species(vmin=0.2, vmax=3.0, log_scale=0, brightness=0.2)]
    return synth.Scene(x, y, z, h, v, cam, sp, species=rng.integers(0, 2, n).astype(np.uint8),
                       rho0=rng.uniform(0.0, 2.0, n).astype(np.float32))


@pytest.mark.parametrize("ordered", [False, True])
@pytest.mark.parametrize("n", [1, 3, 4, 5, 8, 9, 12, 63, 64, 65, 68, 127, 128, 129, 193, 1500])
def test_walk_equals_lists(n, ordered, orc):
    import torch
    scene = crowd(n, ordered, 100 + n)
    parts, pal = B.scene_to_device(scene)
    img = {}
    for tile in (8, 16, 32):
        for variant in (1, 2):
            img[variant] = B.render(parts, scene.camera, pal, scene.species_params, tile=tile,
                                    splat_variant=variant).cpu().numpy()
        assert np.array_equal(img[1], img[2]), f"tile {tile}"
    ref = orc.render(scene)
    for tile in (0, 64):
        got = B.render(parts, scene.camera, pal, scene.species_params, tile=tile,
                       compensated=True).cpu().numpy().astype(np.float64)
        torch.cuda.synchronize()
        den = np.abs(ref).max(axis=(1, 2), keepdims=True)
        assert np.all(np.abs(got - ref) <= 1e-4 * np.where(den > 0, den, 1.0)), f"tile {tile}"
