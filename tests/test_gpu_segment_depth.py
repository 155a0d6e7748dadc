"""GPU: the transmittance behind many segments.  65,536 equal particles lie on
the centre of one pixel, where each adds exactly 2^-14 to the optical depth: 4
in all, whatever the segments, and every sum on the way is exact.  The pixel
then shows 1 - exp(-4) in front of an incoming image of 1024.

Bound: the transmittance is one binary32 exponential (2^-23 relative), its
product with the incoming image one rounding (2^-24); the particles' own light,
5 % of the pixel, is a compensated sum of terms with two such exponentials.
Together below 2^-22.  (A product of the segments' rounded transmittances is
off by 40 times that.)"""
import numpy as np
import pytest

from paper_1004_1302_amd import binding as B
from paper_1004_1302_amd import synth

pytestmark = pytest.mark.gpu
N = 1 << 16


@pytest.mark.parametrize("variant", [1, 2, 3])
@pytest.mark.parametrize("tile,seg", [(8, 64), (16, 256), (16, 0), (32, 0), (8, 1 << 24)])
@pytest.mark.parametrize("emission", ["equal", "general"])
def test_transmittance_behind_many_segments(tile, seg, variant, emission):
    import torch
    cam = synth.ortho_unit_square(64, 64)
    i, j = 36, 35
    fill = lambda v: torch.full((N,), v, dtype=torch.float32, device="cuda")  # noqa: E731
    parts = dict(x=fill((i + 0.5) / 64), y=fill((j + 0.5) / 64), z=fill(0.5), h=fill(0.6 / 64),
                 value=fill(0.0), rho0=fill(2.0 ** -14))
    pal = torch.ones((2, 3), device="cuda")
    # general: no light of their own, every record an absorber with E != A
    species = [synth.Species(mode=synth.ORDERED, absorption=1.0, vmin=0.0, vmax=1.0,
                             brightness=1.0 if emission == "equal" else 0.0)]
    image = torch.full((3, 64, 64), 1024.0, device="cuda")
    B.render(parts, cam, pal, species, image=image, accumulate=True, compensated=True, tile=tile,
             seg_records=seg, splat_variant=variant)
    got = image.cpu().numpy().astype(np.float64)
    hit = np.argwhere(got[0] == got[0].min())
    assert len(hit) == 1
    light = -np.expm1(-4.0) if emission == "equal" else 0.0
    want = light + 1024.0 * np.exp(-4.0)
    assert abs(got[:, hit[0][0], hit[0][1]] / want - 1.0).max() <= 2.0 ** -22


@pytest.mark.parametrize("rho", [1e30, 3.0e38])
def test_opaque_segments(rho):
    """Optical depths that overflow hide the incoming image and nothing else:
    the pixel is the particles' own light, 1."""
    import torch
    cam = synth.ortho_unit_square(64, 64)
    fill = lambda v: torch.full((4096,), v, dtype=torch.float32, device="cuda")  # noqa: E731
    parts = dict(x=fill(36.5 / 64), y=fill(35.5 / 64), z=fill(0.5), h=fill(0.6 / 64),
                 value=fill(0.0), rho0=fill(rho))
    pal = torch.ones((2, 3), device="cuda")
    species = [synth.Species(mode=synth.ORDERED, absorption=1.0, vmin=0.0, vmax=1.0)]
    for variant in (1, 2, 3):
        image = torch.full((3, 64, 64), 1024.0, device="cuda")
        B.render(parts, cam, pal, species, image=image, accumulate=True, compensated=True, tile=8,
                 seg_records=64, splat_variant=variant)
        got = image.cpu().numpy()
        assert np.isfinite(got).all()
        assert got.min() == 1.0


@pytest.mark.parametrize("variant", [1, 2, 3])
@pytest.mark.parametrize("tile,seg", [(8, 64), (8, 0)])
def test_plain_sums_behind_many_segments(tile, seg, variant):
    """A frame without compensated sums: each of 65,536 additive particles adds
    (2^16 + 341) 2^-29 to one pixel, so the sums of 64 and of 128 are exact and
    only joining the segments can round.  The joins are compensated: 2^-23 in
    all (plain ones are off by 1e-5).  A sum that overflows is infinite."""
    import torch
    cam = synth.ortho_unit_square(64, 64)
    light = (2 ** 16 + 341) * 2.0 ** -29
    fill = lambda v: torch.full((N,), v, dtype=torch.float32, device="cuda")  # noqa: E731
    parts = dict(x=fill(36.5 / 64), y=fill(35.5 / 64), z=fill(0.5), h=fill(0.6 / 64),
                 value=fill(0.0), rho0=fill(light))
    pal = torch.ones((2, 3), device="cuda")

    def image():
        img = B.render(parts, cam, pal, [synth.Species(vmin=0.0, vmax=1.0)], tile=tile,
                       seg_records=seg, splat_variant=variant)
        return img.cpu().numpy().astype(np.float64)

    assert abs(image().max(axis=(1, 2)) / (N * light) - 1.0).max() <= 2.0 ** -23
    parts["rho0"].fill_(3.0e38)
    assert not np.isnan(image()).any() and np.isinf(image()).any()
