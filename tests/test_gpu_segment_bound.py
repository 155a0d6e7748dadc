"""GPU: frames cut into the default segments against FP64, with up to 606
segments in a list.

Bound: cutting changes where partial sums are joined, nothing in a record's own
term.  A pixel's colour is the sum of T_s C_s over its segments: C_s is rounded
when it is stored (2^-24), T_s is one exponential of a compensated sum of
optical depths (2^-22 with the depths' own rounding), the product rounds once
and the sum is compensated, so the joins add less than 2^-21 of the pixel's
value however many they are.  Within a segment sums are no longer than in the
uncut list.  So the cut frame's largest relative error may exceed the uncut
one's by 2^-21 = 4.8e-7."""
import numpy as np
import pytest

from paper_1004_1302_amd import binding as B
from paper_1004_1302_amd import synth

pytestmark = pytest.mark.gpu


def longest(parts, scene, tile, seg_records=0):
    """Segments of the longest list: at least seg_records and a multiple of
    the tile's pixels, or by the default rule."""
    ts, te, _, pairs = B.bin_pairs(parts, scene.camera, scene.species_params, tile=tile)
    nt = tile * tile
    if seg_records:
        length = -(-seg_records // nt) * nt
    else:
        length = min(max(128, -(-pairs * nt // 2 ** 19)), max(1024, nt))
        length = -(-length // 64) * 64
    return -(-int((te - ts).max()) // length)


@pytest.mark.parametrize("n,tile,segments,at64", [
    (150_000, 8, 221, 441), (400_000, 8, 303, 606), (400_000, 16, 320, 240),
    (400_000, 32, 154, 77), (400_000, 64, 78, 36)])
def test_cut_frames_are_as_exact_as_whole_ones(orc, n, tile, segments, at64):
    import torch
    scene = synth.nfw_halos(n, seed=n, n_halos=6, grid=16, width=150, height=97)
    parts, pal = B.scene_to_device(scene)
    ref = orc.render(scene)
    seen = ref > 0
    kw = dict(B.scene_options(scene), compensated=True, tile=tile)

    def error(**more):
        img = B.render(parts, scene.camera, pal, scene.species_params, **kw, **more)
        torch.cuda.synchronize()
        got = img.cpu().numpy().astype(np.float64)
        assert np.all(got[~seen] == 0)
        return (np.abs(got - ref)[seen] / ref[seen]).max()

    whole = error(seg_records=1 << 24)
    assert longest(parts, scene, tile) == segments
    assert error() <= whole + 2.0 ** -21
    assert longest(parts, scene, tile, 64) == at64
    assert error(seg_records=64) <= whole + 2.0 ** -21
