"""A streamed render that ends in an error has no copy under way: an invalid
colour map is refused before the first copy, and an error found while subsets
are copied (vector colours without their components) is returned when both
subsets that were started have arrived, so the caller may reuse the host set
and the workspace at once."""
import ctypes as C

import numpy as np
import pytest

from paper_1004_1302_amd import binding as B
from paper_1004_1302_amd import synth

pytestmark = pytest.mark.gpu
SUBSET = 2_000_000
FIELDS = ("x", "y", "z", "h", "value")


def call(species, n_entries):
    """One streamed render of two subsets; returns its status and the first
    subsets' fields as the two staging buffers hold them when it returns."""
    import torch
    g = torch.Generator().manual_seed(3)
    host = {k: torch.rand(2 * SUBSET, generator=g).pin_memory() for k in FIELDS}
    P = B.host_particles_struct(host)
    cam = B.camera_struct(synth.ortho_unit_square(64, 64))
    prm = B.params_struct(species)
    size = C.c_size_t(0)
    assert B.lib().splotch_stream_workspace_size(C.byref(P), SUBSET, SUBSET, C.byref(cam),
                                                 C.byref(prm), C.byref(size)) == 0
    ws = torch.full((size.value,), 0xAB, dtype=torch.uint8, device="cuda")
    image = torch.zeros((3, 64, 64), device="cuda")
    pal = torch.ones((2, 3), device="cuda")
    torch.cuda.synchronize()
    prm.workspace, prm.workspace_bytes = C.c_void_p(ws.data_ptr()), size.value
    s = torch.cuda.Stream()
    prm.stream = C.c_void_p(s.cuda_stream)
    cm = B.colourmap_struct(pal)
    cm.n_entries = n_entries
    img = B.Image(C.c_void_p(image.data_ptr()), 64, 64)
    code = B.lib().splotch_render_stream(C.byref(P), SUBSET, SUBSET, C.byref(cam), C.byref(cm),
                                         C.byref(prm), C.byref(img))
    step = -(-SUBSET * 4 // 256) * 256
    staged = ws[:2 * len(FIELDS) * step].clone()
    s.synchronize()
    stages = staged.cpu().numpy().reshape(2, len(FIELDS), step)[:, :, :SUBSET * 4]
    return code, host, stages


@pytest.mark.parametrize("mode", [synth.ADDITIVE, synth.ORDERED])
def test_invalid_colour_map_starts_no_copy(mode):
    code, _, stages = call([synth.Species(mode=mode, absorption=1.0, vmin=0.0, vmax=1.0)], 1)
    assert code == 1  # invalid argument
    assert (stages == 0xAB).all()


def test_error_waits_for_its_copies():
    species = synth.Species(vmin=0.0, vmax=1.0, colour=synth.COLOUR_VECTOR)
    code, host, stages = call([species], 2)
    assert code == 1
    for b in range(2):
        for k, name in enumerate(FIELDS):
            want = host[name][b * SUBSET:(b + 1) * SUBSET].numpy().view(np.uint8)
            assert np.array_equal(stages[b, k], want), (b, name)
