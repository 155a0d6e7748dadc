"""Workspace sizes and pair capacities that a caller may have fixed in a
program: a render needs no more bytes, and a workspace of a given size holds
no fewer pairs, than these (sizes of the layout with 4096-key radix tiles and
partial images for segments of 1024 records; what the sorts and the shorter
segments want beyond it comes from areas that are not in use then)."""
import ctypes as C

import pytest

from paper_1004_1302_amd import binding as B
from paper_1004_1302_amd import synth


def size(n, w, h, tile, mode, pairs, seg_records=0):
    cam = B.camera_struct(synth.ortho_unit_square(w, h))
    prm = B.params_struct([synth.Species(mode=mode, absorption=1.0)], tile=tile,
                          seg_records=seg_records)
    out = C.c_size_t()
    assert B.lib().splotch_workspace_size(n, C.byref(cam), C.byref(prm), pairs,
                                          C.byref(out)) == 0
    return out.value


@pytest.mark.parametrize("n,w,h,tile,mode,pairs,most", [
    (1, 64, 64, 16, 0, 1, 363_008), (900, 150, 97, 8, 1, 1, 422_912),
    (20_000, 96, 64, 16, 1, 1, 1_648_128), (1_000_000, 1024, 1024, 16, 1, 1, 64_872_192),
    (1 << 20, 640, 360, 32, 1, 1, 67_830_272), (4_000_000, 1920, 1080, 16, 1, 1, 257_979_392),
    (300_000, 4096, 4096, 64, 0, 1, 15_171_840), (100_000, 256, 256, 16, 1, 400_000, 18_069_504),
    (1_000_000, 1920, 1080, 16, 1, 1 << 20, 94_454_528)])
def test_workspace_does_not_grow(n, w, h, tile, mode, pairs, most):
    assert size(n, w, h, tile, mode, pairs, seg_records=1024) <= most


@pytest.mark.parametrize("n,subset,slab,most", [
    (1000, 100, 100, 6_448_384), (10 ** 6, 50_000, 300_000, 69_927_168),
    (10 ** 7, 1 << 22, 1 << 20, 1_139_091_200)])
def test_stream_workspace_does_not_grow(n, subset, slab, most):
    cam = B.camera_struct(synth.ortho_unit_square(320, 200))
    prm = B.params_struct([synth.Species(mode=synth.ORDERED, absorption=1.0)], seg_records=1024)
    P = B.Particles()
    P.n = n
    P.x = P.y = P.z = P.h = P.value = 1  # sizes only
    out = C.c_size_t()
    assert B.lib().splotch_stream_workspace_size(C.byref(P), subset, slab, C.byref(cam),
                                                 C.byref(prm), C.byref(out)) == 0
    assert out.value <= most


@pytest.mark.parametrize("n,w,h,tile,nbytes,least", [
    (4_000_000, 1920, 1080, 16, 256 << 20, 373_759), (4_000_000, 1024, 1024, 32, 256 << 20, 168_959),
    (1_000_000, 1024, 1024, 16, 80_000_000, 540_671),
    (1_000_000, 1024, 1024, 16, 100_000_000, 1_252_352),
    (1_000_000, 1024, 1024, 8, 80_000_000, 763_136), (2_000, 4096, 4096, 64, 8 << 20, 36_863),
    (100_000, 256, 256, 16, 12_000_000, 185_216)])
def test_workspace_holds_as_many_pairs(n, w, h, tile, nbytes, least):
    """With the default segments: `least` pairs and the layout for them fit."""
    assert size(n, w, h, tile, 1, least) <= nbytes
