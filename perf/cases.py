"""Performance cases of the renderer: what its users have it do, through the
public entry points of `paper_1004_1302_amd`.

A case is a dict of plain values.  `listed()` gives the fixed ones, `draw()`
one more of the same ranges, `prepare()` makes a case's inputs on the GPU
from a seed, `run()` makes one pass, `work()` says what a pass cannot do
without, and `exact()` gives what `run()` returns, computed in binary64 with
plain torch.

Paths:
  frame      one image of a device-resident set (splotch_render)
  batch      several views of one set (splotch_render_batch)
  stream     one image of a set in pinned host memory (splotch_render_stream)
  learned    decimated render, network and probe (splotch_render_learned)
  reconstruct  the network alone on a decimated render (splotch_nn_reconstruct)
  gradients  forward, loss and backward pass of the network's training
  decimate   the seeded 1/16 subset (splotch_decimate)

Particle sets are the seeded stand-ins of `synth`, drawn with torch on the
GPU: Plummer spheres in a uniform cube (one additive species), NFW halos and
the lognormal field (depth-ordered gas with absorption equal to emission,
and additive dark matter).
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_1004_1302_amd import binding as B
from paper_1004_1302_amd import learned as LN
from paper_1004_1302_amd import synth

DEV = "cuda"
BOX = 100.0


# ------------------------------------------------------------------- cases
def listed():
    return [
        # the smallest call: a preview thumbnail, all launches and latency
        frame("thumbnail_nfw_2e4", "nfw", 20_000, 96, 64),
        # the small configuration of the benchmark: one additive species
        frame("small_plummer_1e5", "plummer", 100_000, 256, 256),
        # the paper's "small" set seen from inside the box: footprints from
        # a pixel to the whole window, so the pair emission splits particles
        frame("inside_nfw_370852", "nfw", 370_852, 1920, 1080, view="inside"),
        # general colours of Section 2 at an odd size: a vector-coloured gas
        # that absorbs otherwise than it emits, plain (uncompensated) sums
        frame("vector_nfw_1e6", "nfw", 1_000_003, 1000, 701, colour="vector", compensated=False),
        # the everyday frame: ten million particles at full HD
        frame("fullhd_nfw_1e7", "nfw", 10_000_000, 1920, 1080),
        # the largest: a billion particles at 4096 x 4096, the benchmark's
        # default workload and settings
        frame("field_lognormal_1e9", "lognormal", 1_000_000_000, 4096, 4096, tile=32,
              max_pairs=1_600_000_000),
        # an orbit of thumbnails and small views for a movie or a survey of
        # viewpoints, four views in flight
        batch("orbit_nfw_1e6", "nfw", 1_000_000, 24, "small", streams=4),
        # a set that stays in host memory, in subsets and depth slabs
        dict(name="hostset_nfw_6e6", path="stream", set="nfw", n=6_000_000, width=1920,
             height=1080, view="outside", colour="equal", compensated=True, tile=0,
             subset=1 << 20, slab=1 << 21),
        # learned decimation of one view, the probe agreeing (no fallback)
        dict(name="learned_plummer_2e7", path="learned", set="plummer", n=20_000_000, size=1024),
        # the network alone, on one image
        dict(name="reconstruct_1024", path="reconstruct", height=1024, width=1024),
        # one training step's gradients, the benchmark's batch of four
        dict(name="gradients_4x1024", path="gradients", images=4, size=1024),
        # the subset for the learned path, once per particle set
        dict(name="decimate_2e7", path="decimate", set="plummer", n=20_000_000),
    ]


def frame(name, kind, n, width, height, view="outside", colour=None, compensated=True, tile=0,
          max_pairs=0, kernel3d=False):
    c = dict(path="frame", set=kind, n=n, width=width, height=height, view=view,
             colour=colour or ("additive" if kind == "plummer" else "equal"),
             compensated=compensated, tile=tile, max_pairs=max_pairs, kernel3d=kernel3d)
    return dict(c, name=name) if name else c


def batch(name, kind, n, views, sizes, streams, persistent=False, compensated=True):
    c = dict(path="batch", set=kind, n=n, views=views, sizes=sizes, streams=streams,
             persistent=persistent, compensated=compensated,
             colour="additive" if kind == "plummer" else "equal")
    return dict(c, name=name) if name else c


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    path = rng.choices(["frame", "batch", "stream", "learned", "reconstruct", "gradients",
                        "decimate"], [50, 14, 8, 6, 8, 8, 6])[0]
    if path == "frame":
        n = _log(rng, 1e4, 2.5e8)
        comp = rng.random() < 0.75
        if n > 2e7:
            # large sets come as fields, on large images
            return frame(None, "lognormal", n, rng.randint(1500, 4096), rng.randint(1500, 4096),
                         compensated=comp, tile=32)
        tile = rng.choice([0, 0, 0, 16, 32, 8, 64]) if n < 1_000_000 else rng.choice([0, 0, 32])
        if rng.random() < 0.35:
            w = _log(rng, 64, min(2048, max(128, 1024 * math.sqrt(2e10 / (420 * n)))))
            return frame(None, "plummer", n, w, w, compensated=comp, tile=tile,
                         kernel3d=rng.random() < 0.15)
        return frame(None, "nfw", n, _log(rng, 64, 2200), _log(rng, 64, 1600),
                     view="inside" if n < 2_700_000 and rng.random() < 0.25 else "outside",
                     colour=rng.choice(["equal", "equal", "equal", "table", "vector", "source",
                                        "additive"]),
                     compensated=comp, tile=tile, kernel3d=rng.random() < 0.15)
    if path == "batch":
        streams = rng.randint(1, 4)
        return batch(None, rng.choice(["nfw", "plummer"]), _log(rng, 3e4, 3e6),
                     rng.randint(3, 24), rng.choice(["small", "large"]), streams,
                     persistent=rng.random() < 0.3, compensated=rng.random() < 0.75)
    if path == "stream":
        kind = rng.choice(["nfw", "plummer"])
        n = _log(rng, 3e5, 6e6)
        return dict(path="stream", set=kind, n=n, width=rng.randint(300, 1920),
                    height=rng.randint(300, 1080), view="outside",
                    colour="additive" if kind == "plummer" else "equal",
                    compensated=rng.random() < 0.75, tile=0,
                    subset=rng.randint(n // 7, n // 2), slab=rng.randint(n // 3, n))
    if path == "learned":
        return dict(path="learned", set="plummer", n=_log(rng, 1e6, 2e7),
                    size=32 * rng.randint(8, 32))
    if path == "reconstruct":
        return dict(path="reconstruct", height=32 * rng.randint(6, 40),
                    width=32 * rng.randint(6, 40))
    if path == "gradients":
        return dict(path="gradients", images=rng.randint(1, 4), size=32 * rng.randint(4, 24))
    return dict(path="decimate", set=rng.choice(["plummer", "nfw"]), n=_log(rng, 1e5, 2e7))


# ------------------------------------------------------------------ inputs
def _gen(seed, salt):
    g = torch.Generator(device=DEV)
    g.manual_seed(1_000_003 * (int(seed) % 1_000_003) + salt)
    return g


def _directions(n, gen):
    cz = torch.rand(n, generator=gen, device=DEV) * 2 - 1
    ph = torch.rand(n, generator=gen, device=DEV) * (2 * math.pi)
    s = torch.sqrt(1 - cz * cz)
    return torch.stack([s * torch.cos(ph), s * torch.sin(ph), cz], dim=1)


def _plummer(n, gen):
    """Half uniform in the unit cube, half in ten Plummer spheres of scale
    0.02 cut at ten scale radii; lognormal smoothing lengths and values."""
    n_p = n - n // 2
    u = torch.rand(n_p, generator=gen, device=DEV) * (1e3 / 101.0 ** 1.5)
    r = 0.02 / torch.sqrt(u.clamp_min(1e-12) ** (-2.0 / 3.0) - 1)
    centre = torch.rand(10, 3, generator=gen, device=DEV) * 0.8 + 0.1
    ball = torch.arange(n_p, device=DEV) * 10 // n_p
    pos = torch.cat([torch.rand(n // 2, 3, generator=gen, device=DEV),
                     centre[ball] + r[:, None] * _directions(n_p, gen)])
    h = torch.exp(math.log(0.005) - 0.125 + 0.5 * torch.randn(n, generator=gen, device=DEV))
    val = torch.exp(torch.randn(n, generator=gen, device=DEV))
    return dict(x=pos[:, 0].contiguous(), y=pos[:, 1].contiguous(), z=pos[:, 2].contiguous(),
                h=h, value=val)


def _nfw(n, gen):
    """NFW halos with a power-law mass function, 20% uniform background,
    smoothing lengths from the local density, two species."""
    halos = 1000 if n >= 300_000 else 12
    grid = 256 if n >= 1_000_000 else (128 if n >= 300_000 else 32)
    n_h = n - n // 5
    u = torch.rand(halos, generator=gen, device=DEV, dtype=torch.float64)
    mass = (1.0 + u * (1000.0 ** -0.9 - 1.0)) ** (-1.0 / 0.9)
    counts = torch.floor(n_h * mass / mass.sum()).to(torch.int64)
    counts[: int(n_h - counts.sum())] += 1
    which = torch.repeat_interleave(torch.arange(halos, device=DEV), counts, output_size=n_h)
    rvir = (5.0 * (mass / mass.max()) ** (1.0 / 3.0)).float()
    xs = torch.cat([torch.zeros(1, device=DEV, dtype=torch.float64),
                    torch.logspace(-6, 1, 4096, device=DEV, dtype=torch.float64)])
    ms = torch.log1p(xs) - xs / (1 + xs)
    q = torch.rand(n_h, generator=gen, device=DEV, dtype=torch.float64) * ms[-1]
    k = torch.searchsorted(ms, q).clamp(1, 4096)
    xr = xs[k - 1] + (xs[k] - xs[k - 1]) * (q - ms[k - 1]) / (ms[k] - ms[k - 1])
    r = xr.float() * rvir[which] / 10.0
    centre = torch.rand(halos, 3, generator=gen, device=DEV) * BOX
    pos = torch.cat([centre[which] + r[:, None] * _directions(n_h, gen),
                     torch.rand(n - n_h, 3, generator=gen, device=DEV) * BOX])
    cell = (pos / BOX * grid).to(torch.int64).clamp(0, grid - 1)
    flat = (cell[:, 0] * grid + cell[:, 1]) * grid + cell[:, 2]
    rho = torch.bincount(flat, minlength=grid ** 3)[flat].float() / (n / grid ** 3)
    h = torch.clamp(BOX / n ** (1 / 3) * rho ** (-1 / 3), 0.01, 2.0)
    species = (torch.rand(n, generator=gen, device=DEV) >= 0.5).to(torch.uint8)
    return dict(x=pos[:, 0].contiguous(), y=pos[:, 1].contiguous(), z=pos[:, 2].contiguous(),
                h=h.contiguous(), value=rho.contiguous(), species=species)


def _lognormal(n, seed):
    """The lognormal field of `synth`, 7.45 particles per cell as in the
    billion-particle set."""
    grid = max(32, round((n / 7.4505806) ** (1 / 3)))
    return synth.lognormal_field(n_target=n, grid=grid, seed=11 + int(seed) % (1 << 30),
                                 device=DEV)[0]


def _particles(case, seed):
    kind, n = case["set"], int(case["n"])
    if kind == "lognormal":
        return _lognormal(n, seed)
    parts = (_plummer if kind == "plummer" else _nfw)(n, _gen(seed, 1))
    if case.get("colour") == "vector":
        gen = _gen(seed, 2)
        for k in ("value_g", "value_b"):
            parts[k] = parts["value"] * torch.exp(0.3 * torch.randn(n, generator=gen, device=DEV))
    return parts


def _species(case):
    """Species settings, and the absorption table where the case has one."""
    colour = case.get("colour", "equal")
    if case["set"] == "plummer":
        return [synth.Species(mode=synth.ADDITIVE)], None
    b = 0.02 if case["set"] == "lognormal" else 0.15
    gas = synth.Species(log_scale=1, brightness=b, absorption=b, mode=synth.ORDERED)
    dark = synth.Species(log_scale=1, brightness=b, absorption=0.0, mode=synth.ADDITIVE)
    table = None
    if colour == "additive":
        gas.mode, gas.absorption = synth.ADDITIVE, 0.0
    elif colour == "vector":
        gas.colour, gas.absorption = synth.COLOUR_VECTOR, 0.5 * b
    elif colour == "table":
        table = np.ascontiguousarray(synth.palette(64)[:, ::-1])
    return [gas, dark], table


def _camera(case):
    w, h = int(case["width"]), int(case["height"])
    if case["set"] == "plummer":
        if w == h:
            return synth.ortho_unit_square(w, h)
        return synth.look_at((0.5, 0.5, -1.5), (0.5, 0.5, 0.5), (0, 1, 0), synth.PERSPECTIVE, w, h,
                             z_near=0.05, z_far=100.0)
    if case["view"] == "inside":
        return synth.look_at((50, 50, 10), (50, 50, 60), (0, 1, 0), synth.PERSPECTIVE, w, h,
                             z_near=0.5, z_far=500.0)
    return synth.look_at((50, 50, -100), (50, 50, 50), (0, 1, 0), synth.PERSPECTIVE, w, h,
                         z_near=1.0, z_far=1000.0)


SIZES = {"small": [(320, 240), (256, 256), (200, 150), (128, 128)],
         "large": [(1920, 1080), (1280, 720), (1024, 1024), (640, 480)]}


def _orbit(case):
    if case["set"] == "plummer":
        return synth.orbit_cameras(int(case["views"]), 7, SIZES[case["sizes"]])
    return synth.orbit_cameras(int(case["views"]), 7, SIZES[case["sizes"]], centre=(50, 50, 50),
                               radius=150.0, z_near=1.0, z_far=1000.0)


def _palette():
    return torch.from_numpy(synth.palette(256)).to(DEV)


def _options(case, table=None):
    kw = dict(compensated=bool(case["compensated"]), tile=int(case.get("tile", 0)))
    if case.get("kernel3d"):
        kw["kernel"] = synth.KERNEL_TRUNC3D
    if case.get("colour") == "source":
        kw["emission_is_source"] = 1
    if table is not None:
        kw["palette_absorb"] = torch.from_numpy(table).to(DEV)
    return kw


def _subset(parts, seed):
    """A random 1/16 of the particles, flux-preserving (h and rho0 scaled)."""
    n = int(parts["x"].numel())
    pick = torch.rand(n, generator=_gen(seed, 3), device=DEV).topk(max(1, n // 16)).indices
    pick = pick.sort().values
    out = {k: v[pick].contiguous() for k, v in parts.items()}
    out["h"] = out["h"] * LN.H_SCALE
    out["rho0"] = torch.full_like(out["h"], LN.H_SCALE)
    return out


def _picture(seed, salt, h, w):
    """An emission image with the smooth structure and range of a render:
    a few hundred blobs over a faint background."""
    gen = _gen(seed, salt)
    img = torch.full((3, h, w), 0.02, device=DEV)
    y = torch.arange(h, device=DEV, dtype=torch.float32)[:, None]
    x = torch.arange(w, device=DEV, dtype=torch.float32)[None, :]
    p = torch.rand(200, 6, generator=gen, device=DEV)
    s = (0.004 + 0.05 * p[:, 2] ** 3) * max(h, w)
    gy = torch.exp(-((y - p[:, 0] * h) / s) ** 2)       # [h, 200]
    gx = torch.exp(-((x.T - p[:, 1] * w) / s) ** 2)     # [w, 200]
    for c in range(3):
        img[c] += (gy * p[:, 3 + c]) @ gx.T
    return img


def prepare(case, seed):
    path = case["path"]
    s = dict(case=case)
    if path in ("frame", "batch", "stream"):
        sp, table = _species(case)
        s.update(species=sp, palette=_palette(), kw=_options(case, table))
        parts = _particles(case, seed)
        if path == "frame":
            cam = _camera(case)
            s.update(parts=parts, cam=cam,
                     image=torch.empty((3, cam.height, cam.width), device=DEV))
            if case["max_pairs"]:
                s["kw"]["max_pairs"] = int(case["max_pairs"])
        elif path == "batch":
            cams = _orbit(case)
            s.update(parts=parts, cams=cams,
                     images=[torch.empty((3, c.height, c.width), device=DEV) for c in cams])
        else:
            host = {}
            for k, v in parts.items():
                host[k] = torch.empty(v.shape, dtype=v.dtype, pin_memory=True)
                host[k].copy_(v)
            cam = _camera(case)
            s.update(parts=host, cam=cam,
                     image=torch.empty((3, cam.height, cam.width), device=DEV))
    elif path == "learned":
        size = int(case["size"])
        parts = _particles(case, seed)
        s.update(parts=parts, dec=_subset(parts, seed), palette=_palette(),
                 species=_species(case)[0], net=LN.UNet(seed=0),
                 cam=synth.orbit_cameras(1, 9, [(size, size)])[0])
    elif path == "reconstruct":
        s.update(rec=LN.Reconstructor(LN.UNet(seed=0)),
                 image=_picture(seed, 4, int(case["height"]), int(case["width"])))
    elif path == "gradients":
        x, t = _training_batch(case, seed)
        s.update(net=LN.UNet(seed=0), x=x, x_bf=x.to(torch.bfloat16).view(torch.int16), target=t)
    elif path == "decimate":
        s.update(parts=_particles(dict(case, colour="equal"), seed))
    return s


def _training_batch(case, seed):
    """Tone-mapped network inputs (RGB in the first of 32 channels) and
    targets of a batch, as NHWC rows."""
    n, size = int(case["images"]), int(case["size"])
    x = torch.zeros((n, size, size, LN.CIN), device=DEV)
    t = torch.zeros_like(x)
    for k in range(n):
        full = _picture(seed, 10 + k, size, size)
        grain = torch.rand(full.shape, generator=_gen(seed, 30 + k), device=DEV)
        dec = full * (0.4 + 1.2 * grain)
        s = dec.mean()
        x[k, :, :, :3] = torch.log1p(dec / s).permute(1, 2, 0)
        t[k, :, :, :3] = torch.log1p(full / s).permute(1, 2, 0)
    return x.reshape(-1), t.reshape(-1)


# --------------------------------------------------------------------- run
def run(s):
    case = s["case"]
    path = case["path"]
    if path == "frame":
        return B.render(s["parts"], s["cam"], s["palette"], s["species"], s["image"], **s["kw"])
    if path == "batch":
        return B.render_batch(s["parts"], s["cams"], s["palette"], s["species"], s["images"],
                              streams=int(case["streams"]), persistent=bool(case["persistent"]),
                              **s["kw"])
    if path == "stream":
        return B.render_stream(s["parts"], s["cam"], s["palette"], s["species"], s["image"],
                               subset=int(case["subset"]), slab=int(case["slab"]), **s["kw"])
    if path == "learned":
        image, info = LN.render_learned(s["parts"], s["dec"], s["cam"], s["palette"],
                                        s["species"], s["net"], threshold_db=0.0,
                                        compensated=True)
        return dict(image=image, fallback=info["fallback"], probe_psnr=info["probe_psnr"])
    if path == "reconstruct":
        return s["rec"].infer(s["image"])
    if path == "gradients":
        n, size, net = int(case["images"]), int(case["size"]), s["net"]
        y = net.forward(s["x"], s["x_bf"], n, size, size)
        g, loss = net.loss_grad(y, s["target"], n, size, size)
        net.backward(g)
        out = dict(y=y, loss=loss)
        for q in net.layers():
            out["w%02d" % q.k], out["b%02d" % q.k] = q.gw, q.gb
        return out
    return LN.decimate(s["parts"], seed=7)


# -------------------------------------------------------------------- work
# Composited (pixel, particle) pairs per particle of the sets, seen as in the
# listed cases: pixels of the footprint disk, which grow with the image and
# with the mean particle distance.
def _members(case, w, h):
    n = int(case["n"])
    if case["set"] == "plummer":
        return 421.0 * (w / 1024.0) * (h / 1024.0) * (1.0 if w == h else 0.3)
    if case["set"] == "lognormal":
        return 55.0 * (w / 4096.0) ** 2 * (1e9 / n) ** (2 / 3)
    return 45.0 * (w / 1920.0) ** 2 * (1e7 / n) ** (2 / 3)


def work(case):
    path = case["path"]
    if path in ("reconstruct", "learned", "gradients"):
        if path == "gradients":
            px, passes = int(case["images"]) * int(case["size"]) ** 2, 3
        elif path == "learned":
            px, passes = int(case["size"]) ** 2, 1
        else:
            px, passes = int(case["height"]) * int(case["width"]), 1
        flops = passes * _network_flops(px)
        nbytes = 24.0 * px if passes == 1 else px * LN.CIN * 16.0
        if path == "learned":
            n = int(case["n"])
            nbytes += n * 20.0 + n / 16 * 24.0
            dec = 16 ** (2 / 3) / 16 + 0.02   # wider footprints of the subset, and the probe
            flops += 23.0 * n * dec * 0.1 * _members(case, int(case["size"]), int(case["size"]))
        return dict(bytes=nbytes, flops=flops)
    n = int(case["n"])
    each = 20.0 if case["set"] == "plummer" else 21.0
    if case["set"] == "lognormal":
        each = 25.0
    if path == "decimate":
        return dict(bytes=n * each * (1 + 1 / 16), flops=float(n))
    if case.get("colour") == "vector":
        each += 8.0
    per = 23.0 if case["colour"] == "additive" else 26.0
    if path == "batch":
        cams = _orbit(case)
        px = sum(c.width * c.height for c in cams)
        mem = sum(_members(case, c.width, c.height) for c in cams)
        return dict(bytes=n * each + 12.0 * px, flops=per * n * mem)
    w, h = int(case["width"]), int(case["height"])
    return dict(bytes=n * each + 12.0 * w * h, flops=per * n * _members(case, w, h))


def _network_flops(px):
    """Multiply-adds of the 3 x 3 convolutions, twice, for px input pixels."""
    lv, total = LN.LEVELS, 0.0
    for k, (cin, cout, level) in enumerate(_convolutions()):
        total += 18.0 * (3 if k == 0 else cin) * (3 if k == 4 * len(lv) - 2 else cout) / 4 ** level
    return total * px


def _convolutions():
    """(input channels, output channels, level) in the network's order."""
    lv = LN.LEVELS
    out = []
    for k, c in enumerate(lv):
        out += [(LN.CIN if k == 0 else lv[k - 1], c, k), (c, c, k)]
    for k in range(len(lv) - 2, -1, -1):
        out += [(lv[k + 1] + lv[k], lv[k], k), (lv[k], lv[k], k)]
    return out + [(lv[0], LN.CIN, 0)]


# ------------------------------------------------------------------- exact
MOST_FRAGMENTS = 1.5e9  # (pixel, particle) candidates one reference may go through


def exact(case, seed):
    path = case["path"]
    if path in ("frame", "stream", "batch"):
        if int(case["n"]) > 20_000_000:
            return None
        sp, table = _species(case)
        parts = _particles(case, seed)
        opts = dict(table=table, kernel3d=bool(case.get("kernel3d")),
                    source=case.get("colour") == "source")
        if path != "batch":
            return _image(parts, _camera(case), sp, MOST_FRAGMENTS, **opts)
        cams = _orbit(case)
        images = [_image(parts, c, sp, MOST_FRAGMENTS / len(cams), **opts) for c in cams]
        return None if any(i is None for i in images) else images
    if path == "learned":
        size = int(case["size"])
        dec = _subset(_particles(case, seed), seed)
        cam = synth.orbit_cameras(1, 9, [(size, size)])[0]
        img = _image(dec, cam, _species(case)[0], MOST_FRAGMENTS)
        return None if img is None else dict(image=_reconstruct(img), fallback=None,
                                             probe_psnr=None)
    if path == "reconstruct":
        return _reconstruct(_picture(seed, 4, int(case["height"]), int(case["width"])).double())
    if path == "gradients":
        return _gradients(case, seed)
    return None


def _normalised(v, lo, hi, log_scale):
    if log_scale:
        if not (lo > 0 and hi > lo):
            return torch.zeros_like(v)
        t = (torch.log10(v.clamp_min(1e-300)) - math.log10(lo)) / (math.log10(hi) - math.log10(lo))
        t = torch.where(v > 0, t, torch.zeros_like(t))
    else:
        t = (v - lo) / (hi - lo) if hi > lo else torch.zeros_like(v)
    return t.clamp(0, 1)


def _lookup(t, table):
    pal = torch.as_tensor(np.ascontiguousarray(table), device=DEV, dtype=torch.float64)
    p = t * (pal.shape[0] - 1)
    k = p.floor().to(torch.int64).clamp(max=pal.shape[0] - 2)
    w = (p - k)[:, None]
    return pal[k] * (1 - w) + pal[k + 1] * w


def _coefficients(parts, sp, table, source):
    """Emission and absorption of every particle per channel, in binary64."""
    n = int(parts["x"].numel())
    tag = parts["species"] if "species" in parts else torch.zeros(n, dtype=torch.uint8, device=DEV)
    E = torch.zeros((n, 3), dtype=torch.float64, device=DEV)
    A = torch.zeros_like(E)
    for s, q in enumerate(sp):
        at = torch.nonzero(tag == s).flatten()
        if at.numel() == 0:
            continue
        fields = ("value", "value_g", "value_b") if q.colour == synth.COLOUR_VECTOR else ("value",)
        v = [parts[k][at].double() for k in fields]
        ok = torch.cat(v)
        ok = ok[ok > 0] if q.log_scale else ok
        lo, hi = float(ok.min()), float(ok.max())
        t = [_normalised(x, lo, hi, q.log_scale) for x in v]
        ce = torch.stack(t, 1) if len(t) == 3 else _lookup(t[0], synth.palette(256))
        ca = _lookup(t[0], table) if table is not None and len(t) == 1 else ce
        # settings reach the library as binary32
        bright, absorb = float(np.float32(q.brightness)), float(np.float32(q.absorption))
        ordered = q.mode == synth.ORDERED
        A[at] = absorb * ca if ordered else 0.0
        E[at] = bright * ce
        if source and ordered:
            E[at] = A[at] * E[at]
    if "rho0" in parts:
        E, A = E * parts["rho0"].double()[:, None], A * parts["rho0"].double()[:, None]
    return E, A


def _image(parts, cam, sp, most, table=None, kernel3d=False, source=False):
    """The image in binary64: the exact solution of the transfer equation
    particle by particle, front to back.  Pixel membership is decided with
    the binary32 fields that define it.  None when more than `most`
    (pixel, particle) candidates would have to be gone through."""
    W, H, f64 = int(cam.width), int(cam.height), torch.float64
    E, A = _coefficients(parts, sp, table, source)
    d = [parts[k].double() - float(e) for k, e in zip("xyz", cam.eye)]
    axis = [d[0] * float(a[0]) + d[1] * float(a[1]) + d[2] * float(a[2])
            for a in (cam.right, cam.up, cam.fwd)]
    z = axis[2]
    if cam.projection == synth.PERSPECTIVE:
        s = float(np.float32(cam.focal_px)) / z
    else:
        s = torch.full_like(z, float(np.float32(cam.px_per_unit)))
    u, v = axis[0] * s + W / 2, axis[1] * s + H / 2
    sig = parts["h"].double() * s
    r = 2.0 * sig
    i0, i1 = torch.ceil(u - r - 0.5).clamp_min(0), torch.floor(u + r - 0.5).clamp_max(W - 1)
    j0, j1 = torch.ceil(v - r - 0.5).clamp_min(0), torch.floor(v + r - 0.5).clamp_max(H - 1)
    seen = (z > float(np.float32(cam.z_near))) & (z <= float(np.float32(cam.z_far)))
    seen &= (i0 <= i1) & (j0 <= j1)
    at = torch.nonzero(seen).flatten()
    at = at[torch.sort(z[at].float(), stable=True).indices]   # by (binary32 depth, index)
    del d, axis, seen
    bw, bh = (i1 - i0 + 1)[at].to(torch.int64), (j1 - j0 + 1)[at].to(torch.int64)
    ends = torch.cumsum(bw * bh, 0)
    total = int(ends[-1]) if at.numel() else 0
    if total > most:
        return None
    L = torch.zeros((3, H * W), dtype=f64, device=DEV)
    C = torch.zeros_like(L)
    step, first, done = 30_000_000, 0, 0
    while first < at.numel():
        last = int(torch.searchsorted(ends, done + step, right=True))
        last = min(max(last, first + 1), at.numel())
        a, w_, h_ = at[first:last], bw[first:last], bh[first:last]
        cnt = w_ * h_
        m = int(cnt.sum())
        q = torch.repeat_interleave(torch.arange(a.numel(), device=DEV), cnt, output_size=m)
        t = torch.arange(m, device=DEV) - (torch.cumsum(cnt, 0) - cnt)[q]
        row = torch.div(t, w_[q], rounding_mode="floor")
        di, dj = (t - row * w_[q]).float(), row.float()
        p = a[q]
        ur, vr = (u - i0)[a].float(), (v - j0)[a].float()
        dx, dy = (di + 0.5) - ur[q], (dj + 0.5) - vr[q]
        keep = torch.nonzero(dx * dx + dy * dy <= (r * r)[a].float()[q]).flatten()
        p, q = p[keep], q[keep]
        i, j = i0[p] + di[keep], j0[p] + dj[keep]
        pix = (j * W + i).to(torch.int64)
        q2 = ((i + 0.5 - u[p]) ** 2 + (j + 0.5 - v[p]) ** 2) / sig[p] ** 2
        del t, row, di, dj, dx, dy, i, j, keep
        wgt = torch.exp(-q2)
        if kernel3d:
            wgt = wgt * torch.erf(torch.sqrt((4.0 - q2).clamp_min(0)))
        pix, order = torch.sort(pix, stable=True)
        p, wgt = p[order], wgt[order]
        k = torch.arange(pix.numel(), device=DEV)
        head = torch.ones_like(pix, dtype=torch.bool)
        head[1:] = pix[1:] != pix[:-1]
        start = torch.cummax(torch.where(head, k, torch.zeros_like(k)), 0).values
        for c in range(3):
            x = A[p, c] * wgt
            before = torch.cumsum(x, 0) - x
            depth = L[c][pix] + (before - before[start])
            phi = torch.where(x > 0, -torch.expm1(-x) / x.clamp_min(1e-300), torch.ones_like(x))
            C[c].index_add_(0, pix, torch.exp(-depth) * E[p, c] * wgt * phi)
            L[c].index_add_(0, pix, x)
        done, first = int(ends[last - 1]), last
    return C.reshape(3, H, W)


def _weights():
    """The network's initial weights: splitmix64 bits, Box-Muller, He-normal
    (the last layer a tenth of it), as [9, cin, cout] rounded to bfloat16
    (the operands of its convolutions)."""
    out, state = [], 0
    layers = _convolutions()
    for k, (cin, cout, _) in enumerate(layers):
        n = 9 * cin * cout
        with np.errstate(over="ignore"):
            z = np.uint64(0x9E3779B97F4A7C15) * np.arange(state + 1, state + 2 * n + 1,
                                                          dtype=np.uint64)
            z = (z ^ (z >> np.uint64(30))) * np.uint64(0xBF58476D1CE4E5B9)
            z = (z ^ (z >> np.uint64(27))) * np.uint64(0x94D049BB133111EB)
            z = z ^ (z >> np.uint64(31))
        state += 2 * n
        u = ((z >> np.uint64(11)).astype(np.float64) + 0.5) / 9007199254740992.0
        g = np.sqrt(-2 * np.log(u[0::2])) * np.cos(6.283185307179586 * u[1::2])
        sd = math.sqrt(2 / (9 * cin)) * (0.1 if k == len(layers) - 1 else 1.0)
        w = torch.from_numpy((g * sd).astype(np.float32)).to(DEV).to(torch.bfloat16).double()
        out.append(w.reshape(9, cin, cout))
    return out


def _conv(x, w, b):
    """3 x 3 convolution (zeros outside) of [n, h, w, c] as nine products."""
    n, h, wd, c = x.shape
    pad = torch.nn.functional.pad(x, (0, 0, 1, 1, 1, 1))
    y = b
    for t in range(9):
        part = pad[:, t // 3:t // 3 + h, t % 3:t % 3 + wd].reshape(-1, c)
        y = y + part @ w[t]
    return y.reshape(n, h, wd, -1)


def _network(x, ws, bs):
    """x + net(x) for [n, h, w, 32] inputs."""
    L, k = len(LN.LEVELS), 0
    skips, e = [], x
    for level in range(L):
        if level:
            n, h, w, c = e.shape
            e = e.reshape(n, h // 2, 2, w // 2, 2, c).mean(dim=(2, 4))
        for _ in range(2):
            e = torch.relu(_conv(e, ws[k], bs[k]))
            k += 1
        skips.append(e)
    for level in range(L - 2, -1, -1):
        e = e.repeat_interleave(2, 1).repeat_interleave(2, 2)
        e = torch.cat([e, skips[level]], 3)
        for _ in range(2):
            e = torch.relu(_conv(e, ws[k], bs[k]))
            k += 1
    return x + _conv(e, ws[k], bs[k])


def _zero_bias(ws):
    return [torch.zeros(w.shape[2], dtype=torch.float64, device=DEV) for w in ws]


def _reconstruct(img):
    s = img.mean()
    x = torch.zeros((1, *img.shape[1:], LN.CIN), dtype=torch.float64, device=DEV)
    x[0, :, :, :3] = torch.log1p(img.clamp_min(0) / s).permute(1, 2, 0)
    ws = _weights()
    with torch.no_grad():
        y = _network(x, ws, _zero_bias(ws))
    return (s * torch.expm1(y[0, :, :, :3])).permute(2, 0, 1).contiguous()


def _gradients(case, seed):
    n, size = int(case["images"]), int(case["size"])
    x, t = _training_batch(case, seed)
    x = x.double().reshape(n, size, size, LN.CIN)
    t = t.double().reshape(n, size, size, LN.CIN)
    ws = _weights()
    bs = _zero_bias(ws)
    for p in ws + bs:
        p.requires_grad_(True)
    y = _network(x, ws, bs)
    torch.square(y - t)[..., :3].mean().backward()
    out = dict(y=y.detach().reshape(-1), loss=None)
    for k, (w, b) in enumerate(zip(ws, bs)):
        out["w%02d" % k], out["b%02d" % k] = w.grad.reshape(-1), b.grad
    return out
