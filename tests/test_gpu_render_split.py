"""Tiles rendered by two blocks against the same tiles rendered by one.

A camera of up to 1280 tiles alone gives every tile two blocks; the same
camera in a call of four splits only its longest lists of 256 entries and
more.  Every pixel's arithmetic is the same, so the images, T, n_contrib and
n_eval must agree bit for bit: at ragged sizes, for every kind of compositing
instance, with lists on both sides of 256 entries.
"""
import numpy as np
import pytest
import torch

import gut_synth as G
from paper_2412_12507_amd import raster as R

pytestmark = pytest.mark.gpu


def camera(kind, w, h):
    Rm, t = G.look_at((0.0, 0.0, -8.0))
    if kind == "pinhole":
        return G.camera("pinhole", w, h, G.pinhole_focal(w), R0=Rm, t0=t)
    c = G.camera("fisheye", w, h, G.fisheye_focal(w), k=G.random_fisheye_k(np.random.default_rng(5)), R0=Rm, t0=t)
    return G.with_motion(c, 0.1, 0.3) if kind == "rolling" else c


@pytest.mark.parametrize("kind,w,h,params,clip", [
    ("pinhole", 637, 483, {}, False),          # 1240 tiles, ragged right and bottom
    ("fisheye", 640, 512, {}, True),           # 1280 tiles, the last size of which all split
    ("rolling", 639, 500, {}, False),
    ("rolling", 500, 333, dict(kernel_degree=5), True),
    ("pinhole", 17, 9, dict(kernel_degree=4), False),
])
def test_split_equals_whole(kind, w, h, params, clip):
    print(f"[split] {kind} {w}x{h} {params} clip {clip}", flush=True)
    gs = R.GaussianScene.from_host(G.clustered_scene(120000, seed=1002))
    cam = camera(kind, w, h)
    cl = None
    if clip:
        g = torch.Generator(device="cuda").manual_seed(7)
        cl = 5.0 + 6.0 * torch.rand(w * h, generator=g, device="cuda")
    _, bins, one = R.forward(gs, [cam], params, with_eval=True, clip=cl)
    _, _, four = R.forward(gs, [cam] * 4, params, with_eval=True, clip=None if cl is None else cl.repeat(4))
    lens = (bins.ranges[:, 1] - bins.ranges[:, 0])
    if w > 100:
        assert int((lens >= 256).sum()) > 20 and int((lens < 256).sum()) > 20
    n = w * h
    for key in ("rgb", "T", "n_contrib", "n_eval"):
        a, b = getattr(one, key), getattr(four, key)
        for c in range(4):
            assert torch.equal(a, b[c * n:(c + 1) * n]), f"{key} of camera {c}"
