"""The two walks of a tile against each other.

A camera alone is rendered by 256-thread blocks whose waves walk lists of pairs
per 4x4 pixel block; four such cameras in one call pass 10000 tiles and are
rendered by 128-thread blocks that walk the pairs one at a time.  Every
pixel's arithmetic is the same, so the images, T, n_contrib and n_eval must
agree bit for bit: at ragged sizes, for every kind of compositing instance,
with lists of every length around a chunk (128) and a batch (256).
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
    ("pinhole", 1003, 637, {}, False),          # 2520 tiles, ragged right and bottom
    ("fisheye", 801, 800, {}, True),
    ("rolling", 800, 799, {}, False),
    ("rolling", 1009, 631, dict(kernel_degree=5), True),
    ("pinhole", 800, 800, dict(kernel_degree=4), False),  # 2500 tiles, four just past the line
])
def test_walks_agree(kind, w, h, params, clip):
    print(f"[walks] {kind} {w}x{h} {params} clip {clip}", flush=True)
    gs = R.GaussianScene.from_host(G.clustered_scene(150000, seed=1002))
    cam = camera(kind, w, h)
    cl = None
    if clip:
        g = torch.Generator(device="cuda").manual_seed(7)
        cl = 5.0 + 6.0 * torch.rand(w * h, generator=g, device="cuda")
    _, bins, one = R.forward(gs, [cam], params, with_eval=True, clip=cl)
    _, _, four = R.forward(gs, [cam] * 4, params, with_eval=True, clip=None if cl is None else cl.repeat(4))
    lens = bins.ranges[:, 1] - bins.ranges[:, 0]
    for lo, hi in ((1, 127), (128, 128), (129, 255), (257, 100000)):
        assert int(((lens >= lo) & (lens <= hi)).sum()) > 0
    n = w * h
    for key in ("rgb", "T", "n_contrib", "n_eval"):
        a, b = getattr(one, key), getattr(four, key)
        for c in range(4):
            assert torch.equal(a, b[c * n:(c + 1) * n]), f"{key} of camera {c}"
