"""One camera by either walk of a tile: the walk follows the launch's tiles and
the particles a tile, so particles behind the camera, which no list holds,
move a render from the pair walk to the list walk and must not move a bit of
its image, T, n_contrib and n_eval.  (At 3600 tiles lists from 24
particles a tile on.)  And a 3840x2160 camera alone, by pairs, against the same camera in a
launch of two.
"""
import numpy as np
import pytest
import torch

import gut_synth as G
from paper_2412_12507_amd import raster as R

pytestmark = pytest.mark.gpu

KEYS = ("rgb", "T", "n_contrib", "n_eval")


def padded(scene, m):
    """The scene with m more particles behind the camera at z = -8."""
    f = lambda a, b: np.concatenate([a, b]).astype(np.float32)
    rep = lambda a: np.repeat(a[:1], m, 0)
    means = np.tile(np.float32([0.0, 0.0, -60.0]), (m, 1))
    return G.Scene(f(scene.means, means), f(scene.scales, rep(scene.scales)), f(scene.quats, rep(scene.quats)),
                   f(scene.opacities, rep(scene.opacities)), f(scene.sh, rep(scene.sh)), scene.sh_degree,
                   f(scene.log_scales, rep(scene.log_scales)), f(scene.logit_opacities, rep(scene.logit_opacities)))


@pytest.mark.parametrize("rolling,params,clip", [
    (False, {}, False), (False, dict(kernel_degree=4), True), (True, {}, False), (True, dict(kernel_degree=3), True)])
def test_rule_by_particles(rolling, params, clip):
    print(f"[walk rule] rolling {rolling} {params} clip {clip}", flush=True)
    w, h = 1277, 715
    scene = G.clustered_scene(20000, seed=1002, log_scale_mean=-3.0)
    Rm, t = G.look_at((0.0, 0.0, -8.0))
    cam = G.camera("pinhole", w, h, G.pinhole_focal(w), R0=Rm, t0=t)
    if rolling:
        cam = G.with_motion(cam, 0.02, 0.1)
    cl = None
    if clip:
        g = torch.Generator(device="cuda").manual_seed(8)
        cl = 5.0 + 6.0 * torch.rand(w * h, generator=g, device="cuda")
    assert R.num_tiles([cam]) == 3600
    _, b0, few = R.forward(R.GaussianScene.from_host(scene), [cam], params, with_eval=True, clip=cl)
    _, b1, many = R.forward(R.GaussianScene.from_host(padded(scene, 80000)), [cam], params, with_eval=True, clip=cl)
    assert b0.n_pairs == b1.n_pairs > 50000
    for key in KEYS:
        assert torch.equal(getattr(few, key), getattr(many, key)), key


def test_4k_camera_alone():
    print("[walk rule] 3840x2160", flush=True)
    w, h = 3840, 2160
    gs = R.GaussianScene.from_host(G.clustered_scene(150000, seed=1002))
    Rm, t = G.look_at((0.0, 0.0, -8.0))
    cam = G.camera("pinhole", w, h, G.pinhole_focal(w), R0=Rm, t0=t)
    _, bins, img = R.forward(gs, [cam], None, with_eval=True)
    assert int((bins.ranges[:, 1] - bins.ranges[:, 0]).max()) > 128
    # the same camera twice in one call: the launch of several cameras
    _, _, two = R.forward(gs, [cam, cam], None, with_eval=True)
    n = w * h
    for key in KEYS:
        a, b = getattr(img, key), getattr(two, key)
        assert torch.equal(a, b[:n]) and torch.equal(a, b[n:]), key
