"""The tile-order backward by pairs (3072 tiles and more with fewer than
tiles / 650 particles a tile) and by lists.

- By pairs against the FP64 oracle on sampled tiles, at the gradients' usual
  bound: pinhole, fisheye and rolling shutter, both responses, with clip
  distances, at a ragged size, on lists of more than half a batch (64) and of more
  than a batch (128).
- By pairs against lists: particles behind the camera move the call over the
  line; the gradients of the others agree to 1e-5 of the largest (the same FP32
  terms, summed over 32 or 16 pixels in FP32 and from there in FP64).
- By pairs, loss gradients that are not finite reach what their pixels blend,
  and nothing else.
"""
import numpy as np
import pytest
import torch

import gut_synth as G
import oracle as O
from paper_2412_12507_amd import raster as R
from parity import sampled_backward_check
from test_gpu_render_walk_rule import padded

pytestmark = pytest.mark.gpu

W, H, N, TILES = 1277, 715, 9000, 3600


def setup(kind, clip=False):
    scene = G.clustered_scene(N, seed=1002, degree=1, log_scale_mean=-1.6)
    Rm, t = G.look_at((0.0, 0.0, -8.0))
    if kind == "pinhole":
        cam = G.camera("pinhole", W, H, G.pinhole_focal(W), R0=Rm, t0=t)
    else:
        cam = G.camera("fisheye", W, H, G.fisheye_focal(W), k=G.random_fisheye_k(np.random.default_rng(5)), R0=Rm, t0=t)
        if kind == "rolling":
            cam = G.with_motion(cam, 0.1, 0.3)
    cl = np.random.default_rng(4600).uniform(6.0, 11.0, (H, W)).astype(np.float32) if clip else None
    assert R.num_tiles([cam]) == TILES and 650 * N < TILES * TILES
    return scene, cam, cl


@pytest.mark.parametrize("kind,degree,clip", [
    ("pinhole", 2, False), ("fisheye", 2, True), ("rolling", 2, False), ("rolling", 3, True), ("pinhole", 4, False)])
def test_pairs_against_oracle(kind, degree, clip):
    print(f"[bwd by pairs, oracle] {kind} degree {degree} clip {clip}", flush=True)
    scene, cam, cl = setup(kind, clip)
    p = O.default_params(kernel_degree=degree)
    gs = R.GaussianScene.from_host(scene)
    bins = R.bin_tiles(R.project(gs, [cam], p), [cam], p)
    lens = bins.ranges[:, 1] - bins.ranges[:, 0]
    for lo, hi in ((65, 127), (129, 100000)):
        assert int(((lens >= lo) & (lens <= hi)).sum()) > 0
    rep = sampled_backward_check(scene, cam, p, clip=cl)
    print({k: (v["rel"], v["elem_fail"]) for k, v in rep.items()})
    for key, v in rep.items():
        assert v["rel"] <= 1e-3 and v["elem_fail"] == 0, (key, v)


@pytest.mark.parametrize("kind,degree,clip", [("pinhole", 2, False), ("fisheye", 3, False), ("rolling", 2, True)])
def test_pairs_against_lists(kind, degree, clip):
    print(f"[bwd pairs against lists] {kind} degree {degree} clip {clip}", flush=True)
    scene, cam, cl = setup(kind, clip)
    p = O.default_params(kernel_degree=degree)
    cl = None if cl is None else torch.as_tensor(cl.reshape(-1), device="cuda")
    gen = torch.Generator(device="cuda").manual_seed(4601)
    d_rgb = torch.randn(W * H, 3, generator=gen, device="cuda")
    d_T = torch.randn(W * H, generator=gen, device="cuda")
    g = []
    for sc in (scene, padded(scene, 16000)):
        gs = R.GaussianScene.from_host(sc)
        proj, bins, img = R.forward(gs, [cam], p, clip=cl)
        g.append(R.render_backward(gs, proj, bins, [cam], img, d_rgb, d_T, p, clip=cl))
    assert 650 * (N + 16000) >= TILES * TILES
    for key, a in g[0].items():
        b = g[1][key]
        assert (b[N:] == 0).all()
        assert (a - b[:N]).abs().max().item() <= 1e-5 * b.abs().max().item(), key


@pytest.mark.parametrize("kind,degree", [("pinhole", 2), ("rolling", 4)])
def test_pairs_nonfinite(kind, degree):
    print(f"[bwd by pairs, nonfinite] {kind} degree {degree}", flush=True)
    scene, cam, _ = setup(kind)
    p = O.default_params(kernel_degree=degree)
    gs = R.GaussianScene.from_host(scene)
    proj, bins, img = R.forward(gs, [cam], p)
    gen = torch.Generator(device="cuda").manual_seed(4602)
    d_rgb = torch.randn(W * H, 3, generator=gen, device="cuda")
    # pixels with contributors, one in each half of a tile
    nc = img.n_contrib.view(H, W)
    ys, xs = torch.nonzero(nc > 20, as_tuple=True)
    low = ys % 16 < 8
    bad = torch.stack([(ys * W + xs)[low][1000], (ys * W + xs)[~low][3000], (ys * W + xs)[low][-1000]])

    def backward(d):
        return R.render_backward(gs, proj, bins, [cam], img, d, None, p)

    d_rgb[bad] = 0.0
    want = backward(d_rgb)
    one = torch.zeros_like(d_rgb)
    one[bad] = 1.0
    g1 = backward(one)
    met = (g1["sh"].abs().amax((1, 2)) > 0) | (g1["opacities"] != 0)
    assert 3 < int(met.sum()) < N // 4
    d_rgb[bad] = torch.tensor([float("inf"), float("nan"), -float("inf")], device="cuda")[:, None]
    got = backward(d_rgb)
    for key, a in got.items():
        a, b = a.reshape(N, -1), want[key].reshape(N, -1)
        assert torch.isfinite(a[~met]).all(), key
        assert (a[~met] - b[~met]).abs().max().item() <= 1e-5 * b.abs().max().item(), key
    assert not torch.isfinite(got["sh"][met]).all()
