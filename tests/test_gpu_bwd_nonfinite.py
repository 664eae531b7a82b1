"""Loss gradients that are infinite or NaN on single pixels (an ordinary event
under loss scaling) reach the particles those pixels blend, and no others.

Lists of over 100 entries whose 4x4 blocks take different shares of them, so
that in most steps some of a wave's rows stand behind the end of their own
list.  The particles that the pixels do not blend must have the gradients of
the same call without those pixels, to 1e-5 of the largest (both calls sum the
same FP32 terms in FP64, in an order that may vary; a k-buffer call sums in
FP32 what the lanes of a wave and a window of batches share).
"""
import numpy as np
import pytest
import torch

import gut_synth as G
import oracle as O
from paper_2412_12507_amd import raster as R

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind,kbuffer,degree,clip", [
    ("pinhole", 0, 2, False), ("rolling", 0, 2, False), ("pinhole", 0, 4, True), ("rolling", 0, 3, True),
    ("pinhole", 16, 2, False), ("rolling", 16, 2, True), ("pinhole", 3, 4, False)])
@pytest.mark.parametrize("where", ["rgb", "T"])
def test_nonfinite_loss_gradients(kind, kbuffer, degree, clip, where):
    print(f"[nonfinite] {kind} kbuffer={kbuffer} degree={degree} clip={clip} {where}", flush=True)
    w, h = 61, 45
    scene = G.uniform_scene(3000, seed=4300, degree=1, log_scale_mean=-3.2)
    Rm, t = G.look_at((0.0, 0.0, -3.0))
    cam = G.camera("pinhole", w, h, 55.0, R0=Rm, t0=t)
    if kind == "rolling":
        cam = G.with_motion(cam, 0.1, 0.3)
    p = O.default_params(kbuffer=kbuffer, kernel_degree=degree)
    gs = R.GaussianScene.from_host(scene)
    cl = None
    if clip:
        cl = torch.as_tensor(np.random.default_rng(4301).uniform(2.5, 4.5, w * h), dtype=torch.float32, device="cuda")
    proj, bins, img = R.forward(gs, [cam], p, clip=cl)
    lens = bins.ranges[:, 1] - bins.ranges[:, 0]
    assert int(lens.max()) > 256 and int((lens > 100).sum()) >= 4

    def backward(d_rgb, d_T):
        return R.render_backward(gs, proj, bins, [cam], img, d_rgb, d_T, p, clip=cl)

    gen = torch.Generator(device="cuda").manual_seed(4302)
    d_rgb = torch.randn(w * h, 3, generator=gen, device="cuda")
    d_T = torch.randn(w * h, generator=gen, device="cuda")
    bad = torch.tensor([22 * w + 29, 5 * w + 40, 30 * w + 7], device="cuda")
    d_rgb[bad] = 0.0
    d_T[bad] = 0.0
    want = backward(d_rgb, d_T)
    # the particles those pixels blend: their colour or opacity has a gradient
    one, oneT = torch.zeros_like(d_rgb), torch.zeros_like(d_T)
    one[bad] = 1.0
    oneT[bad] = 0.5
    g1 = backward(one, oneT)
    met = (g1["sh"].abs().amax((1, 2)) > 0) | (g1["opacities"] != 0)
    assert 10 < int(met.sum()) < 1500
    values = torch.tensor([float("inf"), float("nan"), -float("inf")], device="cuda")
    if where == "rgb":
        d_rgb[bad] = values[:, None]
    else:
        d_T[bad] = values
    got = backward(d_rgb, d_T)
    torch.cuda.synchronize()
    for key, a in got.items():
        b = want[key]
        a, b = a.reshape(scene.n, -1), b.reshape(scene.n, -1)
        assert torch.isfinite(a[~met]).all(), f"{key}: {int((~torch.isfinite(a[~met])).any(1).sum())} particles"
        err = (a[~met] - b[~met]).abs().max().item()
        assert err <= 1e-5 * b.abs().max().item(), (key, err)
    if where == "rgb":
        assert not torch.isfinite(got["sh"][met]).all()
    assert not torch.isfinite(got["opacities"][met]).all()
