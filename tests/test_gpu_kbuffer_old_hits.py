"""k-buffer backward: hits that stay in the buffer until the list has gone on
by more than the LDS window.

A large particle in front of two tiles, and behind it some 580 particles a
tile so small that no pixel ever meets 16 of them: the buffers never fill, and
every hit is blended after the end of the list.  The large one, first in
both lists, has left the window by then (it reaches back to the last multiple
of 256 less 256, here 256), so its values go to the FP64 sums and its colour is
read through the list.

- Against the FP64 oracle, at the gradients' usual bound (1e-3).
- The sums really are FP64 ones: a tile's loss gradients that add up past the
  largest FP32 number, which the other tile's take back below it, scale as the
  same ones 2^100 times smaller (exact scaling; 1e-5 for the FP32 terms' sums
  in lanes, whose order may vary).
"""
import numpy as np
import pytest
import torch

import gut_synth as G
import oracle as O
from paper_2412_12507_amd import raster as R
from parity import grad_compare

pytestmark = pytest.mark.gpu

W, H, N = 32, 16, 1160


def setup(kind):
    rng = np.random.default_rng(4406)
    Rm, t = G.look_at((0.0, 0.0, -3.0))
    cam = G.camera("pinhole", W, H, 60.0, R0=Rm, t0=t)
    if kind == "rolling":
        cam = G.with_motion(cam, 0.002, 0.01)
    z = rng.uniform(0.0, 1.0, N)
    px = np.stack([rng.uniform(0.5, W - 0.5, N), rng.uniform(0.5, H - 0.5, N)], 1)
    cam_xyz = np.stack([(px[:, 0] - W / 2) / 60.0 * (z + 3), (px[:, 1] - H / 2) / 60.0 * (z + 3), z + 3], 1)
    cam_xyz[0] = (0.0, 0.0, 2.0)
    means = (cam_xyz - t) @ Rm  # R^T (x - t)
    log_s = np.full((N, 3), np.log(4e-3))
    log_s[0] = np.log(0.6)
    logit = np.zeros(N)
    logit[0] = 0.8
    quats = np.tile([1.0, 0.0, 0.0, 0.0], (N, 1))
    sh = rng.uniform(-0.8, 0.8, (N, 1, 3))
    return G.scene_from_raw(means, log_s, quats, logit, sh, 0), cam


@pytest.mark.parametrize("kind", ["pinhole", "rolling"])
def test_old_hits(kind):
    print(f"[old hits] {kind}", flush=True)
    scene, cam = setup(kind)
    p = O.default_params(kbuffer=16)
    gs = R.GaussianScene.from_host(scene)
    proj, bins, img = R.forward(gs, [cam], p)
    lens = (bins.ranges[:, 1] - bins.ranges[:, 0]).tolist()
    assert len(lens) == 2 and all(512 < x <= 640 for x in lens), lens
    assert [int(bins.ids[int(r)]) for r in bins.ranges[:, 0]] == [0, 0]
    assert 1 <= int(img.n_contrib.min()) and int(img.n_contrib.max()) <= 16
    # the oracle's gradients
    pr = O.project(scene, cam, p)
    ob = O.bin_tiles(pr, cam, p)
    res = O.render(scene, pr, cam, ob, p)
    amb = O.to_image(res, cam, p, key="n_alt") > 0
    rng = np.random.default_rng(4401)
    wC, wT = rng.normal(size=(H, W, 3)), rng.normal(size=(H, W))
    wC[amb] = 0
    wT[amb] = 0
    assert amb.mean() < 0.5
    g_ora = O.backward(scene, pr, cam, ob, wC, wT, p)

    def backward(d_rgb, d_T=None):
        d_T = None if d_T is None else torch.as_tensor(d_T.reshape(-1), dtype=torch.float32, device="cuda")
        d_rgb = torch.as_tensor(d_rgb.reshape(-1, 3), dtype=torch.float32, device="cuda")
        return R.render_backward(gs, proj, bins, [cam], img, d_rgb, d_T, p)

    got = backward(wC, wT)
    # (spheres: the quaternions' gradient is zero, in the oracle up to its rounding)
    assert np.abs(g_ora.pop("quats")).max() < 1e-10 and got["quats"].abs().max() < 1e-6 * got["means"].abs().max()
    for key, v in grad_compare(got, g_ora).items():
        assert v["rel"] <= 1e-3 and v["elem_fail"] == 0, (key, v)
    # sums past FP32's range
    x = np.zeros((H, W, 3))
    x[:, :16], x[:, 16:] = 1.0, -0.6
    a = backward(np.where(x > 0, x, 0.0))["sh"][0, 0].double().cpu().numpy()  # (the tile's sum, times Y_00)
    scale = 2.0 ** np.ceil(np.log2(3.4e38 * 1.1 * 0.28209479 / np.abs(a).min()))
    assert (np.abs(a) * scale / 0.28209479 * 0.55 < 3.3e38).all()
    big = backward(x * scale)["sh"][0, 0].double().cpu().numpy()
    small = backward(x * (scale * 2.0 ** -100))["sh"][0, 0].double().cpu().numpy() * 2.0 ** 100
    assert np.isfinite(big).all(), big
    assert (np.abs(big - small) <= 1e-5 * np.abs(small)).all(), (big, small)
