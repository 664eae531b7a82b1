"""A hit that the clip distance or the tau_max test rejects stays rejected where
the alpha_min test's right-hand side, K |d_g|^2, overflows FP32.

A disc of thickness 3e-20 through the camera, whose projection is made by
hand: |d_g|^2 reaches 1e38 on some pixels of its 4x4 blocks, times K (about 8)
beyond the largest FP32 number.  With clip distances of zero no pixel may
count it; nor, without them, a pixel for which it lies behind the camera
(half the tile does: the test is made per pixel there).
"""
import numpy as np
import pytest
import torch

import gut_synth as G
from paper_2412_12507_amd import raster as R

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kbuffer", [0, 16, 3])
@pytest.mark.parametrize("rolling", [False, True])
@pytest.mark.parametrize("what", ["clip", "behind"])
def test_rejected_hits(what, rolling, kbuffer):
    print(f"[rejected] {what} rolling {rolling} kbuffer {kbuffer}", flush=True)
    cam = G.camera("pinhole", 16, 16, 8.0, R0=np.eye(3), t0=np.zeros(3))
    if rolling:
        cam = G.with_motion(cam, 0.0, 1e-60)  # (times m^2: still far below the rest)
    m = 3.2e19
    dev = "cuda"
    rec = torch.zeros(1, 16, device=dev)
    # clip: the disc x = 0 around (0, 0, 5).  behind: its plane tilted so that
    # o_g . d_g changes sign at the image's middle row
    rec[0, :4] = torch.tensor([0.0, 0.0, 5.0, 0.99]) if what == "clip" else torch.tensor([0.0, 5.0, 0.0, 0.99])
    rec[0, 4] = m
    rec[0, 9] = 0.2 if what == "behind" else 1.0
    rec[0, 14] = 0.2 if what == "behind" else 1.0
    proj = R.Projection(rect=torch.tensor([[0, 0, 0, 0]], dtype=torch.int16, device=dev),
                        tiles=torch.ones(1, dtype=torch.int32, device=dev), depth=torch.full((1,), 5.0, device=dev),
                        rgb=torch.ones(1, 3, device=dev), record=rec, mean2d=torch.zeros(1, 2, device=dev), cov2d=None,
                        extent=torch.zeros(1, 4, device=dev), n=1, n_cams=1)
    buf = torch.tensor([0, 1, 0], dtype=torch.int32, device=dev)
    bins = R.Bins(ranges=buf[:2].view(1, 2), ids=torch.zeros(1, dtype=torch.int32, device=dev), n_pairs=1, order=buf[2:])
    clip = torch.zeros(256, device=dev) if what == "clip" else None
    img = R.render(proj, bins, [cam], dict(kbuffer=kbuffer), clip=clip)
    nc = img.n_contrib.view(16, 16).cpu()
    if what == "clip":
        assert int(nc.sum()) == 0, nc
    else:
        # o_g . d_g = -0.2^2 * 5 * (y of the ray): rays through the upper half look away
        assert int(nc[:8].sum()) == 0, nc
