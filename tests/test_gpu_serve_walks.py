"""A served request of six 800x600 cameras (11400 tiles: the pair walk) against
each of its cameras served and rendered alone (1900 tiles: the list walk), bit
for bit, under both shutters and for both responses."""
import numpy as np
import pytest
import torch

import gut_synth as G
from paper_2412_12507_amd import raster as R
from paper_2412_12507_amd.serve import Server, render_sequential

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rolling", [False, True])
@pytest.mark.parametrize("params", [{}, dict(kernel_degree=4)])
def test_batch_by_pairs_equals_alone_by_lists(rolling, params):
    print(f"[serve walks] rolling {rolling} {params}", flush=True)
    gs = R.GaussianScene.from_host(G.clustered_scene(30000, seed=1003))
    rng = np.random.default_rng(4500)
    cams = []
    for _ in range(6):
        Rm, t = G.look_at(G.random_eye(rng))
        c = G.camera("fisheye", 800, 600, G.fisheye_focal(800), k=G.random_fisheye_k(rng), R0=Rm, t0=t)
        cams.append(G.with_motion(c, 0.1, 0.3) if rolling else c)
    with Server(gs, params, mem_budget_bytes=2 << 30, max_slots=2, max_batch_cams=8) as srv:
        together = srv.wait(srv.submit(cams)[0])
        one = [srv.wait(srv.submit([c])[0])[0] for c in cams]
    alone = render_sequential(gs, cams, params)
    for a, b, c in zip(together, one, alone):
        assert torch.equal(a, c) and torch.equal(b, c)
