"""gut_bin's lists do not depend on how many blocks the entries go to.

The same projection binned with the workspace gut_bin_workspace_bytes asks for
and with one of ceil(n / 8192) count-matrix rows (the least gut_bin takes),
which makes it use fewer blocks: the ranges and the sorted ids must agree
exactly, at entry counts around a unit (64), a block's least (1024) and most
(8192) entries, for one and three cameras.
"""
import ctypes as C

import numpy as np
import pytest
import torch

import gut_synth as G
from paper_2412_12507_amd import _lib as L
from paper_2412_12507_amd import raster as R

pytestmark = pytest.mark.gpu


def al(x):
    return (x + 255) & ~255


@pytest.mark.parametrize("n_cams", [1, 3])
@pytest.mark.parametrize("n", [1, 63, 65, 1023, 1024, 1025, 8192, 8193, 40000])
def test_blocks(n, n_cams):
    print(f"[bin blocks] n={n} cams={n_cams}", flush=True)
    lib = L.load()
    gs = R.GaussianScene.from_host(G.clustered_scene(n, seed=1002, degree=0))
    cams = [G.config2_cameras(321, 181)[1], G.config2_cameras(250, 99)[0], G.config3_camera(400, 300)][:n_cams]
    proj = R.project(gs, cams)
    bins = R.bin_tiles(proj, cams)
    T, arr, p = R.num_tiles(cams), L.camera_array(cams), L.params_struct()
    cap = bins.ids.shape[0]
    least = al(-(-n // 8192) * T * 4) + 4096 + al(4 * T) + 2 * al(8 * cap)
    full = lib.gut_bin_workspace_bytes(n, arr, n_cams, cap)
    assert least <= full and (least < full or n <= 1024)
    out = []
    for size in (full, least):
        ws = torch.empty(size, dtype=torch.uint8, device="cuda")
        rng = torch.empty(3 * T, dtype=torch.int32, device="cuda")
        ids = torch.empty(cap, dtype=torch.int32, device="cuda")
        P, ps = C.c_int64(0), proj.struct()
        L.check(lib.gut_bin(L.ref(ps), n, arr, n_cams, L.ref(p), C.c_void_p(ws.data_ptr()), size, cap,
                            C.c_void_p(rng.data_ptr()), C.c_void_p(ids.data_ptr()), C.byref(P),
                            C.c_void_p(torch.cuda.current_stream().cuda_stream)), "gut_bin")
        torch.cuda.synchronize()
        out.append((P.value, rng[:2 * T].cpu().numpy(), ids[:P.value].cpu().numpy()))
    assert out[0][0] == out[1][0] == bins.n_pairs
    assert np.array_equal(out[0][1], out[1][1]) and np.array_equal(out[0][2], out[1][2])
    assert np.array_equal(out[0][1], bins.ranges.cpu().numpy().reshape(-1))
