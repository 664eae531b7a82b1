"""The fisheye limit's scan, which passes over spans by a bound, against the
plain one (tests/host/fisheye_limit_test.cpp); and camera marshalling of the
forms a pose may have."""
import os
import shutil
import subprocess

import numpy as np
import pytest
import torch

from paper_2412_12507_amd import _lib as L

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not available")
def test_fisheye_limit(tmp_path):
    exe = str(tmp_path / "fisheye_limit")
    subprocess.run(["g++", "-std=c++17", "-O2", "-I", os.path.join(ROOT, "paper_2412_12507_amd", "csrc"),
                    os.path.join(ROOT, "tests", "host", "fisheye_limit_test.cpp"), "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and "ALL OK" in r.stdout, r.stdout


@pytest.mark.parametrize("form", [lambda a: a, lambda a: a.tolist(), lambda a: list(a), lambda a: a.astype(np.float32),
                                  torch.from_numpy, lambda a: a.T.copy().T, lambda a: a.reshape(-1), lambda a: tuple(a.ravel())])
def test_camera_forms(form):
    R0, R1, t0, t1, k = (np.random.default_rng(6).normal(size=s) for s in ((3, 3), (3, 3), 3, 3, 4))
    c = L.camera_struct(dict(model="fisheye", shutter="rolling", width=8, height=9, fx=1.5, fy=2.5, cx=3.5, cy=4.5,
                             k=form(k), R0=form(R0), R1=form(R1), t0=form(t0), t1=form(t1)))
    for got, a in ((c.R0, R0), (c.R1, R1), (c.t0, t0), (c.t1, t1), (c.k, k)):
        want = np.asarray(form(a), dtype=np.float64).reshape(-1)
        assert list(got) == want.tolist()
    assert (c.model, c.shutter, c.width, c.height, c.fx, c.cy) == (1, 1, 8, 9, 1.5, 4.5)
