"""Camera values as the column arrays that calibration tools return ((4, 1)
distortion coefficients, (3, 1) translations) give the camera that flat lists
give; rows ((1, n)), which have no n elements, are refused."""
import numpy as np
import pytest
import torch

from paper_2412_12507_amd import _lib as L

VALUES = {k: np.random.default_rng(7).normal(size=s) for k, s in
          dict(R0=(3, 3), R1=(3, 3), t0=3, t1=3, k=4).items()}


def camera(**kw):
    cam = dict(model="fisheye", shutter="rolling", width=8, height=9, fx=1.5, fy=2.5, cx=3.5, cy=4.5,
               **{k: v.tolist() for k, v in VALUES.items()})
    return L.camera_struct({**cam, **kw})


FORMS = dict(numpy=lambda a: a, float32=lambda a: a.astype(np.float32), torch=torch.from_numpy,
             objects=lambda a: a.astype(object), list_of_arrays=lambda a: list(a), masked=np.ma.masked_array,
             grad=lambda a: torch.from_numpy(a).requires_grad_(True))


@pytest.mark.filterwarnings("ignore:Conversion of an array:DeprecationWarning")
@pytest.mark.parametrize("form", FORMS)
@pytest.mark.parametrize("key", ["k", "t0", "t1", "R0", "R1"])
def test_column_arrays(key, form):
    a = VALUES[key]
    got = list(getattr(camera(**{key: FORMS[form](a.reshape(-1, 1))}), key))
    want = a.astype(np.float32).astype(np.float64) if form == "float32" else a
    assert got == want.reshape(-1).tolist()


@pytest.mark.parametrize("key,value", [
    ("k", VALUES["k"].reshape(1, 4)), ("t0", VALUES["t0"].reshape(1, 3)), ("k", VALUES["k"].reshape(2, 2)),
    ("t0", VALUES["t0"][:2]), ("R0", np.eye(2)), ("R0", torch.from_numpy(VALUES["R0"].reshape(-1))),
    ("R0", VALUES["R0"].reshape(1, 3, 3)), ("t1", np.float64(1.0))])
def test_other_shapes_are_refused(key, value):
    with pytest.raises((TypeError, IndexError, ValueError)):
        camera(**{key: value})
