"""gut_bin's list sorts on depths they find hard, against np.lexsort.

Entries of one tile each, so the lists are chosen freely: lengths at the edges
of every sorting kernel (64, 128, 256, 1024, 4096, 16384), and depths that
straddle a power of two (nearly every exponent bit differs), lie in a thin
cluster before a far background (most buckets of the range are empty), hold
long runs of equal depth, or are all equal.  Whole numbers: exact.
"""
import numpy as np
import pytest
import torch

import gut_synth as G
from paper_2412_12507_amd import raster as R

pytestmark = pytest.mark.gpu

LENGTHS = (0, 1, 2, 63, 64, 65, 128, 129, 255, 256, 257, 512, 513, 1000, 1023, 1024, 2000, 4095, 4096, 9000,
           16383, 16384, 16385, 33000)


def depths(kind, L, rng):
    if kind == "straddle":
        return rng.uniform(1.9, 2.1, L)
    if kind == "thin":  # all but one key in a 2e-3 slice of the range
        d = rng.normal(4.0, 1e-3, L)
        d[: min(L, 1)] = 28.0
        return d
    if kind == "two_thin":
        d = np.where(rng.random(L) < 0.5, rng.normal(0.25, 1e-5, L), rng.normal(9.0, 1e-4, L))
        d[: min(L, 1)] = 27.0
        return d
    if kind == "ties":  # a tenth of the keys on one depth
        return np.where(rng.random(L) < 0.1, 3.0, rng.uniform(1.0, 20.0, L))
    if kind == "equal":
        return np.full(L, 7.5)
    return rng.uniform(0.0, 1.0, L)  # denormals to 1: every exponent


@pytest.mark.parametrize("kind", ["straddle", "thin", "two_thin", "ties", "equal", "unit"])
def test_list_sort(kind):
    print(f"[list sort] {kind}", flush=True)
    rng = np.random.default_rng(4100)
    T, n = len(LENGTHS), sum(LENGTHS)
    tile = np.repeat(np.arange(T), LENGTHS)
    d = np.concatenate([depths(kind, L, rng) for L in LENGTHS]).astype(np.float32)
    mix = rng.permutation(n)  # a list's entries come from anywhere in the scene
    tile, d = tile[mix], d[mix]
    cam = G.camera("pinhole", 16 * T, 16, 100.0)
    proj = R.alloc_projection(n, 1)
    proj.rect.copy_(torch.as_tensor(np.stack([tile, 0 * tile, tile, 0 * tile], 1).astype(np.int16)))
    proj.tiles.fill_(1)
    proj.depth.copy_(torch.as_tensor(d))
    bins = R.bin_tiles(proj, [cam], dict(tile_cull=0))
    torch.cuda.synchronize()
    assert bins.n_pairs == n
    assert np.array_equal(np.diff(bins.ranges.cpu().numpy(), axis=1)[:, 0], LENGTHS)
    want = np.lexsort((np.arange(n), d.view(np.uint32), tile))
    assert np.array_equal(bins.ids[:n].cpu().numpy(), want)
