"""gut_bin queues only the sorts that a call's lists need: list sets whose
longest is at the edge of each sort, in an image of the most tiles that one
short-list launch takes and of one more, and calls of one block of entries
(which have no column scan).  Against np.lexsort: whole numbers, exact."""
import numpy as np
import pytest
import torch

import gut_synth as G
from paper_2412_12507_amd import raster as R

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tiles", [3328, 3329])
@pytest.mark.parametrize("equal", [False, True])
@pytest.mark.parametrize("longest", [1, 63, 255, 256, 1023, 1024, 4095, 4096, 16385])
def test_longest(longest, equal, tiles):
    print(f"[bin launches] longest={longest} equal={equal} tiles={tiles}", flush=True)
    rng = np.random.default_rng(4300)
    lens = np.array([1, 2, longest, 0, 200, 255, 128][: 3 if longest < 256 else 7])
    tile = np.repeat(rng.choice(tiles, len(lens), replace=False), lens)
    n = len(tile)
    tile = tile[rng.permutation(n)]
    d = (np.full(n, 2.5) if equal else rng.uniform(1.9, 2.1, n)).astype(np.float32)
    cam = G.camera("pinhole", 16 * tiles, 16, 100.0)
    proj = R.alloc_projection(n, 1)
    proj.rect.copy_(torch.as_tensor(np.stack([tile, 0 * tile, tile, 0 * tile], 1).astype(np.int16)))
    proj.tiles.fill_(1)
    proj.depth.copy_(torch.as_tensor(d))
    for _ in range(2):
        bins = R.bin_tiles(proj, [cam], dict(tile_cull=0))
        torch.cuda.synchronize()
        assert bins.n_pairs == n
        assert np.array_equal(np.diff(bins.ranges.cpu().numpy(), axis=1)[:, 0], np.bincount(tile, minlength=tiles))
        want = np.lexsort((np.arange(n), d.view(np.uint32), tile))
        assert np.array_equal(bins.ids[:n].cpu().numpy(), want)
