"""The float32 field kernel's test of bucket entries before they are staged
(buckets of more than 64 entries): it leaves out nothing that the reach test
would pass, so a tiling of long buckets and one of short buckets hold the same
candidates in the same order and give the same bits."""
import numpy as np
import pytest

from paper_2101_05031_amd import api, synth

from gpu_util import bin_lattice

pytestmark = pytest.mark.gpu


def struts_ending_near(length, n=200, R=0.6, seed=5):
    """Struts with one end about the grid's window and the other `length` away."""
    rng = np.random.default_rng(seed)
    a = rng.uniform([-0.5, -0.5, -0.6], [2.4, 2.4, 1.0], size=(n, 3))
    dirs = rng.normal(size=(n, 3))
    dirs /= np.linalg.norm(dirs, axis=1)[:, None]
    nodes = np.concatenate([a, a + length * dirs]).astype(np.float32)
    edges = np.stack([np.arange(n), np.arange(n) + n], axis=1).astype(np.int32)
    edges[::2] = edges[::2, ::-1]
    w = rng.uniform(0.05, 0.5, size=n).astype(np.float32)
    return synth.Lattice(nodes, edges, w, R, 1.0)


# in supports: within the block, ordinary, and where float32 places along the
# strut are coarse against the test's margin of 1e-4 R
@pytest.mark.parametrize("length", [0.2, 5.0, 5000.0])
def test_long_and_short_buckets_alike(length):
    lat = struts_ending_near(length * 0.6)
    grid = synth.Grid(0.0, 0.0, 0.02, 0.02, 93, 87, 0.0, 0.04, 11)
    base = base_stats = None
    for tile, slab in [(8, 8), (64, 8), (8, 1), (32, 16), (64, 3)]:
        print(f"length {length} tile {tile} slab {slab}", flush=True)
        b = bin_lattice(lat, grid, tile=tile, slab=slab)
        f = api.slice_field(b, 0, grid.n_slices).cpu().numpy()
        st = api.slice_field_stats(b, 0, grid.n_slices)
        if base is None:
            base, base_stats = f, st
            assert st["candidates"] > 64 * 64
        assert np.array_equal(f.view(np.uint32), base.view(np.uint32))
        assert st == base_stats
