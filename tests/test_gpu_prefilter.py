"""The float32 field kernel's test of bucket entries before they are staged
(buckets of more than 64 entries): it leaves out nothing that the reach test
would pass, so a tiling of long buckets and one of short buckets hold the same
candidates in the same order and give the same bits.  The general kernel
(float64, the Gaussian, coarse planes) tests its (strut, plane) pairs in
float32 first, where a slab holds more than one plane, to the same effect."""
import dataclasses

import numpy as np
import pytest

from paper_2101_05031_amd import api, synth

from gpu_util import assert_field_close, bin_lattice

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


KINDS = ["f64", "f64 supports", "f64 gauss", "f32 gauss", "f32 wide gauss", "f32 coarse"]


def general_case(kind, length, unit=1.0):
    """Struts and a grid of the general field kernel, all lengths times
    `unit`; the field does not depend on the unit (a term is the weight times a
    length)."""
    lat = struts_ending_near(length * 0.6)
    dtype = np.float64 if kind.startswith("f64") else np.float32
    lat = dataclasses.replace(lat, nodes=(lat.nodes * unit).astype(dtype),
                              weight=(lat.weight / unit).astype(dtype), R=lat.R * unit)
    if "supports" in kind:
        sup = np.random.default_rng(8).uniform(0.3, 1.0, size=lat.n_edges) * lat.R
        lat = dataclasses.replace(lat, support=sup.astype(dtype))
    if "gauss" in kind:
        lat = dataclasses.replace(lat, kernel="gauss", sigma=lat.R / (4 if "wide" in kind else 3))
    dz = 0.3 if kind == "f32 coarse" else 0.04
    grid = synth.Grid(0.0, 0.0, 0.02 * unit, 0.02 * unit, 93, 87, 0.0, dz * unit, 11)
    return lat, grid


def field_bits(lat, grid, tile, slab):
    f = api.slice_field(bin_lattice(lat, grid, tile=tile, slab=slab), 0, grid.n_slices)
    return f.cpu().numpy().view(np.uint64 if f.element_size() == 8 else np.uint32)


# (one plane per slab: no test of pairs.  With per-strut supports the strut
# order starts with the first slab, so the sums' order, not their terms,
# depends on the slab depth.)
@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("length", [0.2, 5.0, 5000.0])
def test_pairs_left_out_do_not_reach(length, kind):
    lat, grid = general_case(kind, length)
    base = field_bits(lat, grid, 8, 1)
    assert np.count_nonzero(base) > base.size // 50
    for tile, slab in [(8, 8), (32, 16), (16, 4), (64, 3), (16, 2)]:
        print(f"{kind} length {length} tile {tile} slab {slab}", flush=True)
        got = field_bits(lat, grid, tile, slab)
        if "supports" in kind:
            assert_field_close(got.view(np.float64), base.view(np.float64), lat.C, 1e-12)
        else:
            assert np.array_equal(got, base)


# units of powers of two: every float64 and float32 step scales exactly
@pytest.mark.parametrize("kind,powers", [(k, (-60, -43, -37, -20, 20, 33, 45, 60)) for k in KINDS[:3]] +
                         [(k, (-43, -37, -20, 20, 33, 45)) for k in KINDS[3:5]] +
                         [("f32 coarse", (-20, 20))])
def test_field_does_not_depend_on_the_unit(kind, powers):
    lat, grid = general_case(kind, 5.0)
    for tile, slab in [(16, 1), (16, 8), (32, 16)]:
        base = field_bits(*general_case(kind, 5.0), tile, slab)
        for p in powers:
            print(f"{kind} unit 2^{p} tile {tile} slab {slab}", flush=True)
            got = field_bits(*general_case(kind, 5.0, 2.0 ** p), tile, slab)
            assert np.array_equal(got, base)
