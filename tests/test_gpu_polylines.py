"""GPU parity of slice_polylines (sub-pixel contours and chaining) with the
oracle (oracle/polylines.py), on the GPU's own field."""
import copy

import numpy as np
import pytest
import torch

from oracle import contours as OC
from oracle import polylines as PL
from paper_2101_05031_amd import _native as N
from paper_2101_05031_amd import api, synth

from gpu_util import bin_lattice

pytestmark = pytest.mark.gpu


def small_kuhn():
    lat = synth.kuhn_lattice(6, 24.0, seed=21)
    grid = synth.grid_for(lat, 301, 283, 27, dz=0.83)     # ragged W, H
    return lat, grid


def p1():
    lat, grid = synth.config("P1")
    return lat, grid


def _close(got, ref):
    """float32 output of a float64-exact value: a few units in the last place."""
    return np.all(np.abs(got - ref) <= 4e-7 * np.maximum(1.0, np.abs(ref)) + 1e-6)


def check_planes(lat, field, segs, off, chain, rank, what):
    fh = field.cpu().numpy().astype(np.float64)
    segs = segs.cpu().numpy().astype(np.float64)
    off = off.cpu().numpy()
    chain = chain.cpu().numpy()
    rank = rank.cpu().numpy()
    n_open = 0
    for k in range(fh.shape[0]):
        a, b = off[k], off[k + 1]
        ref = PL.segments_subpixel(fh[k], lat.C)
        assert b - a == len(ref), what
        assert _close(segs[a:b], ref), f"{what}: plane {k} endpoints"
        succ, rc, rr = PL.chains(fh[k] >= lat.C)
        assert np.array_equal(chain[a:b], rc), f"{what}: plane {k} chains"
        assert np.array_equal(rank[a:b], rr), f"{what}: plane {k} ranks"
        # joints coincide bitwise: s ends where its successor starts
        has = succ >= 0
        assert np.array_equal(segs[a:b][has, 2:], segs[a:b][succ[has], :2])
        n_open += int(np.sum(~has))
    return n_open


@pytest.mark.parametrize("case", ["kuhn", "P1"])
def test_polylines_match_oracle(case):
    lat, grid = {"kuhn": small_kuhn, "P1": p1}[case]()
    b = bin_lattice(lat, grid)
    nk = min(grid.n_slices, 10)
    f = api.slice_field(b, 0, nk)
    segs, off, chain, rank = api.slice_polylines(b, f)
    # same segments and order as slice_contours, endpoints moved
    msegs, moff, _ = api.slice_contours(b, f)
    assert torch.equal(off, moff) and len(segs) == len(msegs) > 0
    n_open = check_planes(lat, f, segs, off, chain, rank, case)
    assert n_open == 0                  # the grid's margin closes every contour


def test_polylines_open_chains_on_a_window():
    """A grid window that cuts through the lattice: contours leave the window,
    so chains start and end on its border."""
    lat, grid = small_kuhn()
    win = copy.copy(grid)
    win.x0 = grid.x0 + 90 * grid.dx
    win.y0 = grid.y0 + 70 * grid.dy
    win.W, win.H = 131, 117
    win.n_slices = 6
    b = bin_lattice(lat, win)
    f = api.slice_field(b, 0, win.n_slices)
    segs, off, chain, rank = api.slice_polylines(b, f)
    n_open = check_planes(lat, f, segs, off, chain, rank, "window")
    assert n_open > 0


def test_polylines_capacity_and_repeatability():
    lat, grid = small_kuhn()
    b = bin_lattice(lat, grid)
    f = api.slice_field(b, 3, 4)
    segs, off, chain, rank = api.slice_polylines(b, f)
    segs2, off2, chain2, rank2 = api.slice_polylines(b, f)
    assert torch.equal(segs.view(torch.int32), segs2.view(torch.int32))
    assert torch.equal(chain, chain2) and torch.equal(rank, rank2)
    import ctypes
    t = ctypes.c_int64()
    small = torch.empty((len(segs) - 1, 4), dtype=torch.float32, device="cuda")
    o3 = torch.empty(5, dtype=torch.int64, device="cuda")
    st = N.lib().slice_polylines(b.handle, 4, api._ptr(f), api._ptr(small), len(segs) - 1,
                                 api._ptr(o3), None, None, ctypes.byref(t), api._stream())
    assert st == N.LSL_ECAPACITY and t.value == len(segs)
    assert torch.equal(o3, off)
    # without chains: the same segments
    s3, _, c3, r3 = api.slice_polylines(b, f, chains=False)
    assert c3 is None and torch.equal(s3.view(torch.int32), segs.view(torch.int32))


def _stripes(H, W, period, sheared):
    """Bars (walls of segments one list index apart per row) or a slope."""
    j, i = np.mgrid[0:H, 0:W]
    t = (i + (j // 3 if sheared else 0)) % (2 * period)
    return np.where(t < period, 1.5, 0.5)


@pytest.mark.parametrize("W,H,nk", [(2, 2, 1), (9, 7, 3), (64, 257, 2), (520, 131, 1)])
@pytest.mark.parametrize("pattern", ["noise", "bars", "shear", "spiral", "ring"])
def test_chains_of_every_shape(pattern, W, H, nk):
    """Chains shorter and longer than the walk between two jump stations:
    single-pixel loops and saddles, long open walls whose segments lie a
    constant stride apart, one long spiral, a loop around the whole plane."""
    rng = np.random.default_rng(W + H)
    if pattern == "noise":
        f = rng.uniform(0.0, 2.0, size=(nk, H, W))
    elif pattern in ("bars", "shear"):
        f = np.stack([_stripes(H, W, 3 + k, pattern == "shear") for k in range(nk)])
    elif pattern == "spiral":
        j, i = np.mgrid[0:H, 0:W]
        x, y = i - W / 2.0, j - H / 2.0
        f = np.stack([1.0 + np.sin(np.hypot(x, y) + np.arctan2(y, x) + k) for k in range(nk)])
    else:
        f = np.zeros((nk, H, W))
        f[:, 1:-1, 1:-1] = 2.0
    lat = synth.tiny_lattice("one", np.float32)
    b = bin_lattice(lat, synth.grid_for(lat, max(W, 8), max(H, 8), nk, dz=0.1))
    g = copy.copy(b.grid)
    g.W, g.H = W, H
    b = bin_lattice(lat, g)
    field = torch.from_numpy(f.astype(np.float32)).cuda()
    segs, off, chain, rank = api.slice_polylines(b, field)
    if len(segs):
        check_planes(lat, field, segs, off, chain, rank, pattern)


@pytest.mark.parametrize("walls,H", [(86, 700), (88, 700), (144, 701), (234, 300), (610, 2000)])
def test_walls_a_constant_stride_apart(walls, H):
    """Bars of one pixel: every row holds one segment of each wall, so a wall's
    segments lie `walls` places apart in the list (144 and 610 are strides that a
    multiple of the golden ratio, reduced, meets rarely).  Each wall is one open chain, up or down the plane."""
    W = walls + 5
    i = np.arange(W)
    row = np.where((i % 2 == 1) & (i < walls), 1.5, 0.5).astype(np.float32)
    lat, _ = small_kuhn()
    b = bin_lattice(lat, synth.Grid(0.0, 0.0, 1.0, 1.0, W, H, 0.0, 1.0, 1))
    f = torch.from_numpy(np.broadcast_to(row, (1, H, W)).copy()).cuda()
    segs, off, chain, rank = api.slice_polylines(b, f)
    assert off.cpu().tolist() == [0, walls * (H - 1)]
    segs = segs.cpu().numpy().reshape(H - 1, walls, 4)
    up = segs[..., 3] > segs[..., 1]
    assert np.array_equal(up, np.broadcast_to(up[0], up.shape)) and 0 < up[0].sum() < walls
    r, j = np.mgrid[0:H - 1, 0:walls]
    assert np.array_equal(rank.cpu().numpy().reshape(r.shape), np.where(up, r, H - 2 - r))
    assert np.array_equal(chain.cpu().numpy().reshape(r.shape),
                          np.where(up, j, (H - 2) * walls + j))
