"""Calls whose grids hold more threads than a launch counts (2^32): their
kernels take several launches."""
import gc

import numpy as np
import pytest
import torch

from paper_2101_05031_amd import api, synth

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def memory():
    yield
    gc.collect()
    api.cache_trim()
    torch.cuda.empty_cache()


def bins(grid, nodes, R=0.3, dtype=np.float64, **kw):
    """Separate struts (rows of two end points)."""
    nodes = np.asarray(nodes, dtype=dtype).reshape(-1, 3)
    n = len(nodes) // 2
    edges = np.arange(2 * n, dtype=np.int32).reshape(n, 2)
    t = [torch.from_numpy(x).cuda() for x in (nodes, edges, np.full(n, 10.0, dtype))]
    return api.lattice_bin(*t, R, 1.0, grid, **kw)


def batch(b, k0, nk, cap=4096):
    """(segments, offsets) of one slice_batch call."""
    st, total, segs, off = api.slice_batch(b, k0, nk, capacity=cap)
    assert st == 0 and 0 < total <= cap
    return segs[:total], off


def test_emission_of_more_than_2_to_the_26_chunks():
    """slice_batch on 2^25 + 64 planes of 513 x 2 pixels (two chunks of 64
    blocks per plane): upright struts at the first planes, across planes 2^24
    and 2^25 and at the last ones give the segments of short calls there."""
    dz, nk = 0.1, 2 ** 25 + 64
    grid = synth.Grid(0.0, 0.0, 0.1, 0.1, 513, 2, 0.0, dz, nk)
    b = bins(grid, [[[x, 0.1, z], [x + 0.03, 0.1, z + 3.0]] for x in (7.0, 30.0, 51.22)
                    for z in (1.0, 2 ** 24 * dz - 1.5, 2 ** 25 * dz - 1.5, nk * dz - 3.5)],
             tile=8, slab=16)
    assert b.info()["n_groups"] == 1
    segs, off = batch(b, 0, nk)
    print("whole range:", len(segs), "segments", flush=True)
    at = 0
    for k0, n in ((0, 100), (2 ** 24 - 100, 200), (2 ** 25 - 100, 164)):
        s, o = batch(b, k0, n)
        assert int(off[k0]) == at
        assert torch.equal(off[k0:k0 + n + 1] - at, o)
        assert torch.equal(segs[at:at + len(s)], s)
        at += len(s)
    assert at == len(segs)


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
def test_adjoint_of_more_than_2_to_the_26_buckets(dtype):
    """slice_field_backward on 8208 planes of 65536 x 2 pixels in tiles of 8 and
    slabs of one plane, a strut along x per plane: every bucket holds one strut,
    so every launch has work, and a strut's gradient is that of a short call
    about its plane (within the call: a strut whose box the call's range cuts has
    fewer pairs to sum, and so other partial sums)."""
    nk, W = 8208, 65536
    assert nk * (W // 8) > 2 ** 26
    grid = synth.Grid(0.0, 0.0, 0.125, 0.125, W, 2, 0.0, 1.0, nk)
    z = np.arange(nk) + 0.5625
    ends = np.stack([np.stack([np.full(nk, x), np.full(nk, 0.125), z], 1) for x in (0.5, W / 8 - 0.5)], 1)
    b = bins(grid, ends, dtype=dtype, tile=8, slab=1, max_pairs=1 << 28)
    info = b.info()
    assert info["n_groups"] == 1 and info["n_binned"] == nk
    gen = torch.Generator(device="cuda").manual_seed(3)
    G = torch.randn((nk, 2, W), generator=gen, device="cuda",
                    dtype=torch.float32 if dtype == np.float32 else torch.float64)
    gw, gn = api.slice_field_backward(b, 0, nk, G)
    print("whole range:", float(gw.abs().max()), float(gn.abs().max()), flush=True)
    gn = gn.reshape(nk, 6)
    for k0, n in ((0, 40), (4080, 32), (8180, 28)):
        sw, sn = api.slice_field_backward(b, k0, n, G[k0:k0 + n].contiguous())
        inner = slice(k0 + 1, k0 + n - 1)
        assert float(sw[inner].abs().min()) > 0
        assert torch.equal(gw[inner], sw[inner])
        assert torch.equal(gn[inner], sn.reshape(nk, 6)[inner])
    assert float(gw.abs().min()) > 0
