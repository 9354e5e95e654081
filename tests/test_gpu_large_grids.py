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


def bins(grid, nodes, R=0.3, **kw):
    """Separate struts (rows of two end points), float64."""
    nodes = np.asarray(nodes, dtype=np.float64).reshape(-1, 3)
    n = len(nodes) // 2
    edges = np.arange(2 * n, dtype=np.int32).reshape(n, 2)
    t = [torch.from_numpy(x).cuda() for x in (nodes, edges, np.full(n, 10.0))]
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
