"""Graph creation from device and host arrays, and the block that graph destruction keeps: graphs made
in memory that an earlier, different graph has used solve as on their own."""
import numpy as np
import pytest

import graphgen as G
import oracle as O

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU visible")
    from paper_1903_12085_amd import binding
    binding.load()
    return binding


def minima(g):
    """minIn, minOut by numpy (UINT32_MAX without an edge)."""
    mi, mo = np.full(g.n, 0xFFFFFFFF, np.uint32), np.full(g.n, 0xFFFFFFFF, np.uint32)
    np.minimum.at(mi, g.col, g.w)
    np.minimum.at(mo, np.repeat(np.arange(g.n), g.outdeg()), g.w)
    return mi, mo


def check(B, dg, g):
    for got, want in zip(dg.minima(), minima(g)):
        assert np.array_equal(got.cpu().numpy().view(np.uint32), want)
    ref, _ = O.dijkstra(g, 0)
    assert np.array_equal(B.solve(dg, 0, B.STATIC_OR).dist_u64(), ref)


@pytest.mark.parametrize("device", [False, True])
def test_creation_in_kept_blocks(B, device):
    import torch
    # about 80, 70 and 140 MB of device arrays (a kept block serves requests down to half its size),
    # small ones between them
    for i, (n, k) in enumerate([(400000, 16), (350003, 16), (5, 2), (700001, 16), (63, 3), (390000, 16)]):
        g = G.er(n, k, 1, 1000 + i, 500 + i)
        if device:
            up = lambda a, t: torch.from_numpy(a.view(t)).cuda()
            dg = B.DeviceGraph(g.n, up(g.row_ptr, np.int64), up(g.col, np.int32), up(g.w, np.int32), device_ptrs=True)
        else:
            dg = B.DeviceGraph.from_graph(g)
        check(B, dg, g)
        dg.close()
    assert B.load().sssp_graph_destroy(None) == 0  # gives the kept block back
    g = G.er(400000, 16, 1, 77, 510)
    dg = B.DeviceGraph.from_graph(g)
    check(B, dg, g)
    dg.close()


@pytest.mark.parametrize("what", ["target", "rows", "first", "last"])
def test_malformed_device_arrays_are_rejected(B, what):
    """Checked on the device before any kernel follows a row or a target; the library stays usable."""
    import torch
    g = G.er(3000, 5, 1, 100, 520)
    rp, col = g.row_ptr.astype(np.int64), g.col.astype(np.int64)
    if what == "target":
        col[1234] = g.n
    elif what == "rows":
        rp[700] = rp[702] + 3
    elif what == "first":
        rp[0] = 1
    else:
        rp[-1] = g.m - 1
    up = lambda a, t: torch.from_numpy(a.astype(t)).cuda()
    with pytest.raises(B.SsspError) as e:
        B.DeviceGraph(g.n, up(rp, np.int64), up(col, np.int32), up(g.w, np.int32), device_ptrs=True)
    assert e.value.code == -1 and "malformed" in str(e.value)
    dg = B.DeviceGraph.from_graph(g)
    check(B, dg, g)
    dg.close()


def test_minima_of_long_and_empty_rows(B):
    """Rows longer than a wavefront's window, empty rows, the largest weight, parallel edges."""
    rng = np.random.default_rng(5)
    deg = np.where(rng.random(4100) < 0.3, 0, rng.integers(0, 9, 4100))
    deg[[0, 1999, 4099]] = [5000, 700, 130]
    m = int(deg.sum())
    rp = np.concatenate([[0], np.cumsum(deg)]).astype(np.uint64)
    w = rng.integers(1, 1 << 32, m, dtype=np.uint64).astype(np.uint32)
    w[::50] = 0xFFFFFFFF
    g = G.Graph(4100, rp, rng.integers(0, 2000, m).astype(np.uint32), w, "uneven")
    dg = B.DeviceGraph.from_graph(g)
    check(B, dg, g)
    dg.close()
