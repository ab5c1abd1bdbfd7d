"""Dynamic criteria above 2^21 vertices, where the term and dirty-set passes of the criteria with stored
terms take windows of 4096 vertices (the SIMPLE ones above 2^22), at the edges of a window and of a thread's sixteen bytes, against the CPU oracle."""
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


@pytest.mark.parametrize("n", [(1 << 21) + 1, (1 << 21) + 4096 + 11, (1 << 22) + 13])
def test_large_windows_match_oracle(B, n):
    g = G.er(n, 2, 1, 40, 402)
    dg = B.DeviceGraph.from_graph(g)
    for crit in (O.SIMPLE_OR, O.FULL_OR, O.IN_STATIC | O.CRIT["OUT_WEAK"]):
        print(n, crit, flush=True)
        ref = O.phased(g, 0, crit)
        r = B.solve_ex(dg, 0, crit, phase_of=True, trace_cap=ref.phases + 4)
        assert np.array_equal(r.dist_u64(), ref.dist)
        assert r.phases == ref.phases and r.stats["sum_f"] == ref.sum_f
        assert np.array_equal(r.phase_of.cpu().numpy().view(np.uint32), ref.phase_of)
        assert np.array_equal(r.trace["settled"], ref.trace_s) and np.array_equal(r.trace["min_d"], ref.trace_mind)
    dg.close()


def test_large_sparse_graphs_keep_their_speed(B):
    """IN|OUT on 2^23 random vertices of degree 2: 30.6 ms with windows of 4096, 37.9 with 1024."""
    import time
    g = G.er(1 << 23, 2, 1, (1 << 20) - 1, 7)
    dg, t = B.DeviceGraph.from_graph(g), []
    src, dist = int(G.sources(g, 1, 5)[0]), B.new_dist(g.n)
    for _ in range(4):
        t0 = time.perf_counter()
        B.solve(dg, src, B.FULL_OR, dist)
        t.append(1e3 * (time.perf_counter() - t0))
    print(["%.1f" % x for x in t])
    assert min(t[1:]) < 35
    dg.close()


def test_windows_by_stored_terms_and_switches(B):
    """SIMPLE criteria keep windows of 1024 up to 2^22 vertices and full ones take 4096: a solve that
    switches from one kind to the other, and both on one handle with phases replayed from a graph."""
    n = (1 << 21) + 5000
    g = G.er(n, 3, 1, 30, 403)
    dg = B.DeviceGraph.from_graph(g)
    ref = O.dijkstra(g, 0)[0]
    for use_graph in (0, 1):
        dg.set_launch(use_graph=use_graph, single=2)
        for crit in (B.SIMPLE_OR, B.FULL_OR, B.IN_SIMPLE | B.OUT_STATIC, B.SIMPLE_OR):
            assert np.array_equal(B.solve(dg, 0, crit).dist_u64(), ref), (use_graph, crit)
        for then in (B.FULL_OR, B.SIMPLE_OR):
            assert np.array_equal(B.solve_switch(dg, 0, B.STATIC_OR, then, (1, 2)).dist_u64(), ref), (use_graph, then)
    dg.close()
