"""Solves of few and large phases (small weights on large graphs, wide buckets on skewed ones) are no
slower than on the phase kernels, whichever kernels the default takes for them."""
import time

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


def best_ms(fn, reps=7):
    fn()
    t = []
    for _ in range(reps):
        t0 = time.perf_counter()
        fn()
        t.append(1e3 * (time.perf_counter() - t0))
    return min(t)


W = (1 << 20) - 1
GRAPHS = {"rmat22_unit": lambda: G.rmat(22, 16, 1, 1, 701), "rmat21_w4": lambda: G.rmat(21, 16, 1, 4, 702),
          "er_64m_unit": lambda: G.er(1 << 20, 64, 1, 1, 703), "rmat20": lambda: G.rmat(20, 16, 1, W, 704),
          "rmat16": lambda: G.rmat(16, 16, 1, W, 705), "rmat20_w256": lambda: G.rmat(20, 16, 1, 256, 706),
          "er_dense": lambda: G.er(5000, 120, 1, W, 707), "er_1m": lambda: G.er(1 << 20, 16, 1, W, 708),
          "er_small_unit": lambda: G.er(8000, 128, 1, 1, 709)}


# which kernels have to serve a call, where one side is clearly the faster
FORMS = {"rmat22_unit": dict(static="phases", simple="phases", checkpoint="phases", delta="phases"),
         "er_64m_unit": dict(simple="phases", checkpoint="phases"),
         "rmat20": dict(static="resident", simple="resident", delta="phases"), "rmat20_w256": dict(static="resident"),
         "rmat16": dict(static="resident", simple="resident", checkpoint="resident", delta="phases"),
         "er_1m": dict(static="resident", simple="resident", checkpoint="resident", delta="resident", delta_third="resident"),
         "er_small_unit": dict(static="resident", simple="resident", delta="resident")}


@pytest.mark.parametrize("name", list(GRAPHS))
def test_default_is_no_slower_than_the_phase_kernels(B, name):
    from paper_1903_12085_amd import selector as S
    sel = S.load_trained()
    g = GRAPHS[name]()
    dg = B.DeviceGraph.from_graph(g)
    src, dist = int(G.sources(g, 1, 710)[0]), B.new_dist(g.n)
    w = int(g.w.max())
    ref = O.dijkstra(g, src)[0] if g.m < 2e7 else None
    for what, call in (("static", lambda: B.solve(dg, src, B.STATIC_OR, dist)),
                       ("simple", lambda: B.solve(dg, src, B.SIMPLE_OR, dist)),
                       ("checkpoint", lambda: B.solve_checkpoint(dg, src, sel, dist)),
                       ("delta", lambda: B.delta_step(dg, src, w, dist)),
                       ("delta_third", lambda: B.delta_step(dg, src, max(1, w // 3), dist))):
        dg.set_launch(single=2)
        phases = best_ms(call)
        got = B.to_u64(dist).copy()
        dg.set_launch(single=0)
        ours = best_ms(call)
        print("%s %s: %.3f ms (%s), phase kernels %.3f ms" % (name, what, ours, dg.last_form(), phases), flush=True)
        assert np.array_equal(B.to_u64(dist), got if ref is None else ref)
        assert ours <= 1.1 * phases + 0.02, (name, what, ours, phases)
        assert dg.last_form() == FORMS.get(name, {}).get(what, dg.last_form()), (name, what)
    dg.close()


def test_zero_weights(B):
    """All distances are 0: one phase for the source, one for the rest."""
    g = G.er(3000, 6, 1, 5, 711)
    g = G.Graph(g.n, g.row_ptr, g.col, np.zeros(g.m, np.uint32), "zero")
    dg = B.DeviceGraph.from_graph(g)
    ref = O.dijkstra(g, 0)[0]
    for call in (lambda: B.solve(dg, 0, B.STATIC_OR), lambda: B.solve(dg, 0, B.SIMPLE_OR), lambda: B.delta_step(dg, 0, 3)):
        assert np.array_equal(call().dist_u64(), ref) and dg.last_form() == "resident"
    dg.close()
