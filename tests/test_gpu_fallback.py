"""Resident solves that give up: with a wait limit of one poll hardly a workgroup sees the others arrive,
all leave, and the kernels without such waits serve the call with the oracle's distances and phase
counts. With the default limit the resident solve serves it."""
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


GRAPHS = {"one_xcd": lambda: G.er(5003, 9, 1, 1000, 601), "shared_rows": lambda: G.rmat(14, 16, 1, 1 << 20, 602),
          "128_workgroups": lambda: G.er(150001, 12, 1, 1 << 20, 603)}


def calls(B, crits):
    from paper_1903_12085_amd import selector as S
    yield "noalloc", lambda g, s: B.solve_noalloc(g, s, B.STATIC_OR), lambda g, s: O.phased(g, s, O.STATIC_OR), "phases"
    yield "delta", lambda g, s: B.delta_step(g, s, 300), lambda g, s: O.delta_step(g, s, [300]), "phases"
    for c in crits:
        yield c, lambda g, s, c=c: B.solve(g, s, c), lambda g, s, c=c: O.phased(g, s, c), "phases"
    sel = S.load_trained()
    yield "learned", lambda g, s: B.solve_checkpoint(g, s, sel), lambda g, s: O.dijkstra(g, s)[0], "phases"


@pytest.mark.parametrize("name", list(GRAPHS))
def test_solves_that_give_up_are_served_by_the_phase_kernels(B, name):
    g = GRAPHS[name]()
    dg = B.DeviceGraph.from_graph(g)
    src = int(G.sources(g, 1, 604)[0])
    for what, call, oracle, other in calls(B, [B.STATIC_OR, B.IN_SIMPLE | B.OUT_STATIC] if g.n > 20000 else
                                           [B.STATIC_OR, B.IN_STATIC, B.OUT_STATIC, B.SIMPLE_OR]):
        ref = oracle(g, src)
        for polls, form in ((1, other), (0, "resident")):
            print(name, what, polls, flush=True)
            dg.set_wait_limit(polls)
            r = call(dg, src)
            assert dg.last_form() == form, (name, what, polls, dg.last_form())
            if what == "learned":
                assert np.array_equal(r.dist_u64(), ref)
            else:
                assert np.array_equal(r.dist_u64(), ref.dist)
                assert r.phases == (ref.rounds if what == "delta" else ref.phases)
    dg.close()


def test_batches_that_give_up_are_served_by_the_one_launch(B):
    graphs = [G.er(40009, 8, 1, 1 << 20, 610), G.rmat(15, 16, 1, 1 << 20, 611), G.er(530003, 3, 1, 1 << 20, 612)]
    dgs = [B.DeviceGraph.from_graph(g) for g in graphs]
    refs = [O.phased(g, 1, O.STATIC_OR) for g in graphs]
    for pick in ([0, 1], [0], [1, 2, 0]):
        for polls, form in ((1, "workgroups"), (0, "resident")):
            for dg in dgs:
                dg.set_wait_limit(polls)
            dists, phases = B.solve_batch([dgs[i] for i in pick], [1] * len(pick), B.STATIC_OR)
            assert dgs[pick[0]].last_form() == form, (pick, polls)
            for i, d, p in zip(pick, dists, phases):
                assert np.array_equal(B.to_u64(d), refs[i].dist) and p == refs[i].phases, (pick, polls, i)
    for dg in dgs:
        dg.close()


def test_forms_by_launch_option(B):
    g = G.er(3001, 6, 1, 500, 613)
    dg = B.DeviceGraph.from_graph(g)
    assert dg.last_form() == "none"
    for single, form in ((0, "resident"), (1, "workgroups"), (2, "phases")):
        dg.set_launch(single=single)
        B.solve(dg, 0, B.STATIC_OR)
        assert dg.last_form() == form
    B.solve_ex(dg, 0, B.STATIC_OR)
    assert dg.last_form() == "phases"
    B.solve_batch([dg, dg], [0, 1], B.STATIC_OR, cfg=dict(block=256))
    assert dg.last_form() == "workgroups"
    dg.close()
