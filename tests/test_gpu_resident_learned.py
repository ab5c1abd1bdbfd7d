"""Learned checkpoint solves whose static stage runs resident (no trace, no settle phases asked for)
against the same solves by the phase kernels (which record settle phases) and the CPU oracle:
distances bit-exact, phases and counts equal, on every launch shape, with networks that never switch,
switch early or switch late, and with rows that are shared between workgroups."""
import numpy as np
import pytest

import graphgen as G
import oracle as O

pytestmark = pytest.mark.gpu

GRAPHS = {
    "n1": lambda: G.random_small(1, 0, 50, 350),
    "short": lambda: G.random_small(40, 160, 50, 351),           # done before the first choice holds
    "er_small": lambda: G.er(5003, 9, 1, 1000, 352),
    "grid": lambda: G.grid(61, 47, 1, 1 << 16, 353),
    "er_mid": lambda: G.er(40009, 16, 1, 1 << 20, 354),
    "rmat_shared": lambda: G.rmat(14, 16, 1, 1 << 20, 355),
    "er_128wg": lambda: G.er(150001, 12, 1, 1 << 20, 356),
    "rmat_128wg": lambda: G.rmat(17, 16, 1, 1 << 20, 357),
    "heavy": lambda: G.random_small(700, 3000, 0xFFFFFFFF, 358),
}


@pytest.fixture(scope="module")
def B():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU visible")
    from paper_1903_12085_amd import binding
    binding.load()
    return binding


def networks(params):
    """Weights by what they choose: random ones, and output biases that force each choice."""
    rng = np.random.default_rng(359)
    w = (rng.standard_normal(params) * 0.3).astype(np.float32)
    yield "random", w
    for c in range(3):
        f = w.copy()
        f[-6 + c] = 100.0
        yield "choice%d" % c, f


@pytest.mark.parametrize("name", list(GRAPHS))
def test_resident_checkpoint_matches(B, name):
    g = GRAPHS[name]()
    dg = B.DeviceGraph.from_graph(g)
    src = 0 if g.m == 0 else int(G.sources(g, 1, 360)[0])
    for net, w in networks(B.SELECTOR_PARAMS):
        print(name, net, src, flush=True)
        sel = B.Selector(w)
        a = B.solve_checkpoint(dg, src, sel)
        b = B.solve_checkpoint(dg, src, sel, phase_of=True)
        assert np.array_equal(a.dist_u64(), b.dist_u64()), (name, net)
        assert a.phases == b.phases, (name, net, a.phases, b.phases)
        for f in ("sum_f", "n_reach", "m_reach", "relax_edges"):
            assert a.stats[f] == b.stats[f], (name, net, f)
        assert a.stats["n_reach"] - 1 <= a.stats["improving"] <= a.stats["relax_edges"], (name, net)
        if g.n < 60000:
            ref = O.phased(g, src, O.STATIC_OR, mlp_w=w, checkpoint=True)
            assert np.array_equal(a.dist_u64(), ref.dist) and a.phases == ref.phases, (name, net)
            assert a.stats["sum_f"] == ref.sum_f and a.stats["relax_edges"] == ref.relax_edges, (name, net)
    dg.close()
