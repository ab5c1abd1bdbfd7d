"""Resident solves with the SIMPLE criteria against the CPU oracle: distances bit-exact and phase
counts equal over every combination that holds one, where heads move past settled ends (long rows,
equal weights, vertices without in- or out-edges), on every launch shape."""
import numpy as np
import pytest

import graphgen as G
import oracle as O
from test_gpu_resident import GRAPHS

pytestmark = pytest.mark.gpu

CRITS = {"simple_or": O.IN_SIMPLE | O.OUT_SIMPLE, "in": O.IN_SIMPLE, "out": O.OUT_SIMPLE,
         "in_outstatic": O.IN_SIMPLE | O.OUT_STATIC, "instatic_out": O.IN_STATIC | O.OUT_SIMPLE}


@pytest.fixture(scope="module")
def B():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU visible")
    from paper_1903_12085_amd import binding
    binding.load()
    return binding


@pytest.mark.parametrize("name", list(GRAPHS))
def test_resident_simple_matches_oracle(B, name):
    g = GRAPHS[name]()
    dg = B.DeviceGraph.from_graph(g)
    src = 0 if g.m == 0 else int(G.sources(g, 1, 340)[0])
    for cname, crit in CRITS.items() if g.n < 60000 else [("simple_or", CRITS["simple_or"])]:
        print(name, cname, src, flush=True)
        ref = O.phased(g, src, crit)
        for _ in range(2):  # the second solve finds heads where the first left them
            r = B.solve(dg, src, crit)
            assert np.array_equal(r.dist_u64(), ref.dist), (name, cname)
            assert r.phases == ref.phases, (name, cname, r.phases, ref.phases)
    dg.close()
