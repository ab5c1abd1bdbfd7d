"""Dynamic criteria at the edges of the term and dirty-set passes' windows (256 vertices up to 2^18
vertices, 1024 above) against the CPU oracle: every observable of solve_ex."""
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


@pytest.mark.parametrize("crit", [O.SIMPLE_OR, O.FULL_OR, O.CRIT["IN_SIMPLE"] | O.OUT_STATIC,
                                  O.IN_STATIC | O.CRIT["OUT_WEAK"]])
@pytest.mark.parametrize("n", [1, 255, 257, 1 << 18, (1 << 18) + 1, (1 << 18) + 1027])
def test_windows_match_oracle(B, n, crit):
    g = G.random_small(n, 4 * n, 60, 400 + n) if n < 1000 else G.er(n, 3, 1, 400, 401)
    ref = O.phased(g, 0, crit)
    dg = B.DeviceGraph.from_graph(g)
    r = B.solve_ex(dg, 0, crit, phase_of=True, trace_cap=ref.phases + 4)
    assert np.array_equal(r.dist_u64(), ref.dist)
    assert r.phases == ref.phases and r.stats["sum_f"] == ref.sum_f
    assert np.array_equal(r.phase_of.cpu().numpy().view(np.uint32), ref.phase_of)
    assert np.array_equal(r.trace["settled"], ref.trace_s) and np.array_equal(r.trace["min_d"], ref.trace_mind)
    assert np.array_equal(B.solve(dg, 0, crit).dist_u64(), ref.dist)
    dg.close()
