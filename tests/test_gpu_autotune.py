"""The autotuner and the choice between the resident solve and the phase kernels (`single`): a criterion
that runs resident gets whichever is faster, one that never does leaves the choice alone."""
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


@pytest.mark.parametrize("crit", ["STATIC_OR", "SIMPLE_OR", "IN_SIMPLE|OUT_STATIC"])
def test_resident_criteria_keep_the_resident_solve(B, crit):
    """On a small random graph the resident solve takes less than half as long with each of these."""
    crit = B.IN_SIMPLE | B.OUT_STATIC if "|" in crit else getattr(B, crit)
    g = G.er(5003, 9, 1, 1000, 401)
    dg = B.DeviceGraph.from_graph(g)
    cfg, _ = B.autotune(dg, 0, crit)
    assert cfg["single"] == 0 and dg.launch()["single"] == 0
    r, ref = B.solve(dg, 0, crit), O.phased(g, 0, crit)
    assert np.array_equal(r.dist_u64(), ref.dist) and r.phases == ref.phases
    dg.close()


def test_default_that_takes_the_phase_kernels_is_kept(B):
    """Unit weights on a large skewed graph: static solves run the phase kernels by default, others on the
    handle still run resident."""
    dg = B.DeviceGraph.from_graph(G.rmat(21, 16, 1, 1, 403))
    cfg, _ = B.autotune(dg, 1, B.STATIC_OR)
    B.solve(dg, 1, B.STATIC_OR)
    assert dg.last_form() == "phases" and cfg["single"] in (0, 1) and dg.launch()["single"] == cfg["single"]
    dg.close()


@pytest.mark.parametrize("single", [0, 1, 2])
def test_other_criteria_leave_the_choice_alone(B, single):
    g = G.er(2001, 6, 1, 1000, 402)
    dg = B.DeviceGraph.from_graph(g)
    dg.set_launch(single=single)
    cfg, _ = B.autotune(dg, 0, B.FULL_OR)
    assert cfg["single"] == single and dg.launch()["single"] == single
    r, ref = B.solve(dg, 0, B.FULL_OR), O.phased(g, 0, B.FULL_OR)
    assert np.array_equal(r.dist_u64(), ref.dist) and r.phases == ref.phases
    dg.close()
