"""Teams of the default batch that solve several queries one after the other, against the oracle."""
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


def hub(n, leaves, seed):
    """0 -> 1..leaves, each leaf -> one vertex of a short ring: shared records in the first phase."""
    rng = np.random.default_rng(seed)
    e = [(0, 1 + i, int(w)) for i, w in enumerate(rng.integers(1, 1000, leaves))]
    e += [(1 + i, 1 + leaves + i % 50, int(w)) for i, w in enumerate(rng.integers(1, 1000, leaves))]
    return G.from_edges(n, e + [(1 + leaves + i, 1 + leaves + (i + 1) % 50, 7) for i in range(50)])


def path(n, length):
    return G.from_edges(n, [(i, i + 1, 3) for i in range(length - 1)])


def run(B, groups):
    """groups: (graph, how many queries from vertex 0), in the order in which the teams take them."""
    queries = [g for g, count in groups for _ in range(count)]
    refs = {id(g): O.phased(g, 0, O.STATIC_OR) for g, _ in groups}
    handles = {id(g): B.DeviceGraph.from_graph(g) for g, _ in groups}
    dists, phases = B.solve_batch([handles[id(g)] for g in queries], [0] * len(queries), B.STATIC_OR)
    for i, (g, d, p) in enumerate(zip(queries, dists, phases)):
        ref = refs[id(g)]
        assert np.array_equal(B.to_u64(d), ref.dist) and p == ref.phases, (i, g.n, p, ref.phases)
    for h in handles.values():
        h.close()


@pytest.mark.parametrize("length", [25, 26, 27, 55])
def test_team_shares_records_again_after_a_query_without(B, length):
    """Teams of two workgroups (256 of them, the costlier graphs first): a query with shared records, one
    without of a given number of phases, one with. Counts left by the first must not serve the third."""
    first, middle, last = hub(32000, 3000, 1), path(24000, length), hub(17000, 2000, 2)
    assert O.phased(middle, 0, O.STATIC_OR).phases == length
    run(B, [(first, 260), (middle, 260), (last, 260)])
