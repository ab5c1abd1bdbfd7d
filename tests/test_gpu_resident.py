"""Resident solves (sssp_solve and sssp_solve_noalloc with static criteria, sssp_delta_step) against
the CPU oracle: distances bit-exact, phase and round counts equal, where the resident kernel's cuts can go wrong: vertex
counts at the edges of its groups, every launch shape its rule picks, rows long enough to be shared
between workgroups, phases that settle more vertices than its lists hold, and weights so large that
values of one phase differ by more than 32 bits."""
import numpy as np
import pytest

import graphgen as G
import oracle as O

pytestmark = pytest.mark.gpu

STATIC = [O.DIJK, O.IN_STATIC, O.OUT_STATIC, O.STATIC_OR, O.DIJK | O.OUT_STATIC]


@pytest.fixture(scope="module")
def B():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU visible")
    from paper_1903_12085_amd import binding
    binding.load()
    return binding


def star_of(leaves, tail):
    """0 -> 1..leaves with equal weights, each leaf with `tail` edges into a ring of later vertices:
    the second phase settles every leaf at once."""
    ring = 1000
    n = 1 + leaves + ring
    leaf = np.arange(1, leaves + 1, dtype=np.int64)
    to = 1 + leaves + (leaf[:, None] * 7 + np.arange(tail) * 131) % ring
    nxt = 1 + leaves + (np.arange(ring) + 1) % ring
    deg = np.concatenate([[leaves], np.full(leaves, tail), np.ones(ring)]).astype(np.uint64)
    rp = np.concatenate([[0], np.cumsum(deg)]).astype(np.uint64)
    col = np.concatenate([leaf, to.ravel(), nxt]).astype(np.uint32)
    w = np.concatenate([np.full(leaves, 5), 1 + (to.ravel() * 37) % 90, np.full(ring, 3)]).astype(np.uint32)
    return G.Graph(n, rp, col, w, "star_of_%d_%d" % (leaves, tail))


GRAPHS = {
    **{"n%d" % n: (lambda n=n: G.random_small(n, 4 * n, 50, 300 + n)) for n in (1, 2, 7, 8, 9, 63, 65, 511, 4097)},
    "no_edges": lambda: G.from_edges(5, []),
    "heavy": lambda: G.random_small(700, 3000, 0xFFFFFFFF, 321),
    "er_small": lambda: G.er(5003, 9, 1, 1000, 301),           # 32 workgroups of 512 on one XCD
    "er_mid": lambda: G.er(40009, 16, 1, 1 << 20, 302),        # 32 of 1024
    "er_128wg": lambda: G.er(150001, 12, 1, 1 << 20, 303),     # 128 of 1024
    "grid": lambda: G.grid(251, 187, 1, 1 << 16, 304),
    "rmat_shared": lambda: G.rmat(14, 16, 1, 1 << 20, 305),    # rows over 128 edges: shared records
    "rmat_128wg": lambda: G.rmat(17, 16, 1, 1 << 20, 306),
    "many_at_once": lambda: G.er(8000, 128, 1, 1, 307),        # wavefront lists overflow
    "star": lambda: star_of(60000, 3),                         # a hub, and shared lists overflow
    "star_long_rows": lambda: star_of(500, 1500),              # many hubs in one phase
}


@pytest.mark.parametrize("name", list(GRAPHS))
def test_resident_matches_oracle(B, name):
    g = GRAPHS[name]()
    dg = B.DeviceGraph.from_graph(g)
    srcs = [0] if g.m == 0 else [0, int(G.sources(g, 1, 330)[0])]
    for crit in STATIC if g.n < 20000 else [O.STATIC_OR, O.IN_STATIC | O.DIJK]:
        for src in srcs:
            print(name, crit, src, flush=True)
            ref = O.phased(g, src, crit)
            for solve in (B.solve, B.solve_noalloc):
                r = solve(dg, src, crit)
                assert np.array_equal(r.dist_u64(), ref.dist), (name, crit, src)
                assert r.phases == ref.phases, (name, crit, src, r.phases, ref.phases)
    dg.close()


@pytest.mark.parametrize("name", list(GRAPHS))
def test_resident_delta_matches_oracle(B, name):
    """Widths from one that makes nearly every edge heavy to one window over all distances."""
    g = GRAPHS[name]()
    dg = B.DeviceGraph.from_graph(g)
    wmax = int(g.w.max()) if g.m else 1
    src = 0 if g.m == 0 else int(G.sources(g, 1, 331)[0])
    for delta in sorted({max(1, wmax // 16), max(1, wmax // 3), wmax, (1 << 64) - 1}):
        print(name, delta, src, flush=True)
        ref = O.delta_step(g, src, [delta])
        r = B.delta_step(dg, src, delta)
        assert np.array_equal(r.dist_u64(), ref.dist), (name, delta)
        assert r.phases == ref.rounds, (name, delta, r.phases, ref.rounds)
    dg.close()


def test_resident_more_than_2_23_vertices(B):
    """The larger groups: a star's distances are its weights and it takes two phases (also one more
    vertex, reached in a third phase)."""
    n = (1 << 23) + 13
    w = 1 + (np.arange(n - 2, dtype=np.uint64) * 2654435761 % 4000)
    rp = np.full(n + 1, n - 2, np.uint64)
    rp[0] = 0
    rp[n - 1:] = n - 1                       # vertex n - 2 -> n - 1
    col = np.concatenate([np.arange(1, n - 1), [n - 1]]).astype(np.uint32)
    wt = np.concatenate([w, [9000]]).astype(np.uint32)
    dg = B.DeviceGraph(n, rp, col, wt)
    r = B.solve(dg, 0, B.STATIC_OR)
    want = np.concatenate([[0], w, [w[-1] + np.uint64(9000)]]).astype(np.uint64)
    assert np.array_equal(r.dist_u64(), want)
    assert r.phases == 3
    r = B.delta_step(dg, 0, 16384)           # one window: three light rounds and a heavy one
    assert np.array_equal(r.dist_u64(), want) and r.phases == 4
    dg.close()


def test_launch_option_single_selects_the_solver(B):
    """0: resident, 1: one workgroup, 2: the phase kernels; values above mean 2. Same answers."""
    g = G.er(3001, 6, 1, 500, 340)
    ref = O.phased(g, 0, O.STATIC_OR)
    dg = B.DeviceGraph.from_graph(g)
    assert dg.launch()["single"] == 0
    for single, kept in ((1, 1), (2, 2), (7, 2), (0, 0)):
        dg.set_launch(single=single)
        assert dg.launch()["single"] == kept
        r = B.solve(dg, 0, B.STATIC_OR)
        assert np.array_equal(r.dist_u64(), ref.dist) and r.phases == ref.phases
        r = B.delta_step(dg, 0, 100)
        assert np.array_equal(r.dist_u64(), ref.dist) and r.phases == O.delta_step(g, 0, [100]).rounds
    dg.close()
