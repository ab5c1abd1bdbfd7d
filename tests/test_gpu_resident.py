"""Resident solves (sssp_solve and sssp_solve_noalloc with static criteria, sssp_delta_step, default
batches) against the CPU oracle: distances bit-exact, phase and round counts equal, where the resident kernel's cuts can go wrong: vertex
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


@pytest.mark.parametrize("crit", [O.STATIC_OR, O.IN_STATIC, O.OUT_STATIC, O.DIJK])
def test_resident_batch_matches_oracle(B, crit):
    """One batch of every graph above and of random graphs at the edges of the team classes, with more
    queries than workgroups (the small ones repeated), and the same batch with a launch shape given."""
    graphs = [f() for name, f in GRAPHS.items() if name not in ("star",)]
    graphs += [G.er(n, 3, 1, 300, 350 + n) for n in (16384, 16385, 32768, 32769)]
    if crit == O.STATIC_OR:
        graphs.append(GRAPHS["star"]())
    handles, sources, refs = [], [], []
    for g in graphs:
        if crit == O.DIJK and g.n > 10000:
            continue
        dg = B.DeviceGraph.from_graph(g)
        for s in [0] if g.m == 0 else [int(x) for x in G.sources(g, 2, 351)]:
            ref = O.phased(g, s, crit)
            for _ in range(60 if g.n <= 65 else 1):
                handles.append(dg)
                sources.append(s)
                refs.append(ref)
    assert len(handles) > 512
    for cfg in (None, dict(block=256)):
        print("batch", crit, len(handles), cfg, flush=True)
        dists, phases = B.solve_batch(handles, sources, crit, cfg=cfg)
        for dg, d, p, ref in zip(handles, dists, phases, refs):
            assert np.array_equal(B.to_u64(d), ref.dist) and p == ref.phases, (dg.n, p, ref.phases, cfg)


def test_resident_batch_team_sizes(B):
    """Few queries get larger teams, up to a whole gang, and a graph beyond a gang's reach the device."""
    graphs = [G.er(3000, 5, 1, 500, 360), G.er(200003, 4, 1, 1 << 20, 361), G.grid(61, 47, 1, 1000, 362),
              G.er(530000, 3, 1, 1 << 20, 363)]
    dgs = [B.DeviceGraph.from_graph(g) for g in graphs]
    refs = [O.phased(g, 1, O.STATIC_OR) for g in graphs]
    for pick in ([0, 2], [1], [0, 1, 2], [3, 0], [0, 1, 2, 3, 0, 2]):
        dists, phases = B.solve_batch([dgs[i] for i in pick], [1] * len(pick), B.STATIC_OR)
        for i, d, p in zip(pick, dists, phases):
            assert np.array_equal(B.to_u64(d), refs[i].dist) and p == refs[i].phases, (pick, i)


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
