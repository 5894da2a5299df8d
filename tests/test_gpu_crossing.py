"""Improved maintenance (cut-link) on graphs whose crossing edges are counted over more than
64 groups of 64 vertices, so that the drawn edge is looked for beyond the first pass, and on a
graph whose held trees take 512 threads: trees, f and weights against the oracle."""
import numpy as np
import pytest

from test_gpu_ism import _compare, kc  # noqa: F401  (the fixture)
from test_gpu_routes import random_graph

pytestmark = pytest.mark.gpu

GRAPHS = {
    "grid-sweep": lambda gen: gen.grid(66, 66),              # 4,356 vertices: 69 groups
    "lean-walk": lambda gen: random_graph(gen, 4500, 6),     # 71 groups, 256 threads, path sums
    "road-sweep": lambda gen: gen.road_like(9000, seed=4),   # more than 100 groups
    "hub-512-threads": lambda gen: random_graph(gen, 33001, 6, hub=2500),
}


def late_deletions(oracle_lib, gen, g, W, want):
    """Edges of resident trees between the last vertices, their removal leaving the graph connected,
    such that a tree's crossing edges without it all start past vertex 4,096."""
    out = []
    for par in W.S.parents:
        for v in range(g.n - 1, g.n - 200, -1):
            p = int(par[v])
            if p < 4200 or (par == v).any():  # v a leaf: its crossing edges are those of its row
                continue
            row = g.indices[g.offsets[v]:g.offsets[v + 1]]
            if len(row) < 2 or row.min() < 4096 or p not in row:
                continue
            h = gen.remove_edges(g, [(v, p)])
            if not gen.is_connected(h):
                continue
            cross, c, _ = oracle_lib.crossing_edges(h.offsets, h.indices, par, v, p)
            assert c == v and min(x for x, _ in cross) >= 4096
            out.append((v, p))
            g = h
            break
        if len(out) == want:
            break
    return out


@pytest.mark.parametrize("name", sorted(GRAPHS))
def test_cut_link_beyond_the_first_groups(kc, oracle_lib, gen, name):  # noqa: F811
    from test_gpu_updates import deletion_batches
    g = GRAPHS[name](gen)
    assert g.n > 4096
    count = 6
    W = oracle_lib.ism_init(g.offsets, g.indices, seed=17, count=count)
    hit = 0
    with kc.Graph.from_graph(g) as G:
        print(name, g.n, G.info["traversal"], flush=True)
        G.set_option(kc.KC_OPT_MAINTENANCE, kc.KC_MAINT_IMPROVED)
        G.samples_init(17, count)
        _compare(G, W, g.two_m, oracle_lib)
        late = late_deletions(oracle_lib, gen, g, W, 3)
        assert len(late) == 3
        for a, b in late:
            g = gen.remove_edges(g, [(a, b)])
            W, k_ref = oracle_lib.ism_delete(W, g.offsets, g.indices, a, b)
            hit += k_ref
            assert G.apply_updates([a], [b]) == k_ref
            _compare(G, W, g.two_m, oracle_lib)
        assert hit >= 1
        # anywhere, three in one call; then insertions (their counts come from the cut trees too)
        batch = deletion_batches(gen, g, [3], seed=5)[0]
        k_ref = 0
        for a, b in batch:
            g = gen.remove_edges(g, [(a, b)])
            W, k = oracle_lib.ism_delete(W, g.offsets, g.indices, a, b)
            k_ref += k
        assert G.apply_updates([a for a, _ in batch], [b for _, b in batch]) == k_ref
        _compare(G, W, g.two_m, oracle_lib)
        for u, v in gen.insertion_batch(g, 2, np.random.default_rng(3)):
            g = gen.add_edges(g, [(u, v)])
            W, k_ref = oracle_lib.ism_insert(W, g.offsets, g.indices, u, v)
            assert G.apply_updates([u], [v], [1]) == k_ref
            _compare(G, W, g.two_m, oracle_lib)
