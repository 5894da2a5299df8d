"""f on shallow reference trees (path sums without a numbering) on trees far from
uniform: the reference tree itself (every tau0 edge in the tree, so every internal
vertex is marked), its reversals, deep depth-first trees (one long climb) and random
ones, bit for bit against the oracle; invalid parent arrays are refused.  Both table
depths (reference trees of depth at most 4, and 5 to 8), sizes around the workgroup's,
and one beyond the 2^19 bits of the map."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def kc():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2511_16356_amd as kc
    kc.library()
    return kc


def random_tree(g, root, rng, depth_first):
    """A spanning tree by a search from the root in random order."""
    par = np.full(g.n, -1, np.int32)
    seen = np.zeros(g.n, bool)
    seen[root] = True
    open_ = [root]
    while open_:
        k = len(open_) - 1 if depth_first else int(rng.integers(len(open_)))
        x = open_[k]
        row = g.indices[g.offsets[x]:g.offsets[x + 1]]
        row = row[~seen[row]]
        if row.size == 0:
            open_[k] = open_[-1]
            open_.pop()
            continue
        y = int(rng.choice(row))
        seen[y] = True
        par[y] = x
        open_.append(y)
    return par


CASES = [("complete", 40), ("complete", 513), ("star", 300), ("social", 1500), ("social", 6000), ("dense", 4000),
         ("ba", 900), ("tree8", 121)]


def graph(gen, name, n):
    if name == "tree8":  # a ternary tree with a few extra edges: a reference tree deeper than 4
        v = np.arange(1, n)
        rng = np.random.default_rng(3)
        eu = np.concatenate([v, rng.integers(n // 2, n, 6)])
        ev = np.concatenate([(v - 1) // 3, rng.integers(n // 2, n, 6)])
        return gen.from_edges("tree8", n, eu[eu != ev], ev[eu != ev])
    return {"complete": lambda: gen.complete(n), "star": lambda: gen.star(n),
            "social": lambda: gen.chung_lu(n, 2.2, 10.0, 5 * n ** 0.5, seed=4),
            "dense": lambda: gen.chung_lu(n, 2.0, 76.0, 17 * n ** 0.5, seed=4),
            "ba": lambda: gen.barabasi_albert(n, 4, 2)}[name]()


@pytest.mark.parametrize("name,n", CASES)
def test_trees_of_every_shape(kc, oracle_lib, gen, name, n):
    import torch
    g = graph(gen, name, n)
    print("paths", name, g.n, flush=True)
    P = oracle_lib.prepare_graph(g)
    rng = np.random.default_rng(n)
    trees = [np.array(P.p0, np.int32)] + [random_tree(g, P.root, rng, k % 2 == 0) for k in range(4)]
    trees += list(oracle_lib.sample(P, seed=2, s0=0, count=3, threads=4)[0])
    trees = np.stack(trees)
    trees[:, P.root] = -1
    ref = np.array([oracle_lib.f_of_tree(P, t) for t in trees], np.int64)
    with kc.Graph.from_graph(g) as G:
        assert G.info["depth0"] <= 8
        G.set_option(kc.KC_OPT_TRAVERSAL, kc.KC_TRAV_WALK)
        dev = torch.from_numpy(trees).cuda()
        assert np.array_equal(G.evaluate_trees(dev).cpu().numpy(), ref)
        G.set_option(kc.KC_OPT_SLOTS, 1)
        assert np.array_equal(G.evaluate_trees(dev).cpu().numpy(), ref)
        bad = dev.clone()  # a cycle away from the root
        a, b = [v for v in range(g.n) if v != P.root][:2]
        bad[1, a], bad[1, b] = b, a
        for t in (bad, torch.cat([dev[:1], bad[1:2]])):
            with pytest.raises(kc.KcError) as e:
                G.evaluate_trees(t)
            assert e.value.status == 1
        assert np.array_equal(G.evaluate_trees(dev).cpu().numpy(), ref)  # usable afterwards


def test_more_vertices_than_map_bits(kc, oracle_lib, gen):
    import torch
    g = gen.chung_lu(620000, 2.2, 10.0, 3000.0, seed=5)
    assert g.n > 1 << 19
    print("paths", g.n, flush=True)
    P = oracle_lib.prepare_graph(g)
    par, _, _ = oracle_lib.sample(P, seed=8, s0=3, count=2, threads=2)
    trees = np.concatenate([par, np.array(P.p0, np.int32)[None]])
    ref = np.array([oracle_lib.f_of_tree(P, t) for t in trees], np.int64)
    with kc.Graph.from_graph(g) as G:
        assert G.info["depth0"] <= 8
        assert np.array_equal(G.evaluate_trees(torch.from_numpy(trees).cuda()).cpu().numpy(), ref)
        est, f, _ = G.estimate(8, 3, 2, per_sample=True)
        assert np.array_equal(f.cpu().numpy(), ref[:2])
