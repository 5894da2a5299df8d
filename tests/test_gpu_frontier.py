"""The frontier sampler and the workgroup-wide evaluation at the sizes where they can
go wrong, bit for bit against the CPU oracle (exact integers: no tolerance).

  - fewer vertices than threads, exact multiples of them and one off;
  - the last size whose words fit the LDS fields (32,767 vertices) and the next, which
    takes another route;
  - long walks and single large cycles (paths, cycles), hubs (stars), rows beyond the
    inline neighbours (complete and power-law graphs);
  - a preorder step of the sweep in which more tau0 subtrees close than a workgroup has
    threads (paths and cycles: all of them in the last step).
"""
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


def graph(gen, name):
    kind, size = name.rsplit("-", 1)
    n = int(size)
    if kind == "grid":
        rows = next(r for r in range(int(n ** 0.5), 0, -1) if n % r == 0)
        return gen.grid(rows, n // rows)
    if kind == "lean":  # mean degree 10 on a ring, so that it is connected with exactly n vertices
        rng = np.random.default_rng(n)
        u = np.concatenate([np.arange(n), rng.integers(0, n, 4 * n)])
        v = np.concatenate([(np.arange(n) + 1) % n, rng.integers(0, n, 4 * n)])
        return gen.from_edges(name, n, u[u != v], v[u != v])
    if kind == "power":
        return gen.chung_lu(n, 2.2, 10.0, 5 * n ** 0.5, seed=1)
    return {"path": gen.path, "cycle": gen.cycle, "star": gen.star, "complete": gen.complete}[kind](n)


@pytest.mark.parametrize("name,count", [
    ("path-2", 5), ("path-63", 6), ("path-700", 2), ("cycle-65", 6), ("cycle-1100", 2), ("star-255", 6),
    ("star-40000", 3), ("complete-257", 6), ("grid-256", 12), ("grid-1024", 40), ("grid-1025", 8),
    ("lean-512", 9), ("lean-32766", 3), ("lean-32767", 3), ("lean-32768", 3), ("grid-32767", 1),
    ("grid-32768", 1), ("power-40000", 5)])
def test_samples_and_values(kc, oracle_lib, gen, name, count):
    import torch
    g = graph(gen, name)
    print("frontier", name, g.n, flush=True)
    P = oracle_lib.prepare_graph(g)
    par, cnt, steps = oracle_lib.sample(P, seed=19, s0=70, count=count, threads=8)
    f, _ = oracle_lib.estimate_f(P, seed=19, s0=70, count=count, threads=8)
    with kc.Graph.from_graph(g) as G:
        got = G.sample_trees(19, 70, count)
        assert np.array_equal(got[0].cpu().numpy(), par)
        assert np.array_equal(got[1].cpu().numpy().astype(np.uint32), cnt)
        assert np.array_equal(got[2].cpu().numpy(), steps)
        _, gf, gs = G.estimate(19, 70, count, per_sample=True)
        assert np.array_equal(gf.cpu().numpy(), f) and np.array_equal(gs.cpu().numpy(), steps)
        G.set_option(kc.KC_OPT_SLOTS, 2)  # each slot's state returns to its start
        for trav in (kc.KC_TRAV_SWEEP, kc.KC_TRAV_WALK):
            G.set_option(kc.KC_OPT_TRAVERSAL, trav)
            if trav == kc.KC_TRAV_WALK and G.info["depth0"] > 400:
                continue
            ev = G.evaluate_trees(torch.from_numpy(par).cuda())
            assert np.array_equal(ev.cpu().numpy(), f), trav


def test_mixed_batch(kc, oracle_lib, gen):
    """One launch over graphs of every route the frontier sampler has, replayed."""
    gs = [graph(gen, x) for x in ("grid-1024", "lean-33000", "power-3000")]
    counts = [9, 3, 7]
    with kc.Graph.from_graph(gs[0]) as A, kc.Graph.from_graph(gs[1]) as B, kc.Graph.from_graph(gs[2]) as C:
        with kc.Batch([A, B, C], [4, 5, 6], [0, 10, 20], counts) as batch:
            for launch in range(3):
                batch.launch()
                ests, done = batch.results()
                assert done == launch + 1
                for j, (g, first) in enumerate(zip(gs, (0, 10, 20))):
                    P = oracle_lib.prepare_graph(g)
                    f, _ = oracle_lib.estimate_f(P, seed=4 + j, s0=first + launch * counts[j], count=counts[j], threads=8)
                    assert np.array_equal(batch.f(j).cpu().numpy(), f)
                    K, se, s1, _ = oracle_lib.reduce_estimate(f, g.two_m)
                    assert ests[j].kappa == K and ests[j].sum_f == s1
