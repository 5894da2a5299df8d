"""Every way a graph's trees are sampled, bit for bit against the CPU oracle (exact
integers: no tolerance), on graphs the dispatch sends there.

The rounds a call reports (sampler_iterations) tell the samplers apart: with one walker
the chain sampler takes many times the rounds, the frontier sampler as many as before.
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


def random_graph(gen, n, deg, hub=0, seed=1):
    """Mean degree deg on a ring; with hub, vertex 0 is joined to that many others."""
    rng = np.random.default_rng(seed)
    k = n * (deg - 2) // 2
    u = np.concatenate([np.arange(n), rng.integers(0, n, k), np.zeros(hub, np.int64)])
    v = np.concatenate([(np.arange(n) + 1) % n, rng.integers(0, n, k), np.arange(1, 1 + hub)])
    return gen.from_edges("random", n, u[u != v], v[u != v])


def samples_match(G, oracle_lib, P, seed, first, count):
    par, cnt, steps = oracle_lib.sample(P, seed=seed, s0=first, count=count, threads=8)
    got = G.sample_trees(seed, first, count)
    assert np.array_equal(got[0].cpu().numpy(), par)
    assert np.array_equal(got[1].cpu().numpy().astype(np.uint32), cnt)
    assert np.array_equal(got[2].cpu().numpy(), steps)
    f, _ = oracle_lib.estimate_f(P, seed=seed, s0=first, count=count, threads=8)
    est, gf, gs = G.estimate(seed, first, count, per_sample=True)
    assert np.array_equal(gf.cpu().numpy(), f) and np.array_equal(gs.cpu().numpy(), steps)
    return est


def on_chains(kc, G, seed, first, count):
    rounds = []
    for walkers in (64, 1):
        G.set_option(kc.KC_OPT_WALKERS, walkers)
        rounds.append(G.estimate(seed, first, count).sampler_iterations)
    G.set_option(kc.KC_OPT_WALKERS, 64)
    return rounds[1] > 4 * rounds[0]


def test_large_lean_graph_with_a_deep_reference_tree(kc, oracle_lib, gen):
    """The frontier sampler with its words in memory, tau0 breadth-first (path sums) and
    depth-first (the sweep, a workgroup of that sampler's threads)."""
    g = random_graph(gen, 33001, 10, hub=2500)
    P = oracle_lib.prepare_graph(g)
    with kc.Graph.from_graph(g) as G:
        samples_match(G, oracle_lib, P, 21, 5, 4)
        G.set_tau0(kc.KC_TAU0_DFS)
        assert G.info["depth0"] > 1000 and G.info["traversal"] == kc.KC_TRAV_SWEEP
        Q = oracle_lib.with_tau0(P, oracle_lib.dfs_tree(g.offsets, g.indices, P.root))
        samples_match(G, oracle_lib, Q, 21, 5, 4)
        assert not on_chains(kc, G, 21, 5, 4)


def test_batch_of_words_in_lds_and_in_memory(kc, oracle_lib, gen):
    gs = [gen.grid(32, 32), random_graph(gen, 33000, 10, hub=2500), gen.chung_lu(3000, 2.2, 10.0, 270.0, seed=1)]
    counts = [9, 3, 7]
    Gs = [kc.Graph.from_graph(g) for g in gs]
    with kc.Batch(Gs, [4, 5, 6], [0, 10, 20], counts) as batch:
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
    for G in Gs:
        G.close()


def test_many_samples_on_the_chains_equal_few_in_lds(kc, gen):
    """A grid that leaves one workgroup per CU: above 1,792 samples a call takes the chains, its
    parts do not; a workspace without slots for the chains keeps LDS.  The sums and each f agree."""
    count = 2000
    with kc.Graph.from_graph(gen.grid(135, 135)) as G:
        whole, f, steps = G.estimate(17, 900, count, per_sample=True)
        assert on_chains(kc, G, 17, 900, 1793) and not on_chains(kc, G, 17, 900, 8)
        parts = [G.estimate(17, 900 + a, 500, per_sample=True) for a in range(0, count, 500)]
        for i, (_, pf, ps) in enumerate(parts):
            assert (pf == f[500 * i:500 * i + 500]).all() and (ps == steps[500 * i:500 * i + 500]).all()
        pooled = G.combine([p[0] for p in parts])
        assert (pooled.sum_f, pooled.sum_f2, pooled.total_steps) == (whole.sum_f, whole.sum_f2, whole.total_steps)
        par, cnt, _ = G.sample_trees(17, 900, 1800)
        few, fewcnt, _ = G.sample_trees(17, 1400, 40)
        assert (par[500:540] == few).all() and (cnt[500:540] == fewcnt).all()
        with kc.Batch([G], [17], [900], [count]) as batch:
            for launch in range(2):
                batch.launch()
                est, _ = batch.results()
                if launch == 0:
                    assert est[0].sum_f == whole.sum_f and (batch.f(0) == f).all()
        G.set_option(kc.KC_OPT_SLOTS, 300)
        assert not on_chains(kc, G, 17, 900, 1793)
        assert G.estimate(17, 900, count).sum_f == whole.sum_f


def test_captured_batch_with_more_than_64_kb_of_words(kc, oracle_lib, gen):
    gs = [gen.grid(150, 200), gen.grid(12, 12)]
    Gs = [kc.Graph.from_graph(g) for g in gs]
    with kc.Batch(Gs, [8, 9], [3, 1000], [2, 30]) as batch:
        for launch in range(2):
            batch.launch()
            batch.results()
            for j, (g, first, c) in enumerate(zip(gs, (3, 1000), (2, 30))):
                P = oracle_lib.prepare_graph(g)
                f, _ = oracle_lib.estimate_f(P, seed=8 + j, s0=first + launch * c, count=c, threads=8)
                assert np.array_equal(batch.f(j).cpu().numpy(), f)
    for G in Gs:
        G.close()


@pytest.mark.parametrize("kind,size,count", [
    ("path", 2, 1100), ("path", 63, 5000), ("path", 65, 1025), ("cycle", 65, 9000), ("star", 255, 5000), ("star", 512, 1025),
    ("star", 513, 1025), ("complete", 129, 1500), ("grid", (32, 32), 5000), ("grid", (64, 64), 1025), ("grid", (17, 241), 1025),
    ("cycle", 4096, 1025)])
def test_many_small_trees(kc, oracle_lib, gen, kind, size, count):
    """Evaluations in more than 1,024 slots: one wavefront per tree up to 4,096 vertices (sweep) or
    512 (path sums), each with a fixed share of the trees; then a call with a parent array that is
    no tree, and the trees again."""
    import torch
    g = gen.grid(*size) if kind == "grid" else {"path": gen.path, "cycle": gen.cycle, "star": gen.star,
                                                 "complete": gen.complete}[kind](size)
    P = oracle_lib.prepare_graph(g)
    rng = np.random.default_rng(g.n)
    if kind == "cycle":  # a tree is a path: cut at a random edge
        trees = []
        for cut in rng.integers(0, g.n, 7):
            par = np.full(g.n, -1, np.int32)
            for step in (1, -1):
                v = P.root
                while (v if step == 1 else (v - 1) % g.n) != cut:
                    par[(v + step) % g.n] = v
                    v = (v + step) % g.n
            trees.append(par)
        trees = np.array(trees, np.int32)
    else:
        trees = oracle_lib.sample(P, seed=2, s0=0, count=7, threads=8)[0]
    ref = np.array([oracle_lib.f_of_tree(P, t) for t in trees], np.int64)
    pick = rng.integers(0, len(trees), count)
    par = torch.from_numpy(trees[pick]).cuda()
    with kc.Graph.from_graph(g) as G:
        if g.n <= 600:
            G.set_option(kc.KC_OPT_TRAVERSAL, kc.KC_TRAV_SWEEP)
            assert np.array_equal(G.evaluate_trees(par).cpu().numpy(), ref[pick])
            G.set_option(kc.KC_OPT_TRAVERSAL, kc.KC_TRAV_AUTO)
        assert np.array_equal(G.evaluate_trees(par).cpu().numpy(), ref[pick])
        bad = par.clone()
        bad[count // 2, (P.root + 1) % g.n] = (P.root + 1) % g.n
        with pytest.raises(kc.KcError) as ei:
            G.evaluate_trees(bad)
        assert ei.value.status == 1
        assert np.array_equal(G.evaluate_trees(par).cpu().numpy(), ref[pick])
        G.set_option(kc.KC_OPT_SLOTS, 3)
        assert np.array_equal(G.evaluate_trees(par[:40]).cpu().numpy(), ref[pick[:40]])


CHAIN_GRAPHS = {
    "random": lambda gen: random_graph(gen, 33001, 8),     # lean looks by default
    "grid": lambda gen: gen.grid(182, 182),                # long walks, no lean looks
}


@pytest.fixture(scope="module")
def chain_reference(oracle_lib, gen):
    ref = {}
    for name, make in CHAIN_GRAPHS.items():
        g = make(gen)
        P = oracle_lib.prepare_graph(g)
        first = (1 << 40) + 3 if name == "random" else 12
        trees = oracle_lib.sample(P, seed=23, s0=first, count=4, threads=8)
        ref[name] = (g, first, trees, oracle_lib.estimate_f(P, seed=23, s0=first, count=4, threads=8)[0])
    return ref


@pytest.mark.parametrize("options", [
    {"WALKERS": 1}, {"WALKERS": 7, "SLOTS": 3}, {"WALKERS": 63, "SLOTS": 1}, {"START_ORDER": 0}, {"START_ORDER": 1},
    {"START_ORDER": 2}, {"CHAINS": 2048}, {"CHAINS": 2048, "WALKERS": 5, "START_ORDER": 1}, {"LEAN_LOOKS": 1},
    {"LEAN_LOOKS": 2}, {"LEAN_LOOKS": 2, "CHAINS": 2048}, {"LEAN_LOOKS": 1, "CHAINS": 2048, "SLOTS": 2}],
    ids=lambda o: "-".join("%s%d" % (k.lower(), v) for k, v in o.items()))
@pytest.mark.parametrize("name", sorted(CHAIN_GRAPHS))
def test_chain_sampler_options_change_nothing(kc, chain_reference, name, options):
    """Walkers, start order, table size, lean looks and slots on graphs the chain sampler takes."""
    g, first, (par, cnt, steps), f = chain_reference[name]
    print("chains", name, options, flush=True)
    with kc.Graph.from_graph(g) as G:
        if options == {"START_ORDER": 2}:
            # the chain sampler is in effect: with fewer walkers it takes more rounds
            few = []
            for walkers in (64, 4):
                G.set_option(kc.KC_OPT_WALKERS, walkers)
                few.append(G.estimate(23, first, 4).sampler_iterations)
            G.set_option(kc.KC_OPT_WALKERS, 64)
            assert few[1] > 2 * few[0]
        for key, value in options.items():
            G.set_option(getattr(kc, "KC_OPT_" + key), value)
        got = G.sample_trees(23, first, 4)
        assert np.array_equal(got[0].cpu().numpy(), par)
        assert np.array_equal(got[1].cpu().numpy().astype(np.uint32), cnt)
        assert np.array_equal(got[2].cpu().numpy(), steps)
        _, gf, gs = G.estimate(23, first, 4, per_sample=True)
        assert np.array_equal(gf.cpu().numpy(), f) and np.array_equal(gs.cpu().numpy(), steps)


@pytest.mark.parametrize("n,deg", [(70001, 10), (66000, 6)])
def test_path_sums_by_one_wavefront_with_more_vertices_than_bits(kc, oracle_lib, gen, n, deg):
    """A chain-sampled tree on a shallow tau0: its map of tau0 vertices has 65,536 bits."""
    g = random_graph(gen, n, deg)
    P = oracle_lib.prepare_graph(g)
    with kc.Graph.from_graph(g) as G:
        if deg == 10:
            assert 4 < G.info["depth0"] <= 8
        samples_match(G, oracle_lib, P, 3, 70, 4)


@pytest.mark.parametrize("other", ["grid", "social"])
def test_batch_with_a_job_of_the_chain_sampler(kc, oracle_lib, gen, other):
    """Every job of such a batch takes the chains (with lean looks if all of them would)."""
    gs = [random_graph(gen, 33001, 10), gen.grid(12, 12) if other == "grid" else gen.chung_lu(2000, 2.2, 10.0, 200.0, seed=1)]
    Gs = [kc.Graph.from_graph(g) for g in gs]
    with kc.Batch(Gs, [8, 9], [3, 1000], [2, 30]) as batch:
        for launch in range(3):
            batch.launch()
            ests, done = batch.results()
            assert done == launch + 1
            for j, (g, first, c) in enumerate(zip(gs, (3, 1000), (2, 30))):
                P = oracle_lib.prepare_graph(g)
                f, _ = oracle_lib.estimate_f(P, seed=8 + j, s0=first + launch * c, count=c, threads=8)
                assert np.array_equal(batch.f(j).cpu().numpy(), f)
                assert ests[j].sum_f == int(f.astype(object).sum())
    for G in Gs:
        G.close()


@pytest.mark.parametrize("hub", [0, 2500])
def test_trees_through_an_inserted_edge(kc, oracle_lib, gen, hub):
    """Basic maintenance draws replacements from two roots: on the chains (no hub) and by the
    frontier sampler with its words in memory."""
    g = random_graph(gen, 33001, 8, hub=hub)
    S = oracle_lib.samples_init(g.offsets, g.indices, seed=6, count=8)
    replaced = 0
    with kc.Graph.from_graph(g) as G:
        G.samples_init(6, 8)
        for serial, (u, v) in enumerate(gen.insertion_batch(g, 4, np.random.default_rng(1))):
            g = gen.add_edges(g, [(u, v)])
            S, k, _ = oracle_lib.bsm_insert(S, g.offsets, g.indices, u, v, serial)
            replaced += k
            assert G.apply_updates([u], [v], [1]) == k
            par, f, ids = G.samples_get()
            assert np.array_equal(par.cpu().numpy(), S.parents) and np.array_equal(ids, S.ids)
            assert np.array_equal(f.cpu().numpy(), S.f)
    assert replaced > 0


@pytest.mark.parametrize("name", ["path", "caterpillar", "grid"])
def test_step_limit_counts_two_frontier_rounds_as_one(kc, gen, name):
    """Where walks are longest bulk pops take up to 9% more rounds than the chains, for which
    limits were chosen: a limit a third below a sample's rounds holds, one far below does not."""
    i = np.arange(200)
    g = {"path": lambda: gen.path(300), "grid": lambda: gen.grid(32, 32),
         "caterpillar": lambda: gen.from_edges("cat", 400, np.concatenate([i[:-1], i]), np.concatenate([i[1:], i + 200]))}[name]()
    with kc.Graph.from_graph(g) as G:
        whole = G.estimate(3, 5, 1)
        G.set_option(kc.KC_OPT_STEP_LIMIT, max(1, whole.sampler_iterations * 2 // 3))
        assert G.estimate(3, 5, 1).sum_f == whole.sum_f
        G.set_option(kc.KC_OPT_STEP_LIMIT, max(1, whole.sampler_iterations // 3))
        with pytest.raises(kc.KcError) as ei:
            G.estimate(3, 5, 1)
        assert ei.value.status == 6


def test_path_sums_by_one_wavefront_on_a_power_law(kc, oracle_lib, gen):
    """The chains sample a power law whose root is a leaf; few vertices have terms of their own, so
    its one wavefront takes path sums, with more vertices than its map has bits."""
    g = gen.chung_lu(72000, 2.2, 10.0, 1300.0, seed=1)
    root = int(np.argmin(g.degrees))
    assert g.n > 65536
    P = oracle_lib.prepare_graph(g, root=root)
    with kc.Graph.from_graph(g, root=root) as G:
        assert G.info["depth0"] <= 8
        samples_match(G, oracle_lib, P, 3, 70, 3)
        assert on_chains(kc, G, 3, 70, 3)


@pytest.mark.parametrize("kind,n", [("ba2", 12000), ("random", 9001), ("ba2", 40000), ("hub", 40000)])
def test_numbering_on_a_shallow_tau0(kc, oracle_lib, gen, kind, n):
    """Graphs many of whose vertices have terms of their own: estimates and held trees."""
    import torch
    g = gen.barabasi_albert(n, 2, 1) if kind == "ba2" else random_graph(gen, n, 6, hub=3000 if kind == "hub" else 0)
    P = oracle_lib.prepare_graph(g)
    with kc.Graph.from_graph(g) as G:
        samples_match(G, oracle_lib, P, 5, 7, 4)
        par, _, _ = oracle_lib.sample(P, seed=5, s0=7, count=4, threads=8)
        f, _ = oracle_lib.estimate_f(P, seed=5, s0=7, count=4, threads=8)
        assert np.array_equal(G.evaluate_trees(torch.from_numpy(par).cuda()).cpu().numpy(), f)
