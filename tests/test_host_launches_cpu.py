"""What the library's host code launches, on the CPU: the built library over a stand-in
runtime (hip_stub.cpp) that writes the launches down and runs none of them.  Each test is a
program of its own, so that the stand-in never meets the real runtime's state."""
import json
import os
import subprocess
import sys
import textwrap

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)

PRELUDE = """
import ctypes, json, sys
stub = ctypes.CDLL(%(stub)r, ctypes.RTLD_GLOBAL)
for f in ("stub_name", "stub_out"):
    getattr(stub, f).restype = ctypes.c_char_p if f == "stub_name" else ctypes.c_void_p
stub.stub_lds.restype = ctypes.c_size_t
stub.stub_set.argtypes = [ctypes.c_size_t, ctypes.c_int]
sys.path.insert(0, %(root)r)
import numpy as np
import graphgen as gen
import paper_2511_16356_amd as kc
lib = kc.library()
def graph(g, root=-1):
    off, idx = np.ascontiguousarray(g.offsets, np.int64), np.ascontiguousarray(g.indices, np.int32)
    h = ctypes.c_void_p()
    st = lib.kc_graph_create(g.n, off.ctypes.data, 1, idx.ctypes.data, root, None, ctypes.byref(h))
    assert st == 0, lib.kc_last_error()
    return h
def launches(clear=True):
    out = [dict(name=stub.stub_name(i).decode(), grid=stub.stub_grid(i), block=stub.stub_block(i), lds=stub.stub_lds(i),
                out=stub.stub_out(i), levels=stub.stub_levels(i)) for i in range(stub.stub_launches())]
    if clear: stub.stub_clear()
    return out
def estimate(h, count):
    stub.stub_clear()
    st = lib.kc_estimate(h, 1, 0, count, ctypes.byref(kc._Result()), None, None, None)
    return st, launches()
def sampler(ls):
    return [l for l in ls if "persistent_kernel" in l["name"] or "frontier" in l["name"] or "batch_kernel" in l["name"]][0]
def kind(ls):
    l = sampler(ls)
    return "chains" if "frontier" not in l["name"] else "lds" if l["block"] == 256 else "global"
"""


@pytest.fixture(scope="module")
def run(tmp_path_factory):
    import paper_2511_16356_amd as kc
    if not os.path.exists(kc.LIB_PATH):
        from paper_2511_16356_amd import build_lib
        build_lib.build()
    import graphgen
    graphgen.build()
    so = str(tmp_path_factory.mktemp("stub") / "libhip_stub.so")
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-o", so, os.path.join(HERE, "hip_stub.cpp")], check=True)

    def go(body):
        code = PRELUDE % {"stub": so, "root": ROOT} + textwrap.dedent(body)
        r = subprocess.run([sys.executable, "-c", code], capture_output=True, text=True, timeout=300)
        assert r.returncode == 0, r.stderr[-3000:]
        return json.loads(r.stdout.strip().splitlines()[-1])
    return go


def test_a_result_block_without_a_device_view_is_not_used(run):
    """The pinned block is replaced when a launch has more slots than it holds counters; if its
    device view cannot be had, the call fails, and later reductions must not write through null."""
    r = run("""
        h = graph(gen.grid(8, 8))
        assert lib.kc_samples_init(h, 1, 16, None) == 0
        stub.stub_fail(b"hipHostGetDevicePointer")
        st, _ = estimate(h, 400)
        stub.stub_clear()
        q = lib.kc_samples_query(h, ctypes.byref(kc._Result()), None)
        out = [l["out"] for l in launches() if "reduce_kernel" in l["name"]]
        st2, _ = estimate(h, 400)
        print(json.dumps(dict(st=st, q=q, out=out, st2=st2)))
    """)
    assert r["st"] != 0 and r["q"] == 0 and r["st2"] == 0
    assert len(r["out"]) == 1 and r["out"][0]


ROUTE_GRAPHS = """
def random_graph(n, deg, seed=1):
    rng = np.random.default_rng(seed)
    k = n * (deg - 2) // 2
    u = np.concatenate([np.arange(n), rng.integers(0, n, k)])
    v = np.concatenate([(np.arange(n) + 1) % n, rng.integers(0, n, k)])
    return gen.from_edges("random", n, u[u != v], v[u != v])
def hubs(n, deg, hub=2000, seed=1):  # the same with a vertex that `hub` others are joined to
    g = random_graph(n, deg, seed)
    e = np.array([(x, y) for x, y in g.edges()])
    return gen.from_edges("hubs", n, np.concatenate([e[:, 0], np.zeros(hub, int)]), np.concatenate([e[:, 1], np.arange(2, 2 + hub)]))
"""


def test_route_follows_the_graph_not_tau0(run):
    """Above the LDS sizes the frontier sampler takes a lean graph whose root holds many edge ends,
    with any reference tree; random graphs without such a root (long walks) and sparse ones go to
    the chains."""
    r = run(ROUTE_GRAPHS + """
        out = {}
        h = graph(hubs(33000, 10))
        out["hubs"] = kind(estimate(h, 64)[1])
        assert lib.kc_set_tau0(h, kc.KC_TAU0_DFS, None, None) == 0
        info = kc._Info(); lib.kc_graph_get_info(h, ctypes.byref(info))
        out["depth"] = info.depth0
        out["hubs dfs"] = kind(estimate(h, 64)[1])
        assert lib.kc_set_tau0(h, kc.KC_TAU0_BFS, None, None) == 0
        out["hubs bfs"] = kind(estimate(h, 64)[1])
        out["leaf root"] = kind(estimate(graph(hubs(33000, 10), root=30000), 64)[1])
        out["random"] = kind(estimate(graph(random_graph(33000, 12)), 64)[1])
        out["grid"] = kind(estimate(graph(gen.grid(200, 200)), 64)[1])
        out["small"] = kind(estimate(graph(random_graph(2000, 12)), 64)[1])
        print(json.dumps(out))
    """.replace("\n        ", "\n"))
    assert r.pop("depth") > 100
    assert r == {"hubs": "global", "hubs dfs": "global", "hubs bfs": "global", "leaf root": "chains", "random": "chains",
                 "grid": "chains", "small": "lds"}


@pytest.mark.parametrize("per_cu,count,expect", [(1, 1792, "lds"), (1, 1793, "chains"), (2, 7168, "lds"), (2, 7169, "chains"),
                                                 (3, 100000, "lds")])
def test_many_samples_of_a_lattice_take_the_chains(run, per_cu, count, expect):
    """Words in LDS let few trees be in flight; the limits are whole waves of them."""
    r = run("""
        stub.stub_set(64 << 30, %d)
        h = graph(gen.grid(135, 135))
        ls = estimate(h, %d)[1]
        print(json.dumps(dict(kind=kind(ls), slots=sampler(ls)["grid"])))
    """ % (per_cu, count))
    assert r["kind"] == expect
    most = min(count, 2560 if expect == "chains" else 256 * per_cu)
    assert most // 2 < r["slots"] <= most


def test_many_samples_with_few_slots_or_a_short_way_to_the_root_stay_in_lds(run):
    r = run(ROUTE_GRAPHS + """
stub.stub_set(64 << 30, 1)
out = {}
h = graph(gen.grid(135, 135))
lib.kc_set_option(h, kc.KC_OPT_SLOTS, 2000)
out["slots"] = kind(estimate(h, 5000)[1])
lib.kc_set_option(h, kc.KC_OPT_SLOTS, 0)
info = kc._Info(); lib.kc_graph_get_info(h, ctypes.byref(info))
lib.kc_set_option(h, kc.KC_OPT_MEM_BUDGET, 500 * info.sample_bytes)
ls = estimate(h, 5000)[1]
out["budget"] = [kind(ls), sampler(ls)["grid"] <= 256]
lib.kc_set_option(h, kc.KC_OPT_MEM_BUDGET, 0)
lib.kc_trim(h, None)
out["none"] = kind(estimate(h, 5000)[1])
out["star"] = kind(estimate(graph(gen.star(20000)), 20000)[1])
out["random"] = [kind(estimate(graph(random_graph(20000, 8)), c)[1]) for c in (3072, 3073)]
def batch(*jobs):
    hs = (ctypes.c_void_p * len(jobs))(*[graph(g).value for g, _ in jobs])
    sd, fi = np.zeros(len(jobs), np.uint64), np.zeros(len(jobs), np.int64)
    co, b = np.array([c for _, c in jobs], np.int32), ctypes.c_void_p()
    stub.stub_clear()
    assert lib.kc_batch_create(hs, len(jobs), sd.ctypes.data, fi.ctypes.data, co.ctypes.data, None, ctypes.byref(b)) == 0
    return kind(launches())
out["batch"] = [batch((gen.grid(135, 135), 2000)), batch((gen.grid(135, 135), 1500)), batch((gen.grid(135, 135), 2000), (gen.grid(8, 8), 10))]
print(json.dumps(out))
""")
    assert r == {"slots": "lds", "budget": ["lds", True], "none": "chains", "star": "lds", "random": ["lds", "chains"],
                 "batch": ["chains", "lds", "lds"]}


BATCH = """
def batch(*jobs):
    hs = (ctypes.c_void_p * len(jobs))(*[graph(g).value for g, _ in jobs])
    sd, fi = np.zeros(len(jobs), np.uint64), np.zeros(len(jobs), np.int64)
    co, b = np.array([c for _, c in jobs], np.int32), ctypes.c_void_p()
    stub.stub_clear()
    assert lib.kc_batch_create(hs, len(jobs), sd.ctypes.data, fi.ctypes.data, co.ctypes.data, None, ctypes.byref(b)) == 0
    return launches()
"""


def test_a_batch_asks_for_the_lds_of_its_own_threads(run):
    """No more than a launch over its largest graph alone, but for a sweep by more threads."""
    r = run(ROUTE_GRAPHS + BATCH + """
out = []
for gs in ([gen.grid(32, 32), gen.grid(16, 16)], [gen.grid(32, 32), hubs(33000, 10)], [gen.grid(150, 200), gen.grid(8, 8)]):
    one = [sampler(estimate(graph(g), 10)[1]) for g in gs]
    b = sampler(batch(*[(g, 10) for g in gs]))
    out.append([b["block"], b["lds"], max(l["block"] for l in one), max(l["lds"] for l in one)])
print(json.dumps(out))
""")
    (b0, l0, *one0), (b1, l1, *one1), (b2, l2, *one2) = r
    assert [b0, l0] == one0 and [b2, l2] == one2
    assert b1 == one1[0] == 512 and l1 == 2 * 512 * 24 + 2048 * 8


def test_a_launch_asks_for_the_lds_its_traversal_takes(run):
    """The sweep's 1,024 or 512 items of 24 bytes and 2,048 nodes of 8, the path sums' bit per
    vertex (at most 2^19), or the words if those are more."""
    r = run("""
        def evaluate(h, n):
            par, f = np.zeros(n, np.int32), np.zeros(1, np.int64)
            stub.stub_clear()
            assert lib.kc_evaluate_trees(h, par.ctypes.data, 1, f.ctypes.data, None) == 0
            return launches()
        def lds(ls):
            return [[l["block"], l["lds"]] for l in ls if "tree_kernel" in l["name"] or "frontier" in l["name"]]
        out = []
        for g in (gen.cycle(300000), gen.star(300000), gen.star(600000), gen.grid(20, 20), gen.star(400), gen.grid(100, 150)):
            h = graph(g)
            out += lds(evaluate(h, g.n))
            if g.n < 32768: out += lds(estimate(h, 4)[1])
        print(json.dumps(out))
    """)
    sweep = 2 * 256 * 24 + 2048 * 8
    assert r == [[256, sweep], [512, 1 << 16], [512, 1 << 16], [256, sweep], [256, sweep], [256, 64], [256, 1600],
                 [256, sweep], [256, 60000]]


def test_no_call_lowers_the_lds_limit_of_another(run):
    """The limit belongs to the kernel: one thread may set it and launch while another sets it for a
    smaller graph.  After any call it covers the largest graph's words."""
    r = run(BATCH + """
stub.stub_limit.restype = ctypes.c_size_t
out = []
for g in (gen.grid(150, 200), gen.grid(130, 140), gen.grid(10, 10)):
    st, ls = estimate(graph(g), 4)
    assert st == 0
    out.append(["frontier_kernel", stub.stub_limit(b"frontier_kernel")])
for g in (gen.grid(150, 200), gen.grid(130, 140)):
    batch((g, 3))
    out.append(["frontier_batch_kernel", stub.stub_limit(b"frontier_batch_kernel")])
print(json.dumps(out))
""")
    assert all(limit >= 4 * 32767 for _, limit in r)


def test_autotune_tries_what_the_sampler_has(run, tmp_path):
    """Chains and walkers are tried for the chain sampler alone, and a choice kept for it (a key
    without the sampler's name) is not applied to a graph that another sampler takes."""
    r = run("""
        def tune(h, path):
            t = kc._Tune()
            assert lib.kc_autotune(h, 100, path, ctypes.byref(t), None) == 0, lib.kc_last_error()
            return t
        out = []
        for name, g in (("lds", gen.grid(60, 60)), ("chains", gen.grid(182, 182))):
            h = graph(g)
            info = kc._Info(); lib.kc_graph_get_info(h, ctypes.byref(info))
            path = %r + name
            key = "unknown|n=%%d|two_m=%%d|dmax=%%d|depth0=%%d|count=100" %% (info.n, info.two_m, info.max_degree, info.depth0)
            first = tune(h, path.encode())
            again = tune(h, path.encode())
            with open(path + ".old", "w") as fh:
                fh.write(json.dumps({"key": key, "chains": 2048, "slots": 77, "walkers": 32, "traversal": 0}) + "\\n")
            old = tune(h, (path + ".old").encode())
            out.append([name, first.trials, again.from_cache, old.from_cache, old.slots == 77])
        print(json.dumps(out))
    """ % str(tmp_path / "tune-"))
    assert r == [["lds", 3, 1, 0, False], ["chains", 5, 1, 1, True]]


def test_path_sums_where_few_vertices_have_terms(run):
    """A shallow tau0's table goes to the kernels where the path sums are the faster evaluation."""
    r = run(ROUTE_GRAPHS + """
def evaluate(h, n):
    par, f = np.zeros(n, np.int32), np.zeros(1, np.int64)
    stub.stub_clear()
    assert lib.kc_evaluate_trees(h, par.ctypes.data, 1, f.ctypes.data, None) == 0
    return [l["levels"] for l in launches() if "tree_kernel" in l["name"]][0]
out = {}
for name, g in (("small", random_graph(3000, 8)), ("deg8", random_graph(9000, 8)), ("deg12", random_graph(33000, 12)),
                ("social", gen.chung_lu(20000, 2.2, 10.0, 700.0, seed=0)), ("star", gen.star(40000)),
                ("ba2", gen.barabasi_albert(20000, 2, 1))):
    h = graph(g)
    out[name] = [evaluate(h, g.n) > 0, sampler(estimate(h, 4)[1])["levels"] > 0]
print(json.dumps(out))
""")
    assert r == {"small": [True, True], "deg8": [False, False], "deg12": [True, False], "social": [True, True],
                 "star": [True, True], "ba2": [False, False]}


def test_sparse_graphs_with_a_large_root_take_the_frontier_sampler(run):
    r = run("""
        print(json.dumps([kind(estimate(graph(g), 64)[1]) for g in (gen.barabasi_albert(40000, 2, 1), gen.star(40000),
                          gen.chung_lu(60000, 2.2, 4.0, 2000.0, seed=0))]))
    """)
    assert r == ["global", "global", "global"]


def test_lean_looks_by_default_where_walks_are_short(run):
    """The chain sampler's variants by their names' last argument; walks are long on a random graph,
    and a lean graph with a large root takes the chains in a batch with a grid."""
    r = run(ROUTE_GRAPHS + BATCH + """
def lean(ls): return "Lb1E" in sampler(ls)["name"]
h = graph(random_graph(33000, 12))
out = [lean(estimate(h, 4)[1])]
lib.kc_set_option(h, kc.KC_OPT_LEAN_LOOKS, 2)
out.append(lean(estimate(h, 4)[1]))
out.append(lean(batch((random_graph(33000, 12), 4), (hubs(33000, 10), 4))))
print(json.dumps(out))
""")
    assert r == [False, True, False]
