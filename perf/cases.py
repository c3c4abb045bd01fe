"""Timed cases of the library's public entry points (paper_1609_07228_amd.efanna).

The unit of work of a user is a kNN-graph build: efanna_build_trees, efanna_init_graph,
efanna_nndescent, efanna_get_graph on vectors that are resident on the GPU.  The builds listed
here have the shapes and parameters of the configurations in paper_1609_07228_amd/synth.py (the
largest one with fewer rows), and one shape that is a multiple of nothing.  The other cases are
the library's further directions: the conquer step above the leaves, the two other split rules of
the tree builder, refinement of a random start, and search with the finished index in large and
small batches.

A case is a dict:
  op      "build" | "conquer" | "trees" | "refine" | "search"
  data    value distribution, as in synth.py: "gauss", "u8grid", "unit" or "mixed"
  n, d    rows and coordinates;  T trees of leaves of at most S points
  K, L, I graph degree, NN-descent sample size and iterations
  up      (conquer) levels above a typical leaf (depth log2(n / 0.7 S)) that the conquer step visits
  rule    (trees) split rule, efanna.SPLIT_VARIANCE or efanna.SPLIT_PROJECTION
  nq, k, pool, expand, rounds   (search) queries, results per query, and the search's parameters

Every entry point promises the same bits for the same input (fixed order of float32 operations,
set semantics of the list updates), so all outputs are compared exactly.
"""
from __future__ import annotations

import math

import torch

from paper_1609_07228_amd import efanna, synth

SEED = synth.ALGO_SEED


def _case(name, op, data, n, d, K, T, S, I, L, **more):
    return dict(name=name, op=op, data=data, n=n, d=d, K=K, T=T, S=S, I=I, L=L, **more)


def listed():
    return [
        # the small configuration: a build of about a millisecond, where launches and latency count
        _case("build_10k_d32", "build", "gauss", 10_000, 32, 10, 4, 8, 4, 10),
        # the middle configuration: a descriptor set of 10^5 vectors, degree 20
        _case("build_100k_d128", "build", "u8grid", 100_000, 128, 20, 8, 16, 6, 20),
        # the headline configuration: a million integer-valued descriptors, degree 10
        _case("build_1m_d128", "build", "u8grid", 1_000_000, 128, 10, 8, 16, 8, 10),
        # long vectors: a million global image descriptors
        _case("build_1m_d960", "build", "unit", 1_000_000, 960, 10, 8, 16, 10, 10),
        # high degree: the K = 100 configuration with a quarter of its rows
        _case("build_1m_d96_k100", "build", "mixed", 1_000_000, 96, 100, 16, 64, 8, 50),
        # sizes that are multiples of nothing: embeddings of 50 coordinates, odd row length and leaves
        _case("build_200003_d50_k15", "build", "gauss", 200_003, 50, 15, 6, 13, 6, 13),
        # a better initial graph instead of more iterations: conquer three levels up (headline data)
        _case("conquer_1m_d128", "conquer", "u8grid", 1_000_000, 128, 10, 8, 16, 0, 0, up=3),
        # trees alone, split by variance, with the node table that search and conquer need
        _case("trees_variance_1m_d128", "trees", "u8grid", 1_000_000, 128, 0, 8, 16, 0, 0, rule=efanna.SPLIT_VARIANCE),
        # trees alone by random projections, which are meant for long vectors
        _case("trees_projection_200k_d960", "trees", "unit", 200_000, 960, 0, 8, 16, 0, 0,
              rule=efanna.SPLIT_PROJECTION),
        # NN-descent from a random graph (the plain method), on the entry point that allocates nothing
        _case("refine_random_100k_d128", "refine", "u8grid", 100_000, 128, 10, 0, 0, 10, 10),
        # a large batch of queries against the headline index
        _case("search_100k_queries_1m_d128", "search", "u8grid", 1_000_000, 128, 10, 8, 16, 4, 10,
              nq=100_000, k=10, pool=200, expand=50, rounds=4),
        # an online batch: what a server that collects requests for a moment hands in
        _case("search_64_queries_100k_d128", "search", "u8grid", 100_000, 128, 20, 8, 16, 3, 20,
              nq=64, k=10, pool=100, expand=50, rounds=4),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """A case of the ranges the listed ones stand for: any dimension, any row count, degrees and
    leaves up to the configurations' own."""
    op = rng.choices(["build", "conquer", "trees", "refine", "search"], [5, 1, 1, 1, 2])[0]
    data = rng.choice(["gauss", "u8grid", "unit", "mixed"])
    lo_n, hi_n, lo_d, hi_d = {"gauss": (2_000, 300_000, 8, 64), "u8grid": (20_000, 1_000_000, 64, 128),
                              "unit": (10_000, 300_000, 129, 960), "mixed": (10_000, 250_000, 48, 128)}[data]
    if op == "refine":
        hi_n = min(hi_n, 120_000)            # what fits the fixed scratch array at the degrees drawn below
    n, d = _log_int(rng, lo_n, hi_n), _log_int(rng, lo_d, hi_d)
    if op == "search" or rng.random() < 0.6:
        d = (d + 3) // 4 * 4                 # (search takes dimensions that are multiples of four)
    if data == "mixed" and op == "build":    # the high-degree regime
        K, S, T = rng.randint(40, 100), rng.randint(32, 64), rng.randint(4, 12)
        L = max(8, K // rng.randint(2, 4))
    elif data == "unit":                     # long vectors: joins of at most 32 (K + 2 L) of them
        K, S, T = rng.randint(6, 12), rng.randint(8, 16), rng.randint(3, 8)
        L = min(K, 10)
    else:
        K, S, T = rng.randint(6, 24), rng.randint(5, 20), rng.randint(3, 8)
        L = max(5, K - rng.randint(0, 3))
    I = rng.randint(3, 8)
    if op == "refine":
        K = L = min(K, 11)
    c = dict(op=op, data=data, n=n, d=d, K=K, T=T, S=S, I=I, L=L)
    if op == "conquer":
        c.update(up=rng.randint(1, 4))
    elif op == "trees":
        c.update(rule=rng.choice([efanna.SPLIT_VARIANCE, efanna.SPLIT_PROJECTION]))
    elif op == "search":
        pool = _log_int(rng, 40, 400)
        c.update(nq=_log_int(rng, 1, 100_000), k=rng.randint(1, 20), pool=pool,
                 expand=max(1, pool // rng.randint(2, 5)), rounds=rng.randint(2, 5), I=3)
    return c


def _mixture(data, n, d, gen, centres=None):
    """n vectors of the mixture `data`, one component per thousand rows, drawn on the GPU."""
    dev = "cuda"
    lo, hi, sigma = {"gauss": (-10.0, 10.0, 1.0), "u8grid": (0.0, 128.0, 16.0),
                     "unit": (0.0, 1.0, 0.05), "mixed": (-1.0, 1.0, 0.1)}[data]
    if centres is None:
        centres = lo + (hi - lo) * torch.rand((max(10, n // 1000), d), generator=gen, device=dev)
    comp = torch.randint(0, centres.shape[0], (n,), generator=gen, device=dev)
    X = torch.empty((n, d), dtype=torch.float32, device=dev)
    X.normal_(0.0, sigma, generator=gen)
    for r in range(0, n, 1 << 18):           # (in pieces: the gathered centres are as large as the rows)
        X[r:r + (1 << 18)] += centres[comp[r:r + (1 << 18)]]
    if data == "u8grid":
        X.clamp_(0.0, 255.0).round_()
    elif data == "unit":
        X.clamp_(0.0, 1.0)
    elif data == "mixed":
        spread = torch.rand(n, generator=gen, device=dev) < 0.5
        X[spread] = 2.0 * torch.rand((int(spread.sum()), d), generator=gen, device=dev) - 1.0
    return X, centres


def _max_leaves(case):
    return case["n"] // max(1, case["S"] // 4) + 16      # mean splits leave leaves well above a quarter full


def _conquer_depth(case):
    return max(0, int(math.log2(max(2.0, case["n"] / (0.7 * case["S"])))) - case["up"] + 1)


def _random_start(n, K, gen):
    """K random neighbours per point, never itself; a repeated draw is an empty slot."""
    ids = torch.randint(0, n - 1, (n, K), generator=gen, device="cuda")
    own = torch.arange(n, device="cuda")[:, None]
    ids = (ids + (ids >= own)).sort(dim=1).values
    ids[:, 1:][ids[:, 1:] == ids[:, :-1]] = -1
    return ids.int()


def prepare(case, seed):
    """The vectors, and the buffers, index or start that a program holds before the call."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    n, d, K, T, S, L, op = (case[x] for x in ("n", "d", "K", "T", "S", "L", "op"))
    X, centres = _mixture(case["data"], n, d, gen)
    st = {"case": case, "X": X}
    lib = efanna.lib()

    def space(nbytes):
        return torch.empty(max(256, nbytes), dtype=torch.uint8, device="cuda")

    if op != "refine":
        st["ws_trees"] = space(lib.efanna_trees_workspace_bytes(n, d, T, S, 0 if op == "build" else 1))
    if op == "build":
        st["ws_init"] = space(lib.efanna_init_workspace_bytes(n, 0))
        st["ws_nnd"] = space(lib.efanna_nndescent_workspace_bytes(n, K, L))
        st["graph"] = torch.empty((n, K), dtype=torch.int64, device="cuda")
        st["stats"] = torch.zeros((case["I"], 4), dtype=torch.int64, device="cuda")
    elif op == "conquer":
        st["ws_init"] = space(lib.efanna_init_workspace_bytes(n, 64))      # the most levels a call can ask for
        st["graph"] = torch.empty((n, K), dtype=torch.int64, device="cuda")
    elif op == "refine":
        start = _random_start(n, K, gen)
        own = torch.arange(n, dtype=torch.int32, device="cuda")[:, None].expand(n, K)
        st["ids"], st["a"], st["b"] = start, own.reshape(-1).contiguous(), start.clamp(min=0).reshape(-1).contiguous()
        st["stats"] = torch.zeros((case["I"], 4), dtype=torch.int64, device="cuda")
    elif op == "search":
        trees = efanna.efanna_build_trees(X, T, S, SEED, max_leaves=_max_leaves(case), workspace=st.pop("ws_trees"),
                                          with_nodes=True)
        graph = efanna.efanna_init_graph(X, trees[0], trees[1], trees[2], S, K)
        efanna.efanna_nndescent(X, graph, case["I"], L, SEED)
        st["trees"], st["graph_ids"] = trees, efanna.efanna_get_graph(graph)[0]
        st["Q"] = _mixture(case["data"], case["nq"], d, gen, centres)[0]
        st["ws_search"] = space(lib.efanna_search_workspace_bytes(case["nq"], d, T, S, trees[5], K, case["pool"],
                                                                  case["rounds"]))
    return st


def run(st):
    c, X = st["case"], st["X"]
    T, S, K, op = c["T"], c["S"], c["K"], c["op"]
    if op == "build":
        perm, off, n_leaves = efanna.efanna_build_trees(X, T, S, SEED, max_leaves=_max_leaves(c),
                                                        workspace=st["ws_trees"])
        graph = efanna.efanna_init_graph(X, perm, off, n_leaves, S, K, graph=st["graph"], workspace=st["ws_init"])
        efanna.efanna_nndescent(X, graph, c["I"], c["L"], SEED, stats=st["stats"], workspace=st["ws_nnd"])
        return efanna.efanna_get_graph(graph)
    if op == "conquer":
        perm, off, n_leaves, nodes, up, depth = efanna.efanna_build_trees(
            X, T, S, SEED, max_leaves=_max_leaves(c), workspace=st["ws_trees"], with_nodes=True)
        graph = efanna.efanna_init_graph(X, perm, off, n_leaves, S, K, graph=st["graph"], workspace=st["ws_init"],
                                         nodes=nodes, leaf_up=up, tree_depth=depth,
                                         conquer_depth=_conquer_depth(c))
        return efanna.efanna_get_graph(graph, with_flags=True)
    if op == "trees":
        perm, off, n_leaves, nodes, up, depth = efanna.efanna_build_trees_rule(
            X, T, S, SEED, c["rule"], max_leaves=_max_leaves(c), workspace=st["ws_trees"], with_nodes=True)
        # (the call leaves the offsets beyond a tree's leaves as they were: the end of the last leaf there)
        for t, leaves in enumerate(n_leaves):
            off[t, leaves:] = c["n"]
        return perm, n_leaves, depth, off, nodes, up
    if op == "refine":
        dist = efanna.efanna_pair_distances(X, st["a"], st["b"])
        start = dist.view(c["n"], K).masked_fill(st["ids"] < 0, float("inf"))
        graph = efanna.efanna_set_graph(st["ids"], start)
        efanna.efanna_nndescent_noalloc(X, graph, c["I"], c["L"], SEED, st["stats"])
        return (dist,) + efanna.efanna_get_graph(graph, with_flags=True)
    perm, off, n_leaves, nodes, _, depth = st["trees"]
    return efanna.efanna_search(X, perm, off, n_leaves, nodes, depth, S, st["graph_ids"], st["Q"], c["k"], c["pool"],
                                c["expand"], c["rounds"], workspace=st["ws_search"])


def work(case):
    """Each input read once, each output written once; the distances that are certain to be
    evaluated (leaves are about 0.7 S full; the first iteration joins every point's own L entries)."""
    n, d, K, T, S, L, op = (case[x] for x in ("n", "d", "K", "T", "S", "L", "op"))
    rows = 4.0 * n * d
    leaf_pairs = T * n * max(1.0, 0.7 * S - 1) / 2
    first_joins = n * min(K, L) * (min(K, L) - 1) / 2
    if op == "build":
        return {"bytes": rows + 8.0 * n * K, "flops": 3.0 * d * (leaf_pairs + first_joins)}
    if op == "conquer":
        return {"bytes": rows + 9.0 * n * K, "flops": 3.0 * d * (leaf_pairs + T * n * 0.7 * S * case["up"])}
    if op == "trees":
        return {"bytes": rows + T * (4.0 * n + 40.0 * n / (0.7 * S)), "flops": 3.0 * T * n * math.log2(max(2, n / S))}
    if op == "refine":
        return {"bytes": rows + 24.0 * n * K, "flops": 3.0 * d * (n * K + first_joins)}
    nq = case["nq"]
    return {"bytes": 4.0 * d * min(n, nq * case["pool"]) + nq * (4.0 * d + 8.0 * case["k"] + 4),
            "flops": 3.0 * d * nq * case["pool"]}


def tolerance(case):
    return "exact"


def exact(case, seed):
    """The start's distances in 64 bits.  A graph's or a search's own distances have no such value:
    they belong to the neighbours that the method happens to reach."""
    if case["op"] != "refine":
        return None
    st = prepare(case, seed)
    out = [((st["X"][a.long()].double() - st["X"][b.long()].double()) ** 2).sum(1)
           for a, b in zip(st["a"].split(1 << 18), st["b"].split(1 << 18))]
    return (torch.cat(out), None, None, None)
