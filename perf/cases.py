"""The retrieval work a search agent's serving process has this library do, as cases that can be timed.

A case is a dict of plain values.  Its "kind" says which public entry points one pass goes through:

    flat      exact search of B queries over an [N, d] corpus
    rows      exact search in pages of 16 (each page continues after the last), as the k-NN rows of a
              graph index are built cluster by cluster
    graph     best-first graph search; "entry" is "shared" (one entry node for all queries) or "coarse"
              (exact search over one representative per cluster, node ids gathered, search from there)
    nonstall  graph search with the maturity exit and its counters, coarse entries
    order     priority levels and execution order of a batch of requests

Inputs are the clustered corpora, noisy queries and proximity graphs of the generator module, made on
the GPU from the seed.  Sizes are those of the workload table, its scaled forms, the paper-shaped
workload (21 M x 384, k = 5) and the test suite.
"""
import math

import torch

import paper_2505_12065_amd as ann
from paper_2505_12065_amd import synth

DEV = "cuda:0"
DTYPES = {"f16": torch.float16, "bf16": torch.bfloat16, "f32": torch.float32}
BYTES = {"f16": 2, "bf16": 2, "f32": 4}
PAGE = ann.binding.ANN_K_MAX


def listed():
    return [
        # the scheduler puts the requests of a serving batch in order before every step
        {"name": "order", "kind": "order", "n": 3000, "G": 6},
        # the smallest configuration: a little fp32 knowledge base, a few agents at once
        {"name": "flat f32 small", "kind": "flat", "N": 10_000, "d": 128, "dtype": "f32", "B": 16, "k": 10},
        # the coarse level of a graph search: one representative per cluster, a whole batch of queries
        {"name": "flat coarse", "kind": "flat", "N": 1024, "d": 768, "dtype": "f16", "B": 512, "k": 1},
        # graph index build: the members of one cluster against all points whose pool holds it, 33 rows each
        {"name": "rows", "kind": "rows", "N": 977, "d": 768, "dtype": "f16", "B": 5000, "pages": 3},
        # one agent asks, exactly, over a million passages
        {"name": "flat one", "kind": "flat", "N": 1_000_000, "d": 768, "dtype": "f16", "B": 1, "k": 3},
        # every agent of a large serving batch asks at once
        {"name": "flat batch", "kind": "flat", "N": 1_000_000, "d": 768, "dtype": "f16", "B": 512, "k": 3},
        # the same over the paper's 21 M passages of 384 dimensions, for some tens of agents
        {"name": "flat 21M", "kind": "flat", "N": 21_000_000, "d": 384, "dtype": "f16", "B": 64, "k": 5},
        # odd sizes throughout: a row that is no whole number of 64-byte steps, ragged rows and queries
        {"name": "flat ragged", "kind": "flat", "N": 123_457, "d": 776, "dtype": "bf16", "B": 77, "k": 10},
        # one agent asks approximately: latency of coarse search, gather and graph search in a row
        {"name": "graph one", "kind": "graph", "N": 200_000, "d": 768, "dtype": "f16", "R": 32, "B": 1, "k": 3,
         "ef": 64, "entry": "coarse"},
        # the workload table's graph batch: shared entry node, short candidate list
        {"name": "graph batch", "kind": "graph", "N": 200_000, "d": 768, "dtype": "f16", "R": 32, "B": 512, "k": 3,
         "ef": 64, "entry": "shared"},
        # high recall: a long candidate list
        {"name": "graph long", "kind": "graph", "N": 200_000, "d": 768, "dtype": "f16", "R": 32, "B": 256, "k": 3,
         "ef": 2048, "entry": "coarse"},
        # the paper's non-stall retrieval, in bf16 at its own width and k
        {"name": "nonstall", "kind": "nonstall", "N": 200_000, "d": 384, "dtype": "bf16", "R": 32, "B": 256, "k": 5,
         "ef": 256, "tau": 0.9, "window": 500},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _dim(rng, dtype):
    if rng.random() < 0.75:                              # embedding widths are mostly multiples of 32
        return 32 * _log(rng, 2, 32)
    step = 4 if dtype == "f32" else 8
    return step * _log(rng, 64 // step, 1024 // step)


def draw(rng):
    kind = rng.choice(["flat"] * 5 + ["graph"] * 3 + ["nonstall", "rows", "order"])
    if kind == "order":
        return {"kind": kind, "n": _log(rng, 32, 16384), "G": rng.choice([3, 6, 6, 6, 13])}
    dtype = rng.choice(["f16", "f16", "bf16", "f32"])
    d = _dim(rng, dtype)
    if kind == "rows":
        return {"kind": kind, "N": _log(rng, 64, 4096), "d": d, "dtype": dtype if dtype != "f32" else "f16",
                "B": _log(rng, 256, 8192), "pages": rng.choice([1, 2, 3])}
    if kind == "flat":
        N, B, k = _log(rng, 1000, 4_000_000), _log(rng, 1, 1024), rng.choice([1, 3, 3, 5, 10, 16])
        most = 4e10 if dtype == "f32" else 4e11          # multiply-adds, as flops, of one pass
        if 2.0 * N * d * B > most:                        # the batch gives way
            B = max(1, int(most / (2.0 * N * d)))
        return {"kind": kind, "N": N, "d": d, "dtype": dtype, "B": B, "k": k}
    case = {"kind": kind, "N": _log(rng, 20_000, 200_000), "d": d, "dtype": dtype, "R": rng.choice([8, 16, 24, 31, 32, 32]),
            "B": _log(rng, 1, 1024), "k": rng.choice([1, 3, 5, 10]), "ef": _log(rng, 16, 2048)}
    if case["B"] * case["ef"] > 256 * 2048:
        case["B"] = 256 * 2048 // case["ef"]
    if kind == "graph":
        return dict(case, entry=rng.choice(["shared", "coarse"]))
    return dict(case, tau=rng.choice([0.9, 0.9, 3.0]), window=500)


def prepare(case, seed):
    if case["kind"] == "order":
        g = torch.Generator().manual_seed(seed)
        n = case["n"]
        R = torch.randint(0, 9, (n,), generator=g, dtype=torch.int32)              # retrievals completed
        C = torch.randint(64, 8192, (n,), generator=g, dtype=torch.int32)          # context lengths
        W = torch.rand(n, generator=g, dtype=torch.float64) * 60                   # waiting times, s
        Wcur = (torch.rand(n, generator=g, dtype=torch.float64) * 50).round() / 10  # queueing times; equal ones occur
        return {"case": case, "args": [t.to(DEV) for t in (R, W, C, Wcur)]}
    N, d, dtype = case["N"], case["d"], DTYPES[case["dtype"]]
    clusters = 16 if N <= 20_000 else min(4096, N // 1000)
    if case["kind"] in ("graph", "nonstall"):
        clusters = N // 1000
    corpus = synth.make_corpus(N, d, clusters, seed, dtype=dtype, device=DEV)
    q = synth.make_queries(corpus, case["B"])
    state = {"case": case, "x": corpus.x, "q": q}
    if case["kind"] in ("graph", "nonstall"):
        graph = synth.knn_graph_cluster_restricted(corpus, case["R"], 8)
        if case.get("entry") == "shared":                 # the workload table's graph and entry as they stand
            state["entry"] = synth.mean_entry(corpus.x)
        else:                                             # the navigable form, with a coarse index beside it
            graph = synth.with_reverse_edges(graph, corpus.x)
            state["reps"] = synth.cluster_representatives(corpus)
            state["rep_rows"] = corpus.x[state["reps"].long()].contiguous()
        state["graph"] = graph
    return state


def _coarse_entries(state):
    idx, _ = ann.ann_flat_search_typed(state["rep_rows"], state["q"], 1)
    return ann.ann_gather_ids(state["reps"], idx.view(-1))


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "order":
        return ann.ann_priority_order(*state["args"], case["G"])
    x, q = state["x"], state["q"]
    if kind == "flat":
        return ann.ann_flat_search_typed(x, q, case["k"])
    if kind == "rows":
        k = min(PAGE, case["N"])
        out, after = [], None
        for _ in range(case["pages"]):
            ids, scores = ann.ann_flat_search_typed(x, q, k, after=after)
            out += [ids, scores]
            after = (scores[:, -1].contiguous(), ids[:, -1].contiguous())
        return out
    if kind == "graph":
        if case["entry"] == "shared":
            return ann.ann_graph_search_typed(x, state["graph"], state["entry"], q, case["k"], case["ef"])
        return ann.ann_graph_search_entries_typed(x, state["graph"], _coarse_entries(state), q, case["k"], case["ef"])
    return ann.ann_graph_search_nonstall_typed(x, state["graph"], 0, q, case["k"], case["ef"], entries=_coarse_entries(state),
                                               tau=case["tau"], window=case["window"])


def work(case):
    if case["kind"] == "order":
        return {"bytes": case["n"] * (4 + 8 + 4 + 8 + 4 + 4), "flops": 0}
    N, d, B, size = case["N"], case["d"], case["B"], BYTES[case["dtype"]]
    if case["kind"] == "flat":
        return {"bytes": (N + B) * d * size + B * case["k"] * 8, "flops": 2 * B * N * d}
    if case["kind"] == "rows":                            # every page is a search of its own
        return {"bytes": case["pages"] * ((N + B) * d * size + B * PAGE * 8), "flops": case["pages"] * 2 * B * N * d}
    # A search ends when all ef entries of a full list have been expanded: at least that many nodes are
    # scored (their rows are read) and at least that many adjacency rows are read.  (The number of nodes
    # it really scores depends on the data; it is several times as large.)
    listed_nodes = min(case["ef"], N // 2)
    return {"bytes": B * (listed_nodes * (d * size + case["R"] * 4) + d * size + case["k"] * 8),
            "flops": 2 * B * listed_nodes * d}


def tolerance(case):
    # Scores are sums of exact products (16 bits) or fp32 products, accumulated in fp32; another order of
    # summation moves them by about 1e-6 and can swap two rows whose scores are that close.
    if case["kind"] == "order":
        return "exact"
    return {"rel": 1e-5, "max": 1e-4, "differ": 0.005}
