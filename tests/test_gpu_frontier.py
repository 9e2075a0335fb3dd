"""The graph search without a written list (graph_frontier_kernel) at the edges of its layouts: lists of 64 entries and one
more, answers longer than a wave, more scored nodes than its array holds (a bound is found), rows beyond 128 chunks, one, two and
three workgroups per compute unit, the visited set in memory, hundreds of equal scores, 32 entry nodes with NaN rows among
them.  Ids, scores and counters against the oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_2505_12065_amd as ann
from parity import compare_topk, np_dtype_name, to_np

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def say(*a):
    """Names the case before its GPU work."""
    print(*a, flush=True)


def _random(N, d, R, B, dtype, seed):
    gen = torch.Generator().manual_seed(seed)
    x = torch.nn.functional.normalize(torch.randn(N, d, generator=gen), dim=1).to(dtype)
    q = torch.nn.functional.normalize(torch.randn(B, d, generator=gen), dim=1).to(dtype)
    g = torch.randint(-1, N + 1, (N, R), generator=gen, dtype=torch.int32)        # empty slots, nodes that are none
    return x, q, g


@pytest.mark.parametrize("dtype,N,d,R,B,ef,k,seed", [
    (torch.float16, 5000, 64, 32, 3, 64, 64, 1),         # nothing below the 64 best is kept at all
    (torch.float16, 5000, 64, 32, 3, 65, 65, 2),         # ... and a pool
    (torch.float16, 20_000, 200, 31, 2, 100, 100, 3),    # scores more nodes than the array holds
    (torch.bfloat16, 9000, 776, 8, 257, 66, 5, 4),       # a row that ends inside a run of chunks; two workgroups
    (torch.float32, 6000, 1028, 17, 1, 130, 3, 5),       # 257 chunks
    (torch.float16, 3000, 136, 16, 513, 130, 70, 6),     # three workgroups
    (torch.float16, 120_000, 64, 32, 2, 16_384, 130, 7),  # visited set in memory
    (torch.float16, 40, 8, 1, 2, 40, 40, 8),             # one chunk, one slot: a path
    (torch.bfloat16, 9000, 776, 8, 257, 80, 5, 9),       # two workgroups, with the counters too
])
def test_graph_frontier(dtype, N, d, R, B, ef, k, seed):
    say(f"frontier: {dtype} N={N} d={d} R={R} B={B} ef={ef} k={k}")
    x, q, g = _random(N, d, R, B, dtype, seed)
    xn, qn, name = to_np(x), to_np(q), np_dtype_name(x)
    ids, sc = ann.ann_graph_search_typed(x.to(DEV), g.to(DEV), 3, q.to(DEV), k, ef)
    # an engine that is never ready: the natural stop, with counters and the averages kept
    n_ids, n_sc, stats, _ = ann.ann_graph_search_nonstall_typed(x.to(DEV), g.to(DEV), 3, q.to(DEV), k, ef, tau=0.999, window=10,
                                                                engine_ready=torch.zeros(1, dtype=torch.int32, device=DEV))
    torch.cuda.synchronize()
    o_ids, _, o_sc64, n_dist, n_expand = oracle.graph_search(xn, g.numpy(), 3, qn, k, ef, dtype=name)
    strict, tolerant, n = compare_topk(ids.cpu().numpy(), sc.cpu().numpy(), o_ids, o_sc64, xn, qn, dtype=name)
    assert strict >= n - max(2, n // 100), (strict, n)
    assert torch.equal(ids, n_ids) and torch.equal(sc, n_sc)
    st = stats.cpu().numpy()
    # (scores of the two sides differ by about 1e-7: now and then two nodes change places)
    assert (st[:, 0] == 0).all() and ((st[:, 1] == n_dist) & (st[:, 2] == n_expand)).mean() >= 0.99


@pytest.mark.parametrize("ef,k,B", [(200, 9, 2), (64, 64, 300), (700, 100, 1)])
def test_graph_frontier_equal_scores(ef, k, B):
    """Every score occurs hundreds of times: order and list are decided by the node numbers, to the last one."""
    say(f"frontier, equal scores: ef={ef} k={k} B={B}")
    N, d, R = 6000, 64, 24
    gen = torch.Generator().manual_seed(ef)
    rows = torch.nn.functional.normalize(torch.randn(12, d, generator=gen), dim=1).half()
    x = rows[torch.randint(0, 12, (N,), generator=gen)].contiguous()
    q = torch.nn.functional.normalize(torch.randn(B, d, generator=gen), dim=1).half()
    g = torch.randint(0, N, (N, R), generator=gen, dtype=torch.int32)
    ids, sc = ann.ann_graph_search_typed(x.to(DEV), g.to(DEV), 7, q.to(DEV), k, ef)
    torch.cuda.synchronize()
    o_ids, _, _, _, _ = oracle.graph_search(to_np(x), g.numpy(), 7, to_np(q), k, ef)
    assert np.array_equal(ids.cpu().numpy(), o_ids)


@pytest.mark.parametrize("ef", [16, 64, 300])
def test_graph_frontier_entries_and_nan(ef):
    """32 entry nodes, more than the shortest list holds, some of them named twice, no nodes, or with a NaN score."""
    say(f"frontier, entries and NaN rows: ef={ef}")
    x, q, g = _random(4000, 96, 12, 4, torch.float16, ef)
    x[::7, 3] = float("nan")
    gen = torch.Generator().manual_seed(ef)
    e = torch.randint(0, 4000, (4, 32), generator=gen, dtype=torch.int32)
    e[0, 3], e[1, 5], e[2, 6], e[3, :30] = e[0, 9], -4, 4000, 7
    ids, sc = ann.ann_graph_search_multi_typed(x.to(DEV), g.to(DEV), e.to(DEV), q.to(DEV), 10, ef)
    torch.cuda.synchronize()
    o_ids, _, _, n_dist, n_expand = oracle.graph_search(to_np(x), g.numpy(), 0, to_np(q), 10, ef, entries=e.numpy())
    assert np.array_equal(ids.cpu().numpy(), o_ids)
    ids, _, stats, _ = ann.ann_graph_search_nonstall_typed(x.to(DEV), g.to(DEV), 0, q.to(DEV), 10, ef, entries=e.to(DEV), tau=0.999,
                                                           window=10, engine_ready=torch.zeros(1, dtype=torch.int32, device=DEV))
    torch.cuda.synchronize()
    st = stats.cpu().numpy()
    assert np.array_equal(ids.cpu().numpy(), o_ids) and np.array_equal(st[:, 1], n_dist) and np.array_equal(st[:, 2], n_expand)


@pytest.mark.parametrize("N,ef,k", [(1_247_200, 256, 7), (1_246_000, 130, 130), (1_240_000, 256, 70)])
def test_graph_frontier_in_all_of_lds(N, ef, k):
    """The largest graphs whose visited set fits LDS beside the array, in a buffer that holds none: the array has its fewest
    places, so that a bound is found in every other step (the first two: none for the queue's end either)."""
    say(f"frontier, no workspace: N={N} ef={ef} k={k}")
    x, q, g = _random(N, 8, 16, 8, torch.float16, ef)
    buf = torch.full((4096,), 0xAB, dtype=torch.uint8, device=DEV)
    try:
        ann.ann_set_workspace(buf[:256])
        ids, _, stats, _ = ann.ann_graph_search_nonstall_typed(x.to(DEV), g.to(DEV), 3, q.to(DEV), k, ef, tau=0.999, window=2_000_000_000)
        torch.cuda.synchronize()
    finally:
        ann.ann_set_workspace(None)
    assert bool((buf == 0xAB).all())
    o_ids, _, _, n_dist, n_expand = oracle.graph_search(to_np(x), g.numpy(), 3, to_np(q), k, ef)
    st = stats.cpu().numpy()
    # (rows of 8 numbers: scores of the two sides differ by about 1e-7, and nodes that close change places)
    same = (st[:, 1] == n_dist) & (st[:, 2] == n_expand)
    assert same.mean() >= 0.75 and (ids.cpu().numpy() == o_ids).mean() >= 0.9 and (st[:, 0] == 0).all()


@pytest.mark.parametrize("N,R,B,ef", [
    (4000, 32, 3, 100),      # eight waves, four expansions a step
    (4000, 32, 3, 128),      # ... eight expansions
    (4000, 32, 300, 128),    # four waves: more unknown neighbours than row groups
    (4000, 24, 600, 128),    # ... three workgroups a compute unit
])
def test_graph_frontier_shared_neighbours(N, R, B, ef):
    """Rows that name the same few nodes again and again, within a row and from row to row of a step, some scored by the step before."""
    say(f"shared neighbours: N={N} R={R} B={B} ef={ef}")
    x, q, _ = _random(N, 96, R, B, torch.float16, 21)
    gen = torch.Generator().manual_seed(22)
    g = (torch.arange(N)[:, None] // 20 * 20 + torch.randint(-20, 60, (N, R), generator=gen)).to(torch.int32)
    xn, qn = to_np(x), to_np(q)
    ids, sc, stats, _ = ann.ann_graph_search_nonstall_typed(x.to(DEV), g.to(DEV), 3, q.to(DEV), 10, ef, tau=float("inf"), window=10)
    p_ids, p_sc = ann.ann_graph_search_typed(x.to(DEV), g.to(DEV), 3, q.to(DEV), 10, ef)
    torch.cuda.synchronize()
    o_ids, _, o_sc64, n_dist, n_expand = oracle.graph_search(xn, g.numpy(), 3, qn, 10, ef, dtype="f16")
    strict, tolerant, n = compare_topk(ids.cpu().numpy(), sc.cpu().numpy(), o_ids, o_sc64, xn, qn, dtype="f16")
    assert strict >= n - max(2, n // 100), (strict, n)
    assert torch.equal(ids, p_ids) and torch.equal(sc, p_sc)
    st = stats.cpu().numpy()
    assert ((st[:, 1] == n_dist) & (st[:, 2] == n_expand)).mean() >= 0.99
