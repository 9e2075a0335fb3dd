"""The exact search of few queries against few rows, at the edges of its tiles of 16 rows x 16 queries and of its runs of steps."""
import pytest
import torch

import paper_2505_12065_amd as ann

pytestmark = pytest.mark.gpu
DEV = "cuda"
F16, BF16, F32 = torch.float16, torch.bfloat16, torch.float32


@pytest.mark.parametrize("dtype,N,d,B,k", [
    (F16, 1, 1_000, 1, 1),                 # one launch: one row
    (BF16, 17, 104, 17, 16),               # ... a row and a query in a second tile, a step of 16 bytes
    (F16, 64, 456, 33, 7),                 # ... whole tiles
    (F16, 113, 264, 5, 16),                # ... the last wave has one row
    (F32, 128, 132, 16, 10),               # the streaming kernel's one slab: fp32, a row that ends inside a run, all waves full
    (F32, 128, 96, 16, 10),                # one launch: all waves full
    (F32, 20, 1_092, 40, 5),               # ... more steps than are in flight at once
    (F32, 4, 4_096, 3, 4),                 # one slab: whole runs of long rows
    (F32, 4, 4_092, 3, 4),                 # one launch: queries longer than the LDS holds
    (F16, 16, 1_040, 300, 3),              # ... many queries
    (F16, 128, 240, 2, 3),                 # ... all waves full, 60 KB
    (F16, 100, 1_024, 2, 16),              # scores: up to 128 rows
    (F16, 129, 8, 1, 16),                  # ... one chunk of a step
    (BF16, 1_999, 776, 16, 16),            # ... a run cut after its first chunk, scores not a multiple of 4
    (F16, 2_048, 768, 17, 10),             # ... all steps in flight
    (F16, 2_049, 1_544, 3, 1),             # ... a run of its own behind twice as many, the last tile of one row
    (F32, 10_000, 132, 16, 10),            # ... more scores than a wave picks from
    (F32, 700, 2_052, 9, 4),
    (F16, 21_025, 480, 14, 2),             # ... near the line
])
def test_few_queries_few_rows(dtype, N, d, B, k):
    """Two pages against scores in binary64.  Every product is rounded together with its sum, so a score is off by at most
    d 2^-24 sum |x_i q_i| <= d 2^-24 |x| |q|, and the r-th best differs by no more than the largest of those."""
    print(f"few rows: dtype={dtype} N={N} d={d} B={B} k={k}", flush=True)
    gen = torch.Generator(device=DEV).manual_seed(N + d)
    x = torch.randn(N, d, generator=gen, device=DEV).to(dtype)
    q = torch.randn(B, d, generator=gen, device=DEV).to(dtype)
    x[5::7, d - 1] = float("nan")                                        # never listed
    exact = q.double() @ x.double().T
    bound = d * 2.0 ** -24 * q.double().norm(dim=1, keepdim=True) * x.double().norm(dim=1).nan_to_num().max()
    exact = exact.nan_to_num(nan=float("-inf"))
    first = ann.ann_flat_search_typed(x, q, k)
    second = ann.ann_flat_search_typed(x, q, k, after=(first[1][:, -1].contiguous(), first[0][:, -1].contiguous()))
    ids, sc = torch.cat([first[0], second[0]], 1).long(), torch.cat([first[1], second[1]], 1).double()
    n = min(2 * k, N - len(range(5, N, 7)))
    if n <= k:                                                           # (the first page ends in padding, which excludes every row)
        ids, sc = ids[:, :k], sc[:, :k]
        n = min(k, n)
    assert (ids[:, n:] == -1).all() and (ids[:, :n] >= 0).all()
    ids, sc = ids[:, :n], sc[:, :n]
    assert ((exact.gather(1, ids) - sc).abs() <= bound).all()
    assert ((exact.topk(n).values - sc).abs() <= bound).all()
    assert (ids.sort(1).values.diff(dim=1) > 0).all()                    # no row twice
    order = sc.diff(dim=1)
    assert ((order < 0) | ((order == 0) & (ids.diff(dim=1) > 0))).all()


@pytest.mark.parametrize("N,d,B", [(100, 200, 20), (2_000, 200, 20)])
def test_infinities_at_the_end_of_a_row(N, d, B):
    """What a run reads again behind the end of a row or a query takes no part: infinite last elements give infinite scores, not NaN."""
    gen = torch.Generator(device=DEV).manual_seed(N)
    x = torch.rand(N, d, generator=gen, device=DEV).half() + 0.5
    q = torch.rand(B, d, generator=gen, device=DEV).half() + 0.5
    x[7::11, d - 3] = float("inf")
    q[1::3, d - 1] = float("inf")
    ids, sc = ann.ann_flat_search_typed(x, q, 8)
    assert torch.isinf(sc).all() and (sc > 0).all()
    assert (ids[1::3].long() == torch.arange(8, device=DEV)).all()       # every row ties
    assert (ids[0].long() == torch.arange(8, device=DEV) * 11 + 7).all()


def test_scores_that_tie():
    """Thousands of equal scores: the lowest ids, in order, page after page."""
    x = torch.ones(4_000, 64, device=DEV, dtype=BF16)
    q = torch.ones(3, 64, device=DEV, dtype=BF16)
    after = None
    for page in range(3):
        ids, sc = ann.ann_flat_search_typed(x, q, 16, after=after)
        assert (ids == torch.arange(16, device=DEV) + 16 * page).all() and (sc == 64).all()
        after = (sc[:, -1].contiguous(), ids[:, -1].contiguous())


@pytest.mark.parametrize("dtype,N,d,B,k", [(F16, 128, 768, 64, 4), (BF16, 64, 2_048, 33, 16), (F32, 100, 512, 40, 10), (F16, 80, 768, 512, 1)])
def test_few_rows_on_two_streams_at_once(dtype, N, d, B, k):
    """Searches that need no workspace overlap: two corpora, a stream each, nothing between them."""
    print(f"two streams: dtype={dtype} N={N} d={d} B={B} k={k}", flush=True)
    gen = torch.Generator(device=DEV).manual_seed(d)
    x = [torch.randn(N, d, generator=gen, device=DEV).to(dtype) for _ in range(2)]
    q = [torch.randn(B, d, generator=gen, device=DEV).to(dtype) for _ in range(2)]
    assert ann.ann_flat_workspace_bytes(N, d, dtype, B, k) == 0
    alone = [ann.ann_flat_search_typed(x[i], q[i], k) for i in range(2)]
    streams = [torch.cuda.Stream() for _ in range(2)]
    torch.cuda.synchronize()
    out = [[], []]
    for _ in range(50):
        for i in range(2):
            with torch.cuda.stream(streams[i]):
                out[i].append(ann.ann_flat_search_typed(x[i], q[i], k))
    torch.cuda.synchronize()
    for i in range(2):
        assert all(torch.equal(ids, alone[i][0]) and torch.equal(sc, alone[i][1]) for ids, sc in out[i])


@pytest.mark.parametrize("dtype,N,d,B,k", [(F32, 10_000, 132, 16, 10), (F32, 700, 2_052, 9, 4), (F16, 21_025, 480, 14, 2)])
def test_scores_are_the_streaming_kernels_bits(dtype, N, d, B, k):
    """In a buffer that does not hold the scores the same call goes by lists: the same ids and the same bits, page after page."""
    print(f"bits: dtype={dtype} N={N} d={d} B={B} k={k}", flush=True)
    gen = torch.Generator(device=DEV).manual_seed(N)
    x, q = (torch.randn(n, d, generator=gen, device=DEV).to(dtype) for n in (N, B))
    size = ann.ann_flat_workspace_bytes(N, d, dtype, B, k) - 16
    buf = torch.empty(size, dtype=torch.uint8, device=DEV)
    pages = []
    try:
        for given in (None, buf):
            torch.cuda.synchronize()
            ann.ann_set_workspace(given)
            first = ann.ann_flat_search_typed(x, q, k)
            after = (first[1][:, -1].contiguous(), first[0][:, -1].contiguous())
            pages.append([*first, *ann.ann_flat_search_typed(x, q, k, after=after)])
            torch.cuda.synchronize()
    finally:
        ann.ann_set_workspace(None)
    assert all(torch.equal(a, b) for a, b in zip(*pages))
