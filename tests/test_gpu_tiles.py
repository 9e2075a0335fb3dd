"""The tiles of the matrix-core kernel whose stages hold whole lines of 128 bytes, at their edges."""
import pytest
import torch

import paper_2505_12065_amd as ann

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.mark.parametrize("dtype,N,d,B,k", [
    (torch.float16, 48_897, 40, 100, 3),       # 256 x 128: a stage that the row ends in, one row in the last tile
    (torch.bfloat16, 49_408, 64, 128, 16),     # ... one whole stage, whole tiles
    (torch.float16, 16_001, 200, 400, 5),      # ... four query tiles, rows end after a quarter of a line
    (torch.bfloat16, 4_000, 136, 2_000, 2),    # ... groups of 16
    (torch.bfloat16, 4_000, 520, 2_000, 16),   # ... single rows
    (torch.float16, 4_001, 104, 999, 5),       # 128 x 64: one row in the last tile
    (torch.float16, 4_001, 264, 999, 16),      # ... single rows
    (torch.bfloat16, 700, 264, 3_000, 16),     # ... the corpus is the smaller operand: workgroups by query tile
    (torch.float16, 130_000, 72, 33, 1),       # ... groups of rows, slabs of tiles
    (torch.float16, 1, 8, 65, 1),              # 64 x 64: one row
    (torch.bfloat16, 63, 1_000, 129, 10),      # ... a tile short of one row
    (torch.float16, 1_000, 776, 65, 4),        # ... a line of 16 bytes at the end of a row
    (torch.float16, 2_049, 96, 5_000, 4),      # 256 x 256, by query tile: groups of 4
    (torch.float16, 2_049, 520, 5_000, 16),    # ... single rows
    (torch.bfloat16, 4_000, 768, 1, 3),        # up to 64 queries by these tiles: few long rows
    (torch.float16, 16_384, 384, 32, 1),       # ... one tile for each compute unit
    (torch.float16, 20_001, 768, 17, 16),      # ... up to 32 Ki rows
    (torch.bfloat16, 33_000, 1_544, 33, 4),    # ... rows of three groups of queries that do not fit LDS
    (torch.float16, 70_001, 64, 1, 10),        # ... short rows
    (torch.bfloat16, 131_072, 96, 16, 16),     # ...
    (torch.float16, 131_073, 8, 3, 4),         # 128 x 64 of half lines: a quarter of a stage, one row in the last tile
    (torch.bfloat16, 40_000, 24, 100, 16),     # ... two query tiles
    (torch.float16, 98_303, 200, 64, 16),      # ... 768 tiles, rows that end in a stage
    (torch.bfloat16, 700, 24, 3_000, 16),      # ... single rows, the corpus the smaller operand
    (torch.bfloat16, 60_000, 1_160, 300, 9),   # rows scored once more: three long runs of steps and a last one of half a step
    (torch.float32, 40_000, 392, 400, 3),      # ... fp32, one long run and half a step
    (torch.float16, 3_000, 776, 1_025, 9),     # ... more queries than long runs pay for
    (torch.float16, 3_000, 1_160, 1_025, 9),   # ... for rows of up to 71 steps
    (torch.bfloat16, 30_000, 376, 100, 16),    # ... a step and a half less than a long run
])
def test_line_stages(dtype, N, d, B, k):
    """Two pages against scores in binary64.  Every product is rounded together with its sum, so a score is off by at most
    d 2^-24 sum |x_i q_i| <= d 2^-24 |x| |q|, and the r-th best differs by no more than the largest of those."""
    print(f"line stages: dtype={dtype} N={N} d={d} B={B} k={k}", flush=True)
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
    assert (ids[:, n:] == -1).all() and (ids[:, :n] >= 0).all()
    ids, sc = ids[:, :n], sc[:, :n]
    assert ((exact.gather(1, ids) - sc).abs() <= bound).all()
    assert ((exact.topk(n).values - sc).abs() <= bound).all()
    assert (ids.sort(1).values.diff(dim=1) > 0).all()                    # no row twice
    order = sc.diff(dim=1)
    assert ((order < 0) | ((order == 0) & (ids.diff(dim=1) > 0))).all()


@pytest.mark.parametrize("dtype,N,d,B,k", [
    (torch.float16, 977, 776, 5_000, 16),      # single rows, workgroups by query tile, a line of 16 bytes at the end of a row
    (torch.bfloat16, 1_025, 72, 4_097, 16),    # ... one row, one query in the last tiles
    (torch.float16, 24_001, 264, 200, 3),      # groups of rows, one row in the last tile
    (torch.bfloat16, 38_784, 96, 68, 10),      # ... whole tiles of rows, one query tile half empty
    (torch.bfloat16, 1_025, 72, 5_000, 16),    # ... a line of 16 bytes behind one (B = 4097 goes by half lines, as does d = 96)
    (torch.float16, 50_049, 136, 66, 10),      # ... two queries in the tile
    (torch.float16, 46_408, 384, 883, 5),      # ... slabs of several tiles
])
def test_square_tiles(dtype, N, d, B, k):
    """128 x 128 with two stages."""
    test_line_stages(dtype, N, d, B, k)


@pytest.mark.parametrize("dtype,N,d,B,k", [
    (torch.float16, 70_001, 264, 16, 3),       # up to 16 queries, batches of 3: a step of 16 bytes, one row in the last tile
    (torch.bfloat16, 70_001, 1_000, 3, 10),    # ... of 33 steps, one more than there are
    (torch.float16, 140_003, 160, 5, 4),       # ... of 5, half lines
    (torch.bfloat16, 140_003, 136, 7, 16),     # ... a step of 16 bytes
    (torch.float16, 200_001, 776, 40, 10),     # more queries, batches of 5: eight waves
    (torch.bfloat16, 200_001, 776, 64, 3),     # ... 16 waves
    (torch.float16, 200_000, 456, 17, 16),     # ... two groups of queries
    (torch.float16, 1_000_001, 264, 33, 3),    # ... of 3
    (torch.bfloat16, 70_001, 768, 40, 4),      # ... of 2, whole rows
    (torch.float16, 150_000, 1_024, 64, 10),   # ... 16 waves
    (torch.bfloat16, 600_001, 192, 17, 5),     # ... two groups, large corpora
    (torch.float32, 60_001, 80, 9, 4),         # fp32, of 2: half a batch at the end
    (torch.float32, 50_000, 96, 16, 10),       # ... whole rows
    (torch.float32, 40_001, 2_400, 3, 1),      # ... queries longer than the LDS holds
])
def test_batches_of_the_streaming_kernel(dtype, N, d, B, k):
    test_line_stages(dtype, N, d, B, k)


@pytest.mark.parametrize("dtype,N,d,B,k,offset", [
    (torch.float16, 83_001, 776, 77, 10, 0),   # 256 x 128, as many lines as steps
    (torch.bfloat16, 134_401, 1_000, 66, 16, 7),   # ... a line more, one row in the last tile
    (torch.bfloat16, 680_000, 200, 70, 3, 1),  # ... in the place of 512 x 128; four lines
    (torch.float16, 135_424, 992, 128, 3, 4),  # ... half lines, whole tiles
    (torch.float16, 330_001, 200, 40, 4, 3),   # 128 x 64
    (torch.bfloat16, 480_000, 136, 17, 16, 0),     # ... the shortest rows: a step of one chunk behind two
    (torch.float16, 300_000, 264, 40, 1, 6),
])
def test_stages_of_lines_of_memory(dtype, N, d, B, k, offset):
    """Rows that begin anywhere in a line (offset: 16-byte chunks) against the same search in pieces small enough to go by the rows' own
    stages, two pages of each: same bits.  A NaN or an infinity at either end of a row stays its own."""
    print(f"lines of memory: dtype={dtype} N={N} d={d} B={B} k={k} offset={offset}", flush=True)
    gen = torch.Generator(device=DEV).manual_seed(N + d)
    x = torch.randn(N * d + 64, generator=gen, device=DEV).to(dtype)[8 * offset:8 * offset + N * d].view(N, d)
    q = torch.randn(B, d, generator=gen, device=DEV).to(dtype)
    x[3::11, 0] = float("nan")
    x[5::7, d - 1] = float("nan")
    x[100::20_011, 0] = float("inf")
    x[101::30_011, d - 1] = float("-inf")
    got = two_pages(x, q, k)
    step = 60_000_000 // (2 * d)
    ids, sc = [], []
    for r0 in range(0, N, step):
        i, s = two_pages(x[r0:r0 + step], q, k)
        ids.append(i + r0)
        sc.append(s)
    ids, sc = torch.cat(ids, 1), torch.cat(sc, 1)
    best = sc.sort(dim=1, descending=True, stable=True).indices[:, :2 * k]      # (pieces and their rows come in the order of the ids)
    assert torch.equal(got[0], ids.gather(1, best)) and torch.equal(got[1], sc.gather(1, best))


def two_pages(x, q, k):
    first = ann.ann_flat_search_typed(x, q, k)
    second = ann.ann_flat_search_typed(x, q, k, after=(first[1][:, -1].contiguous(), first[0][:, -1].contiguous()))
    return torch.cat([first[0], second[0]], 1), torch.cat([first[1], second[1]], 1)


@pytest.mark.parametrize("dtype,N,d,B,k,size", [
    (torch.float16, 62_553, 2_056, 33, 9, 140_257),    # 128 x 64, two parts by lines and a short one by rows
    (torch.bfloat16, 42_905, 3_856, 24, 7, 54_955),
])
def test_parts_of_lines_of_memory(dtype, N, d, B, k, size):
    """Two pages in a caller's buffer that holds the maxima of a part of the corpus only, against the same in the library's."""
    print(f"lines of memory in parts: dtype={dtype} N={N} d={d} B={B} k={k} bytes={size}", flush=True)
    gen = torch.Generator(device=DEV).manual_seed(N + d)
    x = torch.randn(N, d, generator=gen, device=DEV).to(dtype)
    q = torch.randn(B, d, generator=gen, device=DEV).to(dtype)
    want = two_pages(x, q, k)
    buf = torch.empty(size, dtype=torch.uint8, device=DEV)
    try:
        ann.ann_set_workspace(buf)
        got = two_pages(x, q, k)
        torch.cuda.synchronize()
    finally:
        ann.ann_set_workspace(None)
    assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])


@pytest.mark.parametrize("N,d,B,k,size", [
    (15_656, 512, 1, 1, 1_163),                # maxima do not fit, lists do
    (85_001, 144, 10, 10, 9_789),              # lists do not fit, the corpus in parts does
])
def test_other_kernel_where_the_workspace_is_short(N, d, B, k, size):
    """In a caller's buffer and, captured, in a library buffer that cannot grow: the answer of the call that has the room."""
    gen = torch.Generator(device=DEV).manual_seed(N)
    x, q = (torch.randn(n, d, generator=gen, device=DEV).half() for n in (N, B))
    assert ann.ann_flat_workspace_bytes(N, d, torch.float16, B, k) > size
    want = ann.ann_flat_search_typed(x, q, k)
    ids, sc = torch.empty_like(want[0]), torch.empty_like(want[1])
    buf = torch.full((size + 4096,), 0xAB, dtype=torch.uint8, device=DEV)    # (the library keeps its address only)
    torch.cuda.synchronize()
    try:
        ann.ann_set_workspace(buf[:size])
        got = ann.ann_flat_search_typed(x, q, k)
        torch.cuda.synchronize()
    finally:
        ann.ann_set_workspace(None)
    assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])
    assert bool((buf[size:] == 0xAB).all()) and bool((buf[:size] != 0xAB).any())
    ann.ann_release_workspace()
    few = ann.ann_flat_search_typed(x[:1_000], q, k)                         # (the buffer has room for this and stays)
    assert 2 * ann.ann_flat_workspace_bytes(1_000, d, torch.float16, B, k) < ann.ann_flat_workspace_bytes(N, d, torch.float16, B, k)
    g = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(g):
        ann.ann_flat_search_typed(x, q, k, ids=ids, scores=sc)
    for _ in range(3):
        ids.fill_(-7)
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(ids, want[0]) and torch.equal(sc, want[1])
        again = ann.ann_flat_search_typed(x[:1_000], q, k)
        torch.cuda.synchronize()
        assert torch.equal(again[0], few[0]) and torch.equal(again[1], few[1])


@pytest.mark.parametrize("N,d,B,k,size", [
    (100_000, 256, 32, 3, 1 << 17),            # all slabs but a few
    (73_541, 128, 25, 10, 204_400),            # k > 4, a third of the slabs
])
def test_one_pass_on_lists_where_parts_take_longer(N, d, B, k, size):
    """Two pages in a caller's buffer that the matrix-core kernel's parts would fit as well, against scores in binary64 (bound: see
    test_line_stages); nothing behind the buffer is written."""
    print(f"lists in a small buffer: N={N} d={d} B={B} k={k} bytes={size}", flush=True)
    gen = torch.Generator(device=DEV).manual_seed(N)
    x, q = (torch.randn(n, d, generator=gen, device=DEV).half() for n in (N, B))
    assert ann.ann_flat_workspace_bytes(N, d, torch.float16, B, k) > size
    buf = torch.full((size + 4096,), 0xAB, dtype=torch.uint8, device=DEV)
    try:
        ann.ann_set_workspace(buf[:size])
        first = ann.ann_flat_search_typed(x, q, k)
        second = ann.ann_flat_search_typed(x, q, k, after=(first[1][:, -1].contiguous(), first[0][:, -1].contiguous()))
        torch.cuda.synchronize()
    finally:
        ann.ann_set_workspace(None)
    assert bool((buf[size:] == 0xAB).all())
    ids, sc = torch.cat([first[0], second[0]], 1).long(), torch.cat([first[1], second[1]], 1).double()
    exact = q.double() @ x.double().T
    bound = d * 2.0 ** -24 * q.double().norm(dim=1, keepdim=True) * x.double().norm(dim=1).max()
    assert ((exact.gather(1, ids) - sc).abs() <= bound).all() and ((exact.topk(2 * k).values - sc).abs() <= bound).all()
    assert (ids.sort(1).values.diff(dim=1) > 0).all()
