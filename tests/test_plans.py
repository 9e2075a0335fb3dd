"""What a call would launch, decided without a GPU: the host rules of plan.hpp, compiled with the C++ compiler alone.

The rules choose between ways of giving the same answer, so a wrong one costs time and no test of results sees it."""
import ctypes
import math
import os
import random
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CUS = 256

SHIM = r"""
#include "plan.hpp"
using namespace ann;
// 0 graph_search_kernel, 1 graph_frontier_kernel, 2 graph_step_kernel (all workspace at hand)
extern "C" int graph_kernel(int cus, int64_t N, int row_bytes, int R, int B, int ef, int counters, float tau) {
    const bool leaves = counters && exit_likely(tau, 2.0f / 501, R, ef);                  // (a window of 500)
    const FrontierLds L = frontier_plan(cus, N, row_bytes / 2, 2, B, ef, counters && tau < 1);
    if (frontier_pays(cus, N, row_bytes, R, B, ef, counters != 0, leaves, L)) return 1;
    return !counters && graph_step_pays(cus, N, row_bytes, R, B, ef) ? 2 : 0;
}
extern "C" int leaves(float tau, int window, int R, int ef) { return exit_likely(tau, 2.0f / ((float)window + 1.0f), R, ef); }
// tight: frontier_in_lds's layout instead of the call's; out: fits, waves, workgroups per compute unit, expansions a step tries, tight,
// visited set in LDS, its words, the query's, visited set's and array's places, places of the array, those a bound may leave, LDS bytes
extern "C" void frontier(int cus, int64_t N, int row_bytes, int B, int ef, int counters, float tau, int in_lds, int64_t *out) {
    FrontierLds L;
    bool fits = true;
    if (in_lds) fits = frontier_in_lds(N, row_bytes / 2, 2, 32, ef, counters != 0, L);
    else L = frontier_plan(cus, N, row_bytes / 2, 2, B, ef, counters && tau < 1);
    const int64_t v[] = {fits, L.waves, L.per_cu, L.width, L.tight, L.vis_mode == FRONTIER_VIS_LDS, L.vis_words, L.q, L.vis, L.keys, L.cap,
                         L.spare, L.total, (int64_t)FrontierLds::WAVES + L.waves * FrontierLds::WAVE_BYTES};
    for (int i = 0; i < 14; ++i) out[i] = v[i];
}
extern "C" int in_lds(int64_t N, int d, int elem_bytes, int R, int ef) {
    FrontierLds L;
    return frontier_in_lds(N, d, elem_bytes, R, ef, true, L);
}
extern "C" int ahead(int waves) { return frontier_ahead(waves); }
extern "C" int runs(int cus, int d, int elem_bytes, int B) { return pick_runs(cus, (size_t)d * elem_bytes, 16 * elem_bytes, B); }
extern "C" int shape(int cus, int64_t N, int d, int B) { return wide_shape(cus, N, d, B); }
extern "C" int batch(int cus, int64_t N, int d, int dtype, int B, int k) {
    const FlatPlan pl = flat_plan(cus, N, d, dtype, B, k, WIDE_WS_MAX);
    return pl.wide || pl.scores || pl.quick ? 0 : pl.st.batch;
}
extern "C" int by_line(int64_t N, int d, int col_tiles) { return wide_by_line(N, d, col_tiles); }
extern "C" int tile(int cus, int64_t N, int d, int B, int k) { return wide_tile(cus, N, d, B, k); }
static int kind(const FlatPlan &pl) { return pl.scores ? 4 : pl.quick ? 5 : pl.wide ? 2 : pl.maxima ? 3 : pl.direct ? 1 : 0; }
// out: kind (0 lists, 1 direct, 2 matrix cores, 3 streaming with maxima, 4 scores, 5 direct by flat_direct_kernel), queries and rows at a time, maxima of a query,
// log2 of the rows they stand for, offset of the k best so far, workspace, maxima of the smallest last part and the rows they stand for, tile;
// by_fill: by the first rule for the tile alone
static void describe(const FlatPlan &pl, int64_t N, int d, int dtype, int B, int64_t *out) {
    const int64_t rows = N % pl.rows ? N % pl.rows : pl.rows;
    const int part = B % pl.part ? B % pl.part : pl.part;
    const FlatPlan last = pl.wide || pl.maxima ? maxima_part(pl, rows, part, d, dtype) : pl;
    const int64_t v[] = {kind(pl), pl.part, pl.rows, pl.w.n, pl.w.gs_log, (int64_t)pl.best_ofs, (int64_t)pl.ws_bytes, last.w.n, last.w.gs_log,
                         pl.w.shape};
    for (int i = 0; i < 10; ++i) out[i] = v[i];
}
extern "C" void flat(int cus, int64_t N, int d, int dtype, int B, int k, int64_t limit, int64_t *out) {
    describe(flat_plan(cus, N, d, dtype, B, k, (size_t)limit), N, d, dtype, B, out);
}
extern "C" void flat_by_fill(int cus, int64_t N, int d, int dtype, int B, int k, int64_t limit, int64_t *out) {
    describe(flat_plan(cus, N, d, dtype, B, k, (size_t)limit, false, true), N, d, dtype, B, out);
}
extern "C" int static_accepts(int cus, int64_t N, int d, int dtype, int B, int k, int64_t bytes) {
    return static_plan(cus, N, d, dtype, B, k, (size_t)bytes).ws_bytes <= (size_t)bytes;
}
extern "C" int static_kind(int cus, int64_t N, int d, int dtype, int B, int k, int64_t bytes) {
    const FlatPlan pl = static_plan(cus, N, d, dtype, B, k, (size_t)bytes);
    return pl.ws_bytes > (size_t)bytes ? -1 : kind(pl);
}
"""
KINDS = ("lists", "direct", "wide", "maxima", "scores", "quick")
STATIC = 8 * 1024 * 1024 + 1024 * 16 * 8             # the static workspace, room for the k best of a part's queries included


@pytest.fixture(scope="module")
def plans(tmp_path_factory):
    tmp = tmp_path_factory.mktemp("plans")
    src, lib = tmp / "shim.cpp", tmp / "shim.so"
    src.write_text(SHIM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-shared", "-fPIC", "-I",
                    os.path.join(ROOT, "paper_2505_12065_amd", "csrc"), "-o", str(lib), str(src)], check=True)
    L = ctypes.CDLL(str(lib))
    L.graph_kernel.argtypes = [ctypes.c_int, ctypes.c_int64] + [ctypes.c_int] * 5 + [ctypes.c_float]
    L.leaves.argtypes = [ctypes.c_float] + [ctypes.c_int] * 3
    L.frontier.argtypes = [ctypes.c_int, ctypes.c_int64] + [ctypes.c_int] * 4 + [ctypes.c_float, ctypes.c_int, ctypes.c_void_p]
    L.shape.argtypes = [ctypes.c_int, ctypes.c_int64] + [ctypes.c_int] * 2
    L.tile.argtypes = [ctypes.c_int, ctypes.c_int64] + [ctypes.c_int] * 3
    L.batch.argtypes = [ctypes.c_int, ctypes.c_int64] + [ctypes.c_int] * 4
    L.by_line.argtypes = [ctypes.c_int64] + [ctypes.c_int] * 2
    L.in_lds.argtypes = [ctypes.c_int64] + [ctypes.c_int] * 4
    L.flat.argtypes = L.flat_by_fill.argtypes = [ctypes.c_int, ctypes.c_int64] + [ctypes.c_int] * 4 + [ctypes.c_int64, ctypes.c_void_p]
    L.static_accepts.argtypes = L.static_kind.argtypes = [ctypes.c_int, ctypes.c_int64] + [ctypes.c_int] * 4 + [ctypes.c_int64]
    return L


def flat(L, N, d, dtype, B, k, limit, by_fill=False):
    out = (ctypes.c_int64 * 10)()
    (L.flat_by_fill if by_fill else L.flat)(CUS, N, d, dtype, B, k, limit, out)
    return dict(zip(("kind", "part", "rows", "n", "gs_log", "best_ofs", "bytes", "last_n", "last_gs_log", "shape"), out))


SEARCH, FRONTIER, STEP = 0, 1, 2
NEVER = float("inf")                                  # no average passes it


# us, or the ratio, of the others (graph_search_kernel, graph_step_kernel) / graph_frontier_kernel, or one by one / in steps
@pytest.mark.parametrize("N,row,R,B,ef,tau,kernel", [
    (200_000, 1536, 32, 256, 48, None, FRONTIER),         # 198 / 174
    (200_000, 1536, 32, 1, 768, None, FRONTIER),          # 1916 / 558
    (200_000, 1536, 32, 256, 3, None, SEARCH),            # 30.4 / 35.8
    (200_000, 4096, 32, 256, 16, None, SEARCH),           # 134 / 156
    (200_000, 1536, 32, 512, 48, None, SEARCH),           # 217 / 257
    (200_000, 1536, 32, 512, 384, None, FRONTIER),        # 1264 / 1041
    (200_000, 1536, 16, 512, 96, None, FRONTIER),         # 362 / 304
    (200_000, 1536, 24, 512, 64, None, SEARCH),           # 253 / 284
    (200_000, 1536, 32, 2048, 192, None, FRONTIER),       # 2074 / 1726
    (1_000_000, 1536, 32, 512, 64, None, SEARCH),         # the corpus of the benchmark
    (1_000_000, 1536, 32, 512, 600, None, SEARCH),        # 2215 / 2516
    (1_000_000, 1536, 32, 512, 2048, None, FRONTIER),     # 6959 / 6364
    (1_000_000, 1536, 32, 512, 8192, None, FRONTIER),     # 24.1 / 19.4 ms
    (1_000_000, 1536, 24, 512, 600, None, FRONTIER),      # 2086 / 1983
    (1_000_000, 1536, 32, 256, 8192, None, FRONTIER),     # 22 838 / 12 592
    (1_000_000, 1536, 32, 2048, 192, None, SEARCH),       # 0.77 one by one against steps: one list, more queries than places
    (1_000_000, 1536, 32, 1024, 512, None, SEARCH),       # 0.77
    (800_000, 1536, 32, 600, 512, None, STEP),            # 1.0 to 1.08
    (1_500_000, 1536, 16, 600, 256, None, STEP),          # 1.0 to 2.1
    (1_500_000, 1536, 32, 1, 512, None, STEP),            # 2.97
    (1_500_000, 1536, 32, 4, 512, None, SEARCH),
    (200_000, 1536, 40, 512, 512, None, SEARCH),          # wide graphs
    (200_000, 768, 32, 256, 32, 0.9, FRONTIER),           # 103 / 94
    (200_000, 768, 32, 256, 256, 0.9, FRONTIER),          # 326 / 249
    (200_000, 768, 16, 256, 32, 0.9, SEARCH),             # 106 / 128
    (200_000, 768, 16, 1024, 64, 0.9, FRONTIER),          # 354 / 291
    (120_000, 1024, 32, 1, 92, 0.9, SEARCH),              # 69 / 79: one query
    (200_000, 256, 16, 1, 124, 0.9, FRONTIER),            # 219 / 127
    (100_000, 1536, 32, 512, 32, 0.9, SEARCH),            # 105 / 112
    (100_000, 1536, 32, 512, 48, 0.9, FRONTIER),          # 144 / 126
    (100_000, 1536, 16, 512, 64, 0.9, SEARCH),            # 186 / 208
    (100_000, 1536, 16, 512, 96, 0.9, FRONTIER),          # 271 / 237
    (100_000, 1536, 8, 512, 64, 0.9, SEARCH),             # 223 / 233
    (100_000, 1536, 8, 1024, 96, 0.9, SEARCH),            # 560 / 618
    (40_000, 4096, 16, 512, 22, None, SEARCH),            # 164 / 186
    (40_000, 4096, 16, 512, 64, None, FRONTIER),          # 329 / 311
    (40_000, 4096, 32, 1024, 96, None, SEARCH),           # 1002 / 1137
    (60_000, 2304, 32, 1024, 128, None, FRONTIER),        # 0.93
    (200_000, 768, 32, 256, 64, NEVER, SEARCH),           # 318 / 319
    (200_000, 768, 32, 512, 256, NEVER, SEARCH),          # 1036 / 1137
    (200_000, 768, 32, 512, 512, NEVER, FRONTIER),        # 2032 / 1891
    (500_000, 256, 32, 64, 128, NEVER, SEARCH),           # 600 / 630
    (60_000, 768, 32, 8, 112, NEVER, FRONTIER),           # 0.98: the median of such calls
    (200_000, 1536, 32, 256, 80, NEVER, SEARCH),          # 1.05
    (200_000, 1536, 32, 256, 160, NEVER, FRONTIER),       # 0.97
    (400_000, 768, 16, 512, 160, NEVER, SEARCH),          # 1.08
    (1_000_000, 512, 16, 512, 300, NEVER, FRONTIER),      # 0.86
    (200_000, 512, 24, 512, 200, NEVER, SEARCH),          # 1.09
    (40_000, 4096, 24, 512, 300, NEVER, FRONTIER),        # 0.94
    (1_000_000, 512, 16, 700, 56, NEVER, FRONTIER),       # 0.88
    (200_000, 512, 32, 1024, 160, NEVER, SEARCH),         # 1.11
    (1_000_000, 512, 32, 512, 2048, NEVER, SEARCH),       # 7438 / 8428: visited sets in memory, two workgroups a compute unit
    (1_000_000, 512, 32, 1024, 1024, NEVER, FRONTIER),    # 7648 / 7185
    (40_000, 768, 32, 1024, 144, NEVER, FRONTIER),        # 0.92: the search covers more of a small graph
    (200_000, 256, 24, 1024, 128, NEVER, SEARCH),         # 857 / 918, 1.06
    (700_000, 256, 32, 1, 80, NEVER, FRONTIER),           # 0.60, 0.86, 0.61, 0.91: four queries
    (1_300_000, 128, 24, 16, 128, NEVER, SEARCH),         # 1.20
    (1_300_000, 128, 32, 64, 512, NEVER, FRONTIER),       # 0.90
    (400_000, 1536, 32, 512, 1024, NEVER, SEARCH),        # rows that come from memory
    (200_000, 1536, 32, 600, 384, NEVER, FRONTIER),       # 0.83
    (1_300_000, 128, 32, 1024, 192, NEVER, SEARCH),       # 1.26
    (1_300_000, 128, 32, 1990, 256, NEVER, FRONTIER),     # 0.94
    (400_000, 1536, 16, 1024, 256, NEVER, SEARCH),        # 1.23
    (400_000, 1536, 8, 1990, 128, NEVER, FRONTIER),       # 0.94
    (800_000, 1536, 24, 600, 700, NEVER, FRONTIER),       # 0.98
    (800_000, 1536, 32, 1024, 512, NEVER, SEARCH),        # 1.31
    (700_000, 256, 8, 600, 64, 0.9, FRONTIER),            # 0.79
    (800_000, 1536, 32, 1024, 128, 0.9, SEARCH),          # 1.04
    (800_000, 1536, 24, 1024, 192, 0.9, FRONTIER),        # 0.93
    # row groups without gaps
    (200_000, 1536, 32, 512, 96, None, SEARCH),           # 359 / 373
    (200_000, 1536, 32, 512, 128, None, FRONTIER),        # 442 / 432
    (200_000, 1536, 32, 700, 16, None, FRONTIER),         # 143 / 136
    (200_000, 1536, 32, 1024, 48, None, SEARCH),          # 373 / 378
    (100_000, 512, 32, 1024, 24, None, FRONTIER),         # 191 / 188
    (100_000, 512, 24, 300, 24, None, SEARCH),            # 103 / 111
    (100_000, 512, 24, 300, 48, None, FRONTIER),          # 187 / 180
    (50_000, 512, 31, 512, 64, None, FRONTIER),           # 190 / 179
    (60_000, 4096, 32, 700, 64, None, FRONTIER),          # 648 / 577
    (100_000, 768, 16, 300, 8, None, SEARCH),             # 52 / 59
])
def test_graph_kernels_where_they_were_measured_to_pay(plans, N, row, R, B, ef, tau, kernel):
    assert plans.graph_kernel(CUS, N, row, R, B, ef, tau is not None, NEVER if tau is None else tau) == kernel


# us of a call with adjacency rows touched ahead / without, 200 k x 768, R = 32, B = 256 and 512
@pytest.mark.parametrize("B,ef,ahead", [
    (256, 2048, True),           # 2121 / 2255: the last of eight waves seldom has a row to score
    (512, 512, False),           # 1110 / 1030: two workgroups of four keep the memory path busy with rows
    (512, 128, False)])          # 443 / 429
def test_adjacency_rows_touched_ahead_where_that_pays(plans, B, ef, ahead):
    out = (ctypes.c_int64 * 14)()
    plans.frontier(CUS, 200_000, 1536, B, ef, 0, NEVER, 0, out)
    assert bool(plans.ahead(int(out[1]))) == ahead


def test_steps_pay_up_to_a_size_of_the_graph(plans):
    """Lists of up to 512 entries without counters go from graph_frontier_kernel to steps to one by one as the graph grows, never back."""
    order = {FRONTIER: 0, STEP: 1, SEARCH: 2}
    for row in (128, 768, 1536, 4096):
        for R in (8, 24, 32):
            for B in (1, 4, 16, 256, 257, 512, 513, 800, 1024, 2048):
                for ef in (192, 320, 512):
                    got = [order[plans.graph_kernel(CUS, N, row, R, B, ef, 0, NEVER)] for N in
                           (400_000, 1_300_000, 4_000_000, 10_000_000, 100_000_000, 2**31 - 1)]
                    assert got == sorted(got), (row, R, B, ef, got)


@pytest.mark.parametrize("in_lds", [0, 1])
def test_frontier_layouts(plans, in_lds):
    """Whatever graph_frontier_kernel is launched with: regions one behind the other inside the share of the compute unit's LDS,
    a bit for every node, and room for what a step adds to a bound's leavings and for the queue's end (tight: not for that)."""
    rng = random.Random(in_lds)
    log = lambda lo, hi: int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    seen = set()
    out = (ctypes.c_int64 * 14)()
    for _ in range(60_000):
        N, row, B, ef = log(1, 2**31 - 1), 16 * log(1, 1024), log(1, 5000), log(1, 16_384)
        if rng.random() < 0.5:
            N = rng.randint(100_000, 1_260_000)
        counters, tau = rng.randint(0, 1), rng.choice([0.9, NEVER])
        plans.frontier(CUS, N, row, B, ef, counters, tau, in_lds, out)
        fits, waves, per_cu, width, tight, bits, words, q, vis, keys, cap, spare, total, scratch = out
        call = (N, row, B, ef, counters, tau, list(out))
        if not fits or (not in_lds and not plans.graph_kernel(CUS, N, row, 32, B, ef, counters, tau) == FRONTIER):
            continue
        assert (waves, per_cu) in ((8, 1), (4, 1), (4, 2), (4, 3)) and width in (4, 8), call
        assert total <= 160 * 1024 // per_cu and scratch <= q and q + row <= vis and vis + 4 * words <= keys and keys + 8 * cap <= total, call
        assert not any(x % 16 for x in (q, vis, keys, total)), call
        assert 32 * words >= N if bits else words == 0 and not in_lds, call
        assert spare >= 0 and ef + spare + 64 + width + (0 if tight else 64) <= cap, call
        assert not tight or (in_lds and counters), call
        seen.add((waves, per_cu, width, tight, bits))
    assert len(seen) >= (2 if in_lds else 7), seen


@pytest.mark.parametrize("N,d,dtype,B,k", [
    (1_000_000, 768, 0, 256, 3), (1_000_000, 768, 0, 512, 3), (21_000_000, 768, 0, 256, 3), (21_000_000, 384, 0, 512, 3),
    (21_000_000, 384, 0, 128, 3), (21_000_000, 384, 1, 66, 16), (4_000_000, 64, 2, 100, 3)])
def test_little_workspace_takes_the_corpus_in_parts(plans, N, d, dtype, B, k):
    """Group maxima that do not fit: every query of the batch against one part of the corpus after the other (the
    products of a few queries against the whole corpus, again and again, took up to 50 times as long)."""
    p = flat(plans, N, d, dtype, B, k, STATIC)
    assert KINDS[p["kind"]] in ("wide", "maxima") and p["bytes"] <= STATIC
    assert p["part"] == B
    cells = 64 * 8 * 1024 * 1024 // 4                # scores whose maxima, one of 64 rows, fill the workspace
    assert -(-N // p["rows"]) <= N * B // cells + 2


@pytest.mark.parametrize("limit", [64 * 1024, 1 << 20, STATIC, 1 << 26, 1 << 30])
def test_parts_stay_inside_the_workspace(plans, limit):
    """Over the sizes the entry points take: the maxima of a part and what stands behind them fit, the last part needs no
    more than the others and uses their groups, and every row has a maximum."""
    rng = random.Random(limit)
    log = lambda lo, hi: int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    kinds = set()
    for _ in range(4000):
        dtype = rng.choice([0, 1, 2])
        step = 4 if dtype == 2 else 8
        N, d, B, k = log(1, 2**31 - 1), step * log(1, 4096 // step), log(1, 100_000), rng.randint(1, 16)
        k = min(k, N)
        p = flat(plans, N, d, dtype, B, k, limit)
        if KINDS[p["kind"]] not in ("wide", "maxima") or p["bytes"] > limit:
            continue
        call = (N, d, dtype, B, k, p)
        kinds.add((p["kind"], p["part"] < B, p["rows"] < N))
        assert 1 <= p["part"] <= B and 1 <= p["rows"] <= N, call
        assert p["n"] % 4 == 0 and p["n"] << p["gs_log"] >= p["rows"], call
        assert p["last_gs_log"] == p["gs_log"] and p["last_n"] <= p["n"], call
        end = p["part"] * p["n"] * 4
        if p["rows"] < N:
            assert p["best_ofs"] >= end and p["best_ofs"] % 8 == 0, call
            end = p["best_ofs"] + p["part"] * k * 8
        assert end <= p["bytes"], call
    assert len(kinds) >= 3, kinds


# bytes: what the library asked for when it kept lists and candidate arrays, so buffers that callers have
@pytest.mark.parametrize("N,d,dtype,B,k,buffer", [
    (1_000_000, 768, 0, 512, 3, 4_212_736), (1_000_000, 768, 0, 65, 3, 1_194_180), (200_000, 768, 0, 100, 10, 6_186_400),
    (21_000_000, 384, 0, 512, 3, 4_212_736), (4092, 2128, 0, 1043, 15, 4_272_128), (459, 1488, 0, 4853, 12, 2_484_736),
    (2839, 40, 0, 743, 9, 2_187_392), (1_000_000, 128, 2, 256, 10, 33_554_432), (100_000, 768, 0, 16, 16, 401_408)])
def test_a_buffer_that_served_still_serves(plans, N, d, dtype, B, k, buffer):
    assert flat(plans, N, d, dtype, B, k, buffer)["bytes"] <= buffer


def test_a_buffer_of_the_size_that_is_asked_for_gives_the_same_plan(plans):
    rng = random.Random(11)
    log = lambda lo, hi: int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    for _ in range(4000):
        dtype = rng.choice([0, 1, 2])
        step = 4 if dtype == 2 else 8
        N, d, B = log(1, 3e7), step * log(1, 4096 // step), log(1, 5000)
        k = min(N, rng.randint(1, 16))
        whole = flat(plans, N, d, dtype, B, k, 1 << 30)
        if whole["part"] == B and whole["rows"] == N:                 # (not in parts in 1 GiB either)
            assert flat(plans, N, d, dtype, B, k, max(1, whole["bytes"])) == whole, (N, d, dtype, B, k)


def test_a_buffer_too_small_for_parts_is_refused(plans):
    for N, d, dtype, B, k in ((40_000, 256, 0, 96, 3), (1_000_000, 768, 0, 512, 3), (1_000_000, 768, 0, 16, 3)):
        assert flat(plans, N, d, dtype, B, k, 256)["bytes"] > 256


@pytest.mark.parametrize("N,d,dtype,B,k,accepted", [
    (2839, 40, 0, 743, 9, True), (459, 1488, 0, 4853, 12, True), (4092, 2128, 0, 1043, 15, True),
    (1_000_000, 768, 0, 512, 4, True), (21_000_000, 768, 1, 255, 16, True), (1000, 64, 2, 512, 10, True),
    (200_000, 64, 0, 2048, 10, False), (1_000_000, 768, 0, 512, 5, False), (1_000_000, 128, 2, 256, 10, False),
    (16_384, 40, 0, 512, 9, True), (127_999, 40, 0, 2048, 16, False)])
def test_what_the_static_workspace_takes(plans, N, d, dtype, B, k, accepted):
    assert bool(plans.static_accepts(CUS, N, d, dtype, B, k, STATIC)) == accepted


# us of a call, lists / matrix cores with all the room there is, where the two differ by a tenth
@pytest.mark.parametrize("N,d,B,k,kind", [
    (17_200_000, 232, 59, 5, "lists"),           # 1623 / 2185: in 8 MiB one pass, and not parts
    (21_000_000, 256, 64, 5, "lists"),           # 1841 / 2571
    (8_600_000, 200, 63, 12, "lists"),           # 800 / 1007
    (15_939_049, 120, 37, 1, "lists"),           # 841 / 1020
    (4_294_538, 248, 64, 3, "lists"),            # 451 / 570
    (6_634_886, 112, 62, 1, "wide"),             # 502 / 438
    (9_365_109, 72, 39, 1, "wide"),              # 516 / 413
    (14_313_870, 56, 31, 1, "wide"),             # 543 / 447
    (1_542_172, 112, 43, 1, "wide"),             # 127 / 92
    (1_545_228, 176, 56, 16, "wide"),            # 183 / 151
    (2_200_000, 256, 64, 3, "lists"),            # 226 / 264
    (4_000_000, 224, 60, 3, "lists"),            # 403 / 468
    (2_200_000, 192, 52, 3, "wide")])            # 234 / 203
def test_many_queries_on_large_corpora(plans, N, d, B, k, kind):
    """The same kernel with all the room and in the static workspace, so that both entry points give the same bits."""
    for limit in (1 << 30, STATIC):
        p = flat(plans, N, d, 0, B, k, limit)
        assert KINDS[p["kind"]] == kind and p["bytes"] <= limit
        assert kind == "wide" or (p["rows"] == N and p["part"] == B)


@pytest.mark.parametrize("N,d,B,kind", [                 # us, lists / maxima
    (66_376, 112, 2, "wide"),                             # 15.6 / 11.7
    (55_000, 192, 1, "wide"),                             # 17.4 / 13.7
    (97_000, 160, 14, "wide"),                            # 20.3 / 14.4
    (72_000, 240, 6, "wide"),                             # 19.3 / 16.6
    (100_000, 248, 2, "lists"),                           # 18.1 / 18.9
    (112_000, 256, 14, "lists"),                          # 18.2 / 19.2
    (211_000, 96, 6, "wide"),                             # 23.8 / 20.2
    (180_000, 224, 12, "lists"),                          # 25.5 / 26.5
    (454_000, 128, 14, "lists"),                          # 29.7 / 31.1
    (1_000_000, 96, 8, "lists"),                          # 48 / 57
])
def test_few_queries_against_the_length_of_rows(plans, N, d, B, kind):
    assert KINDS[flat(plans, N, d, 0, B, 3, 1 << 34)["kind"]] == kind


# us, lists / matrix cores
@pytest.mark.parametrize("N,d,B,k,kind", [
    (300_000, 96, 20, 3, "wide"),        # 28.5 / 21.3
    (300_000, 288, 32, 3, "lists"),      # 1 / 1.07
    (138_238, 464, 44, 5, "wide"),       # 44.8 / 35.1
    (163_627, 512, 60, 1, "wide"),       # 49.4 / 43.5
    (1_000_000, 128, 24, 3, "wide"),     # 64.7 / 59.8
    (1_000_000, 192, 32, 3, "lists"),    # 77.1 / 83.8
    (1_000_000, 256, 48, 3, "lists"),    # 110.6 / 117.2
    (1_000_000, 320, 64, 3, "wide"),     # 162 / 148
    (1_000_000, 384, 64, 3, "lists"),    # 163 / 171
    (949_486, 320, 53, 5, "lists"),      # 142 / 148
    (1_528_200, 256, 63, 16, "lists"),   # 179 / 192
    (3_000_000, 128, 32, 3, "lists"),    # 149 / 183
    (4_426_861, 88, 41, 5, "wide")])     # 289 / 221
def test_groups_of_queries_against_the_length_of_rows(plans, N, d, B, k, kind):
    """The same kernel in the static workspace, so that both entry points give the same bits."""
    assert KINDS[flat(plans, N, d, 0, B, k, 1 << 30)["kind"]] == kind
    assert KINDS[plans.static_kind(CUS, N, d, 0, B, k, STATIC)] == kind


# us, lists / matrix cores
@pytest.mark.parametrize("N,d,B,k,kind", [
    (3_322_254, 192, 59, 3, "wide"),     # 338 / 306
    (3_105_114, 192, 51, 16, "wide"),    # 323 / 293
    (16_756_363, 96, 54, 5, "wide"),     # 1036 / 919
    (207_230, 520, 45, 1, "wide"),       # 67.7 / 55.5
    (224_096, 608, 58, 5, "wide"),       # 78.2 / 68.2
    (1_030_004, 232, 45, 3, "lists"),    # 116 / 124
    (1_167_215, 256, 54, 16, "lists"),   # 141 / 148
    (1_500_000, 256, 64, 3, "lists"),    # 167 / 179
    (15_252_880, 128, 64, 1, "lists")])  # 789 / 1040
def test_a_row_and_settled_lists_against_elements(plans, N, d, B, k, kind):
    """Sizes that a line by a power of the rows and a cut at 1.25 Mi rows sent to the slower kernel, and some beside them."""
    assert KINDS[flat(plans, N, d, 0, B, k, 1 << 30)["kind"]] == kind
    assert KINDS[plans.static_kind(CUS, N, d, 0, B, k, STATIC)] == kind


@pytest.mark.parametrize("N,d,B,k", [(1_000_000, 320, 64, 3), (1_000_000, 224, 48, 3)])
def test_a_buffer_too_small_for_lists_is_refused(plans, N, d, B, k):
    """... where parts on the matrix cores would fit, but the line by queries leaves the call to lists; of a size that those need it is taken."""
    assert KINDS[flat(plans, N, d, 0, B, k, 1 << 30)["kind"]] == "wide"
    assert flat(plans, N, d, 0, B, k, 20_000)["bytes"] > 20_000
    p = flat(plans, N, d, 0, B, k, 600_000)
    assert KINDS[p["kind"]] == "lists" and p["rows"] == N


@pytest.mark.parametrize("N,d,B,k,buffer,slabs", [
    (156_898, 312, 17, 14, 217_662, 409), (138_557, 576, 50, 13, 565_586, 361), (195_451, 600, 54, 14, 766_163, 509)])
def test_a_buffer_too_small_for_lists_is_refused_where_maxima_would_fit(plans, N, d, B, k, buffer, slabs):
    """... at once: the line of what is refused is the one of lists, a quarter of their slabs, for both kernels."""
    asked = flat(plans, N, d, 0, B, k, 1 << 30)
    assert KINDS[asked["kind"]] == "wide" and flat(plans, N, d, 0, B, k, asked["bytes"])["bytes"] == asked["bytes"]
    assert flat(plans, N, d, 0, B, k, buffer)["bytes"] > buffer
    least = (slabs + 3) // 4 * B * 16 * 8                                # (lists of 16 pairs)
    assert buffer < least and flat(plans, N, d, 0, B, k, least)["bytes"] <= least
    assert flat(plans, N, d, 0, B, k, least - 1)["bytes"] > least - 1


# us, batches of 4 / this; 0: not the streaming kernel
@pytest.mark.parametrize("dtype,N,d,B,k,batch", [
    (0, 1_000_000, 264, 1, 3, 3),        # 109 / 101
    (0, 1_000_000, 136, 1, 3, 5),        # 62.5 / 57
    (0, 1_000_000, 104, 1, 3, 4),        # 48.3 / 55.7 by 3
    (0, 1_000_000, 224, 1, 3, 4),        # 84.4 / 86.2 by 3
    (0, 1_000_000, 768, 1, 3, 4),        # 253 / 260 by 3, 268 by 2
    (0, 1_000_000, 776, 48, 3, 5),       # 316 / 300
    (0, 1_000_000, 616, 48, 3, 5),       # 251 / 246
    (0, 1_000_000, 520, 48, 3, 4),       # 225 / 223 by 3
    (0, 21_000_000, 384, 64, 5, 2),      # 2706 / 2657
    (0, 3_000_000, 256, 64, 3, 4),       # 303 / 311 by 2
    (0, 1_000_000, 256, 32, 3, 2),       # 103 / 95.7
    (0, 3_600_000, 128, 18, 1, 4),       # 1 / 1.01 by 2 (1.6 M 86 / 91)
    (2, 1_000_000, 96, 4, 3, 2),         # 80.6 / 73.5
    (2, 1_000_000, 300, 4, 3, 4),        # 236 / 256 by 2
    (2, 200_000, 128, 5, 3, 2),          # 1 / 0.924
    (2, 131_004, 1_024, 4, 5, 4),        # 110 / 121 by 2
    (2, 3_165_301, 64, 13, 3, 4),        # 1 / 1.024 by 2
    (2, 250_000, 208, 4, 3, 2),          # 1 / 0.924
    (2, 2_935_657, 240, 6, 3, 4),        # 1 / 1.023 by 2
    (2, 561_370, 752, 10, 5, 4),         # 304 / 316 by 2
    (2, 400_000, 992, 3, 3, 2),          # 1 / 0.99
    (0, 128, 768, 64, 4, 4),             # one slab
    # the shapes of test_batches_of_the_streaming_kernel reach what they are there for
    (0, 70_001, 264, 16, 3, 3), (1, 70_001, 1_000, 3, 10, 3), (0, 140_003, 160, 5, 4, 5), (1, 140_003, 136, 7, 16, 5), (0, 200_001, 776, 40, 10, 5),
    (1, 200_001, 776, 64, 3, 5), (0, 200_000, 456, 17, 16, 5), (0, 1_000_001, 264, 33, 3, 3), (1, 70_001, 768, 40, 4, 2), (0, 150_000, 1_024, 64, 10, 2),
    (1, 600_001, 192, 17, 5, 2), (2, 60_001, 80, 9, 4, 2), (2, 50_000, 96, 16, 10, 2), (2, 40_001, 2_400, 3, 1, 2)])
def test_batches_where_they_were_measured_to_pay(plans, dtype, N, d, B, k, batch):
    assert plans.batch(CUS, N, d, dtype, B, k) == batch


MID, THIN = 2, 3                                      # 256 x 128, 128 x 64


def col_tiles(B, tile):
    return (B + 127) // 128 if tile == MID else (B + 63) // 64


# us, stages of rows / of lines of memory; tile by both rules
@pytest.mark.parametrize("N,d,B,by_line,first,tile", [
    (123_457, 776, 77, 1, 2, 2),         # 56.4 / 51.3
    (80_000, 776, 77, 0, 2, 2),          # from the caches 39.9 / 40.1
    (168_000, 800, 77, 1, 2, 2),         # half lines, 256 MiB
    (123_457, 800, 77, 0, 2, 2),         # 41.8 / 43.1
    (141_881, 488, 170, 0, 0, 2),        # read again 54.2 / 59.4: two tiles of queries, a stage more
    (136_000, 776, 170, 0, 0, 2),        # ... two tiles of queries
    (130_000, 504, 77, 0, 2, 2),         # ... a stage more, 1 / 1.024
    (247_898, 280, 108, 0, 2, 1),        # ... 38.8 / 42.3
    (360_486, 208, 81, 1, 2, 1),         # read again 45.4 / 48.0 in the place of 512 x 128
    (2_195_041, 216, 99, 1, 1, 1),       # 1 / 1.024, a third of the lines not the row
    (1_000_000, 768, 128, 0, 2, 2),      # whole lines
    (1_500_000, 120, 128, 0, 1, 1),      # less than a line
    (1_000_000, 456, 128, 1, 1, 2),      # 271 / 248, in the place of 512 x 128
    (4_000_000, 184, 100, 1, 1, 1),      # 412 / 414
    (2_000_000, 352, 100, 1, 1, 1)])     # 344 / 349
def test_lines_of_memory_where_they_were_measured_to_pay(plans, N, d, B, by_line, first, tile):
    assert (plans.by_line(N, d, col_tiles(B, MID)), plans.shape(CUS, N, d, B), plans.tile(CUS, N, d, B, 3)) == (by_line, first, tile)


@pytest.mark.parametrize("N,d,B,k,tile", [
    (83_001, 776, 77, 10, MID), (134_401, 1_000, 66, 16, MID), (680_000, 200, 70, 3, MID), (135_424, 992, 128, 3, MID),
    (330_001, 200, 40, 4, THIN), (480_000, 136, 17, 16, THIN), (300_000, 264, 40, 1, THIN)])
def test_the_tests_of_lines_of_memory_reach_them(plans, N, d, B, k, tile):
    """The shapes of test_stages_of_lines_of_memory go by lines, in groups of rows, and the pieces that they are compared with do not."""
    p = flat(plans, N, d, 0, B, k, 1 << 30)
    assert (KINDS[p["kind"]], p["shape"], p["rows"], p["part"]) == ("wide", tile, N, B) and p["gs_log"] > 0
    assert plans.by_line(N, d, col_tiles(B, tile)) and not plans.by_line(60_000_000 // (2 * d), d, 1)


@pytest.mark.parametrize("N,d,B,k,size", [(62_553, 2_056, 33, 9, 140_257), (42_905, 3_856, 24, 7, 54_955)])
def test_the_tests_of_parts_by_lines_of_memory_reach_them(plans, N, d, B, k, size):
    """... of test_parts_of_lines_of_memory: more than one part by lines, and the whole in other groups of rows."""
    whole, p = flat(plans, N, d, 0, B, k, 1 << 30), flat(plans, N, d, 0, B, k, size)
    assert KINDS[p["kind"]] == "wide" and p["bytes"] <= size and p["shape"] == THIN and p["gs_log"] > 0
    assert 2 * p["rows"] <= N and plans.by_line(p["rows"], d, col_tiles(B, THIN))
    assert KINDS[whole["kind"]] == "wide" and whole["rows"] == N and whole["gs_log"] != p["gs_log"]


@pytest.mark.parametrize("N,d,B,k,buffer", [
    (5_000_000, 200, 60, 3, 200_000), (8_600_000, 120, 40, 12, 100_000), (1_500_000, 256, 64, 3, 150_000)])
def test_lists_that_do_not_fit_leave_the_parts(plans, N, d, B, k, buffer):
    """Calls whose lists get less than a quarter of their slabs are taken in parts where there are many queries."""
    p = flat(plans, N, d, 0, B, k, buffer)
    assert KINDS[flat(plans, N, d, 0, B, k, 1 << 30)["kind"]] == "lists"
    assert KINDS[p["kind"]] == "wide" and p["rows"] < N and p["bytes"] <= buffer


# us of a call in a buffer of so many bytes, one pass on lists / parts on the matrix cores
@pytest.mark.parametrize("N,d,B,k,buffer,kind", [
    (1_000_000, 128, 64, 3, 1 << 20, "lists"),       # 107 / 146
    (16_000_000, 64, 32, 3, 1 << 20, "lists"),       # 486 / 905
    (300_000, 128, 32, 3, 1 << 18, "lists"),         # 31 / 53
    (100_000, 256, 32, 3, 1 << 17, "lists"),         # 28 / 55
    (1_884_008, 24, 4, 1, 84_927, "lists"),          # 61 / 96
    (558_736, 32, 4, 3, 17_158, "lists"),            # 54 / 172
    (1_773_482, 1384, 61, 3, 267_598, "lists"),      # 1374 / 2465
    (1_052_988, 96, 41, 3, 205_116, "lists"),        # 163 / 331, a third of the slabs
    (344_490, 2752, 25, 10, 367_182, "lists"),       # 534 / 706
    (16_000_000, 8, 1, 2, 63_000, "wide"),           # 436 / 286, 18 parts
    (16_000_000, 32, 8, 3, 1 << 20, "wide"),         # 487 / 308
    (3_003_528, 40, 24, 1, 3_134_841, "wide"),       # 145 / 75
    (2_000_000, 2048, 40, 3, 1 << 20, "wide"),       # 1982 / 1770
    (1_185_604, 2976, 39, 3, 2_251_554, "wide"),     # 2689 / 1533
    (1_549_591, 1600, 57, 5, 122_708, "wide"),       # 4354 / 2649, a quarter of the slabs
    (258_523, 3392, 41, 16, 180_826, "wide")])       # 1647 / 1030
def test_parts_or_lists_in_a_small_buffer(plans, N, d, B, k, buffer, kind):
    p = flat(plans, N, d, 0, B, k, buffer)
    assert KINDS[p["kind"]] == kind and p["bytes"] <= buffer
    assert (kind == "lists") == (p["rows"] == N)


def test_the_static_workspace_keeps_the_kernel(plans):
    """Up to 64 queries of 16 bits: what one pass would take, if it fits at all."""
    rng = random.Random(3)
    log = lambda lo, hi: int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    parts = 0
    for _ in range(4000):
        N, d, B, k = log(1, 5e7), 8 * log(1, 512), rng.randint(1, 64), rng.randint(1, 16)
        k = min(k, N)
        whole, static = (plans.static_kind(CUS, N, d, 0, B, k, size) for size in (1 << 40, STATIC))
        if static >= 0:
            assert whole == static, (N, d, B, k)
        parts += static == 2 and flat(plans, N, d, 0, B, k, 1 << 30)["bytes"] > STATIC
    assert parts > 20


@pytest.mark.parametrize("N,d,elem_bytes,ef", [
    (1_246_720, 64, 2, 256), (1_246_720, 64, 2, 200), (1_241_088, 416, 2, 117), (1_238_528, 64, 2, 320), (1_223_168, 1024, 2, 257),
    (1_214_976, 1024, 4, 256), (1_213_952, 64, 2, 512), (1_200_640, 64, 2, 700), (165_888, 1024, 2, 16_384)])
def test_searches_that_need_no_workspace(plans, N, d, elem_bytes, ef):
    """The largest graphs whose maturity search keeps its visited set in LDS where no workspace is at hand: the calls that ran
    with none when lists were written out."""
    assert plans.in_lds(N, d, elem_bytes, 32, ef)


# us of a call, the streaming kernel's one slab / flat_direct_kernel
@pytest.mark.parametrize("N,d,dtype,B,kind", [
    (128, 128, 0, 16, "quick"),          # 4.95 / 4.38
    (16, 384, 0, 64, "quick"),           # 4.54 / 4.04
    (64, 512, 0, 16, "quick"),
    (16, 1_536, 0, 16, "direct"),        # 6.67 / 8.41: whole runs of steps, long rows
    (4, 2_048, 1, 512, "direct"),        # 7.76 / 9.62
    (128, 768, 0, 64, "direct"),         # 10.2 / 10.4
    (17, 496, 0, 1, "quick"),            # 6.34 / 4.36: rows that end inside a run
    (35, 3_944, 0, 578, "quick"),        # 22.5 / 17.0
    (74, 528, 0, 1, "quick"),            # 7.47 / 6.39
    (128, 64, 2, 16, "quick"),           # 6.39 / 5.38
    (64, 384, 2, 64, "direct"),          # 8.13 / 9.83
    (93, 448, 2, 1_514, "direct"),       # 11.1 / 14.1
    (128, 384, 2, 64, "direct"),         # 10.6 / 14.1
    (18, 4_048, 2, 554, "quick"),        # 70.9 / 62.3
    (121, 272, 2, 65, "direct"),         # 10.0 / 11.4
    (7, 32, 0, 2, "direct"),             # 4.0 / 4.8
    (3, 832, 2, 11_876, "direct")])      # 25.4 / 37.2
def test_one_launch_for_few_rows(plans, N, d, dtype, B, kind):
    assert KINDS[flat(plans, N, d, dtype, B, 1, 1 << 30)["kind"]] == kind


# us of a call, the streaming kernel's lists or the matrix cores / flat_scores_kernel and a pick
@pytest.mark.parametrize("N,d,dtype,B,k,scores", [
    (21_025, 480, 0, 14, 2, True),       # lists 13.8 / 12.4
    (10_000, 128, 2, 16, 10, True),      # 11.6 / 10.3
    (18_204, 416, 1, 20, 3, True),       # 18.1 / 14.8
    (12_722, 32, 0, 18, 3, True),        # 10.0 / 8.5
    (27_070, 896, 1, 16, 16, False),     # 17.4 / 21.4
    (33_953, 64, 0, 8, 3, False),        # 10.0 / 12.6
    (200, 768, 0, 1, 3, True),           # matrix cores 8.5 / 6.3
    (200, 768, 0, 256, 1, True),         # 9.6 / 7.2
    (128, 384, 0, 9, 10, True),          # more than 64 rows, k > 4: may use the workspace
    (14_587, 320, 0, 30, 10, False),     # 11.4 / 14.0
    (12_383, 768, 1, 22, 5, False),      # 12.7 / 17.5
    (7_912, 1_408, 1, 22, 5, False),     # 12.9 / 17.4
    (5_087, 1_984, 1, 17, 16, False),    # 14.5 / 18.7
    (2_781, 2_496, 0, 38, 1, False),     # 14.7 / 19.2
    (8_691, 192, 0, 57, 10, False),      # 10.5 / 12.8
    (1_024, 768, 0, 512, 1, False)])     # 10.4 / 17.3
def test_scores_where_they_were_measured_to_pay(plans, N, d, dtype, B, k, scores):
    assert (KINDS[flat(plans, N, d, dtype, B, k, 1 << 30)["kind"]] == "scores") == scores


# the shapes of tests/test_gpu_small.py reach what they are there for
@pytest.mark.parametrize("dtype,N,d,B,k,kind", [
    (0, 1, 1_000, 1, 1, "quick"), (1, 17, 104, 17, 16, "quick"), (0, 64, 456, 33, 7, "quick"), (0, 113, 264, 5, 16, "quick"),
    (2, 128, 96, 16, 10, "quick"), (2, 20, 1_092, 40, 5, "quick"), (2, 4, 4_092, 3, 4, "quick"), (0, 16, 1_040, 300, 3, "quick"),
    (0, 128, 240, 2, 3, "quick"), (0, 100, 200, 20, 8, "quick"),
    (0, 100, 1_024, 2, 16, "scores"), (0, 129, 8, 1, 16, "scores"), (1, 1_999, 776, 16, 16, "scores"), (0, 2_048, 768, 17, 10, "scores"),
    (0, 2_049, 1_544, 3, 1, "scores"), (2, 10_000, 132, 16, 10, "scores"), (2, 700, 2_052, 9, 4, "scores"), (0, 21_025, 480, 14, 2, "scores"),
    (0, 2_000, 200, 20, 8, "scores"), (1, 4_000, 64, 3, 16, "scores"),
    (2, 128, 132, 16, 10, "direct"), (2, 4, 4_096, 3, 4, "direct"), (0, 128, 768, 64, 4, "direct"), (1, 64, 2_048, 33, 16, "direct"),
    (2, 100, 512, 40, 10, "direct"), (0, 80, 768, 512, 1, "direct")])
def test_kernels_of_few_rows(plans, dtype, N, d, B, k, kind):
    assert KINDS[flat(plans, N, d, dtype, B, k, 1 << 30)["kind"]] == kind


@pytest.mark.parametrize("dtype,N,d,B,k", [(2, 10_000, 132, 16, 10), (2, 700, 2_052, 9, 4), (0, 21_025, 480, 14, 2)])
def test_scores_give_way_to_lists_in_a_smaller_buffer(plans, dtype, N, d, B, k):
    """What tests/test_gpu_small.py compares the bits of."""
    p = flat(plans, N, d, dtype, B, k, 1 << 30)
    q = flat(plans, N, d, dtype, B, k, p["bytes"] - 16)
    assert KINDS[p["kind"]] == "scores" and KINDS[q["kind"]] == "lists" and q["bytes"] < p["bytes"]


@pytest.mark.parametrize("dtype", [0, 1, 2])
def test_few_rows_need_no_workspace(plans, dtype):
    """Exact searches of so few rows may overlap anything, so none of them, however long its rows and large its batch, may write the
    workspace that the calls of a device share."""
    rng = random.Random(dtype)
    log = lambda lo, hi: int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    step = 4 if dtype == 2 else 8
    calls = [(128, 768, 1, 1), (128, 768, 64, 4), (80, 768, 512, 1), (64, 4096, 16, 16), (65, 3304, 123, 1), (1, 8, 1, 1), (128, 4, 9719, 1)]
    for _ in range(8000):
        N = rng.randint(1, 128)
        calls.append((N, step * log(1, 4096 // step), log(1, 70_000), min(N, rng.choice([1, 3, 4, 5, 10, 16]))))
    for N, d, B, k in calls:
        if N > (128 if dtype == 2 or k <= 4 else 64) or d % step:
            continue
        assert flat(plans, N, d, dtype, B, k, 1 << 30)["bytes"] == 0, (N, d, B, k)
        assert flat(plans, N, d, dtype, B, k, 1)["bytes"] == 0, (N, d, B, k)


# us of flat_pick_kernel with long runs of steps / without
@pytest.mark.parametrize("d,elem_bytes,B,runs", [
    (48, 2, 2765, False),        # 41.2 / 24.3
    (32, 2, 514, False),         # 28.4 / 18.2
    (320, 2, 3989, False),       # 30.5 / 20.7
    (376, 2, 77, False),         # 23 steps and a half
    (384, 2, 77, True),          # 9.1 / 10.5
    (776, 2, 512, True),         # 14.9 / 16.5
    (1024, 2, 4000, False),      # 69.7 / 62.3
    (544, 2, 900, True),         # 10.3 / 12.2
    (544, 2, 1100, False),       # 16.3 / 14.0
    (1152, 2, 1531, True),       # 19.7 / 20.5
    (768, 2, 4000, False),       # 125.9 / 108.9
    (1544, 2, 4000, True),       # 59.0 / 67.4
    (392, 4, 400, True),         # 20.1 / 21.9
    (128, 4, 300, False)])
def test_long_runs_where_they_were_measured_to_pay(plans, d, elem_bytes, B, runs):
    assert bool(plans.runs(CUS, d, elem_bytes, B)) == runs


# taken though one pass with the group sizes of today needs more than the static workspace: in parts, or by larger groups
STATIC_LINE = ((8229, 928, 297, 5), (9226, 64, 2414, 14), (7516, 96, 2011, 7), (210058, 32, 337, 13),
               (135374, 32, 749, 13), (1687, 96, 4734, 10), (4871, 64, 5009, 5), (215654, 64, 581, 9))


def test_the_static_workspace_takes_what_one_pass_fits(plans):
    """Whatever ann_flat_workspace_bytes says fits it, and the calls of long answers that it took by other group sizes."""
    rng = random.Random(8)
    log = lambda lo, hi: int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    for _ in range(20_000):
        N, d, B, k = log(16, 1e6), 8 * log(1, 512), log(256, 20_000), rng.randint(5, 16)
        if flat(plans, N, d, 0, B, k, 1 << 30)["bytes"] <= 8 * 1024 * 1024:
            assert plans.static_accepts(CUS, N, d, 0, B, k, STATIC), (N, d, B, k)
    for N, d, B, k in STATIC_LINE:
        assert plans.static_accepts(CUS, N, d, 0, B, k, STATIC), (N, d, B, k)


LARGE, TALL, MID, THIN, TINY, SHORT = range(6)


# us of a call with 128 x 64 tiles of whole / half lines
@pytest.mark.parametrize("N,d,B,shape", [
    (3_737_423, 8, 6, SHORT),        # 79.8 / 55.9
    (1_243_025, 24, 18, SHORT),      # 33.9 / 26.0
    (1_273_004, 32, 54, SHORT),      # 35.4 / 28.5
    (45_140, 8, 11, SHORT),          # 9.5 / 9.1
    (35_294, 224, 85, SHORT),        # 16.0 / 14.5: 552 tiles
    (90_354, 88, 28, SHORT),         # 13.3 / 11.8: 706 tiles
    (2_746_069, 64, 3, THIN),        # 79.1 / 90.4
    (106_876, 384, 28, THIN),        # 21.9 / 23.7
    (21_798, 448, 183, THIN),        # 17.9 / 18.5: 513 tiles
    (48_119, 112, 7, THIN)])         # 12.9 / 12.8
def test_half_lines_for_short_rows(plans, N, d, B, shape):
    assert plans.shape(CUS, N, d, B) == shape


SQUARE = 6


# us of a call with the first rule's tile / this one
@pytest.mark.parametrize("N,d,B,tile", [
    (977, 768, 5_000, SQUARE),       # 26.6 / 25.2: 320 tiles in one round, 632 of 128 x 64 in two
    (24_000, 768, 200, SQUARE),      # 26.2 / 21.9
    (10_564, 768, 6_152, MID),       # 211 / 195: nine rounds of half the work instead of five
    (2_500, 768, 977, THIN),         # one round of them: stays
    (1_000_000, 768, 512, LARGE),
    (110_746, 768, 301, MID),        # from memory: tiles of few queries read too often, 92 / 101 by 128 x 128
    (10_427, 64, 808, MID),          # short rows: the first rule's, 18.7 / 20.7 by 256 x 256
    (977, 776, 5_000, SQUARE), (1_025, 72, 5_000, SQUARE), (24_001, 264, 200, SQUARE), (50_049, 136, 66, SQUARE), (46_408, 384, 883, SQUARE),
    (1_025, 72, 4_097, SHORT),       # 21.0 / 21.5 by 128 x 128: the half-line tile, which the model does not know, up to 160 elements
    (38_784, 96, 68, SHORT),         # 12.9 / 13.8
    (22_463, 160, 133, SHORT),       # 3 % longer by 128 x 128
    (22_751, 192, 210, SQUARE),      # 0.94 times as long
    (2_268_470, 384, 70, TALL),      # 366 / 381 by 256 x 128: from memory too close to tell
    (40_000, 768, 64, THIN), (1_024, 768, 512, TINY), (1_200_000, 24, 18, SHORT)])
def test_tiles_by_rounds(plans, N, d, B, tile):
    assert plans.tile(CUS, N, d, B, 3) == tile


@pytest.mark.parametrize("N,d,B", [(16_958, 128, 867), (18_158, 160, 778), (15_932, 168, 822)])
def test_long_answers_behind_large_tiles(plans, N, d, B):
    """k = 16: 24.8 us by 256 x 128, 28.2 by 512 x 128; 26.4 / 28.2; 26.3 / 29.1 by 256 x 256, whose pick has more to do."""
    assert plans.tile(CUS, N, d, B, 16) == MID and plans.tile(CUS, N, d, B, 10) != MID


@pytest.mark.parametrize("seed", range(3))
def test_fewest_rounds_only_where_the_maxima_fit_at_once(plans, seed):
    """A call that goes in parts gets the plan of the first rule alone, tile included; one that does not may get another tile, in any room that holds its
    maxima, of larger groups if need be.  What the first rule's plan fits, either fits."""
    rng = random.Random(seed)
    other = parts = 0
    for _ in range(1500):
        N, B = (int(math.exp(rng.uniform(math.log(lo), math.log(hi)))) for lo, hi in ((200, 3e6), (66, 8192)))
        d, k = 8 * rng.randint(1, 128), rng.choice([1, 3, 10, 16])
        k = min(k, N)
        whole = flat(plans, N, d, 0, B, k, 1 << 30)
        for limit in (1 << 30, whole["bytes"], int(whole["bytes"] * rng.uniform(0.01, 0.9))):
            p, first = flat(plans, N, d, 0, B, k, limit), flat(plans, N, d, 0, B, k, limit, by_fill=True)
            assert p["bytes"] <= limit or first["bytes"] > limit, (N, d, B, k, limit)
            if p["part"] < B or p["rows"] < N:
                assert p == first, (N, d, B, k, limit)
                parts += 1
            other += p["shape"] != first["shape"]
        again = flat(plans, N, d, 0, B, k, whole["bytes"])
        assert again["bytes"] <= whole["bytes"] and (again["part"], again["rows"], again["shape"]) == (whole["part"], whole["rows"], whole["shape"])
        if whole["bytes"] <= 8 * 1024 * 1024:
            assert plans.static_accepts(CUS, N, d, 0, B, k, STATIC), (N, d, B, k)
    assert parts > 100 and other > 100, (parts, other)


# share of queries that leave early
@pytest.mark.parametrize("tau,window,R,ef,likely", [
    (0.9, 500, 32, 256, True),            # 0.8 and more
    (0.9, 500, 24, 64, True),
    (0.7, 100, 8, 10, True),              # 0.9
    (0.95, 2000, 32, 64, True),           # 0.5 to 0.9
    (0.95, 2000, 16, 32, False),          # 0.2
    (0.999, 2_000_000_000, 32, 512, False),
    (0.999, 2_000_000_000, 32, 16_384, False),
    (3.0, 500, 32, 2048, False), (NEVER, 500, 32, 2048, False), (1.0, 1, 32, 16_384, False),
    (0.0, 2_000_000_000, 1, 1, True), (-1.0, 500, 1, 1, True), (-NEVER, 500, 1, 1, True)])
def test_whether_the_exit_is_likely(plans, tau, window, R, ef, likely):
    assert bool(plans.leaves(tau, window, R, ef)) == likely
