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
extern "C" int step_pays(int cus, int64_t N, int row_bytes, int R, int B, int ef, int counters, float tau) {
    return graph_step_pays(cus, N, row_bytes / 2, 2, R, B, ef, counters != 0, tau);
}
extern "C" int in_lds(int64_t N, int d, int elem_bytes, int R, int ef) {
    FrontierLds L;
    return frontier_in_lds(N, d, elem_bytes, R, ef, true, L);
}
// out: kind (0 lists, 1 direct, 2 matrix cores, 3 streaming with maxima), queries and rows at a time, maxima of a query,
// log2 of the rows they stand for, offset of the k best so far, workspace, maxima of the smallest last part
extern "C" void flat(int cus, int64_t N, int d, int dtype, int B, int k, int64_t limit, int64_t *out) {
    const FlatPlan pl = flat_plan(cus, N, d, dtype, B, k, (size_t)limit);
    const int64_t rows = N % pl.rows ? N % pl.rows : pl.rows;
    const int part = B % pl.part ? B % pl.part : pl.part;
    const FlatPlan last = pl.wide || pl.maxima ? maxima_part(pl, rows, part, d, dtype) : pl;
    const int64_t v[] = {pl.wide ? 2 : pl.maxima ? 3 : pl.direct ? 1 : 0, pl.part, pl.rows, pl.w.n, pl.w.gs_log,
                         (int64_t)pl.best_ofs, (int64_t)pl.ws_bytes, last.w.n, last.w.gs_log};
    for (int i = 0; i < 9; ++i) out[i] = v[i];
}
extern "C" int static_accepts(int cus, int64_t N, int d, int dtype, int B, int k, int64_t bytes) {
    return static_plan(cus, N, d, dtype, B, k, (size_t)bytes).ws_bytes <= (size_t)bytes;
}
extern "C" int static_kind(int cus, int64_t N, int d, int dtype, int B, int k, int64_t bytes) {
    const FlatPlan pl = static_plan(cus, N, d, dtype, B, k, (size_t)bytes);
    return pl.ws_bytes > (size_t)bytes ? -1 : pl.wide ? 2 : pl.maxima ? 3 : pl.direct ? 1 : 0;
}
"""
KINDS = ("lists", "direct", "wide", "maxima")
STATIC = 8 * 1024 * 1024 + 1024 * 16 * 8             # the static workspace, room for the k best of a part's queries included


@pytest.fixture(scope="module")
def plans(tmp_path_factory):
    tmp = tmp_path_factory.mktemp("plans")
    src, lib = tmp / "shim.cpp", tmp / "shim.so"
    src.write_text(SHIM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-shared", "-fPIC", "-I",
                    os.path.join(ROOT, "paper_2505_12065_amd", "csrc"), "-o", str(lib), str(src)], check=True)
    L = ctypes.CDLL(str(lib))
    L.step_pays.argtypes = [ctypes.c_int, ctypes.c_int64] + [ctypes.c_int] * 5 + [ctypes.c_float]
    L.in_lds.argtypes = [ctypes.c_int64] + [ctypes.c_int] * 4
    L.flat.argtypes = [ctypes.c_int, ctypes.c_int64] + [ctypes.c_int] * 4 + [ctypes.c_int64, ctypes.c_void_p]
    L.static_accepts.argtypes = L.static_kind.argtypes = [ctypes.c_int, ctypes.c_int64] + [ctypes.c_int] * 4 + [ctypes.c_int64]
    return L


def flat(L, N, d, dtype, B, k, limit):
    out = (ctypes.c_int64 * 9)()
    L.flat(CUS, N, d, dtype, B, k, limit, out)
    return dict(zip(("kind", "part", "rows", "n", "gs_log", "best_ofs", "bytes", "last_n", "last_gs_log"), out))


# one-by-one / steps as measured, where the two sides differ by more than a tenth
@pytest.mark.parametrize("N,row,R,B,ef,pays", [
    (1_000_000, 1536, 32, 512, 1024, False),     # 0.68 .. 0.71: the corpus of the benchmark, mid search ranges
    (1_000_000, 1536, 32, 512, 2048, False),     # 0.75
    (1_000_000, 1536, 32, 512, 4096, False),     # 0.87
    (1_000_000, 1536, 32, 512, 12288, True),     # 1.13
    (1_000_000, 1536, 32, 256, 1024, False),     # 0.80: here the visited bits fit LDS
    (1_000_000, 768, 32, 512, 1024, False),      # 0.70
    (1_000_000, 1024, 32, 256, 600, False),      # 0.79
    (200_000, 1536, 32, 256, 2048, True),        # 1.07
    (200_000, 1536, 32, 512, 4096, True),        # 1.36
    (200_000, 768, 32, 256, 600, False),         # 0.90
    (50_000, 1536, 32, 256, 1024, True),         # 1.19
    (200_000, 1536, 16, 512, 1024, True),        # 1.15
    (1_000_000, 1536, 32, 2048, 192, False),     # 0.77: one list, more queries than places
    (1_000_000, 1536, 32, 1024, 512, False),     # 0.77
    (400_000, 1536, 32, 2048, 192, False),       # 0.79
    (200_000, 768, 32, 600, 320, True),          # 1.25
    (200_000, 1536, 32, 4, 320, False),          # 0.90
    (1_000_000, 1536, 32, 1, 512, True),         # 2.97
    (1_000_000, 1536, 32, 512, 64, False),
    (1_000_000, 1536, 32, 512, 9000, False),     # 0.66: two workgroups per compute unit one by one, one in steps
    (50_000, 1536, 32, 512, 9000, True),         # 1.42
    (1_000_000, 1536, 32, 512, 10_000, True),    # 1.18: one and one
    (1_000_000, 1536, 32, 512, 8192, True),      # 1.05: two and two
])
def test_steps_only_where_they_were_measured_to_pay(plans, N, row, R, B, ef, pays):
    assert bool(plans.step_pays(CUS, N, row, R, B, ef, 0, float("inf"))) == pays


def test_steps_pay_up_to_a_size_of_the_graph(plans):
    """Whatever the other sizes are: never again on a larger graph once they no longer do."""
    for row in (128, 768, 1536, 4096):
        for R in (8, 24, 32):
            for B in (1, 4, 16, 256, 257, 512, 513, 800, 1024, 2048):
                for ef in (64, 192, 320, 512, 513, 1024, 4096, 16384):
                    got = [bool(plans.step_pays(CUS, N, row, R, B, ef, 0, float("inf"))) for N in
                           (100, 10_000, 50_000, 200_000, 1_000_000, 10_000_000, 2**31 - 1)]
                    assert got == sorted(got, reverse=True), (row, R, B, ef)


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
