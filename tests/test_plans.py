"""What a call would launch, decided without a GPU: the host rules of plan.hpp, compiled with the C++ compiler alone.

The rules choose between ways of giving the same answer, so a wrong one costs time and no test of results sees it."""
import ctypes
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CUS = 256

SHIM = r"""
#include "plan.hpp"
using namespace ann;
extern "C" int step_pays(int cus, int64_t N, int row_bytes, int R, int B, int ef, int counters, float tau) {
    return graph_step_pays(cus, N, row_bytes, R, B, ef, counters != 0, tau);
}
"""


@pytest.fixture(scope="module")
def plans(tmp_path_factory):
    tmp = tmp_path_factory.mktemp("plans")
    src, lib = tmp / "shim.cpp", tmp / "shim.so"
    src.write_text(SHIM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-shared", "-fPIC", "-I",
                    os.path.join(ROOT, "paper_2505_12065_amd", "csrc"), "-o", str(lib), str(src)], check=True)
    L = ctypes.CDLL(str(lib))
    L.step_pays.argtypes = [ctypes.c_int, ctypes.c_int64] + [ctypes.c_int] * 5 + [ctypes.c_float]
    return L


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
