"""The LDS stages of the matrix-core kernel, by the assembly that the compiler makes of it: a barrier there waits for no memory operation, and
behind it loads go to a buffer that other waves have read.  So no wave may come to it with LDS reads outstanding; that a load takes longer
than a read hides a missing wait from any test of results.  And what the kernel keeps in scratch memory."""
import re
import subprocess

import pytest

from paper_2505_12065_amd.build import CSRC, FLAGS, HIPCC

TILES = ("WideLarge", "WideTall", "WideMid", "WideSquare", "WideThin", "WideTiny", "WideShort")
BY_LINE = ("WideMid", "WideThin")                         # the tiles that have stages of lines of memory as well


def outstanding(body):
    """The most LDS operations of a wave that may be outstanding at each s_barrier of a kernel, over all paths; how many barriers, reads and
    direct loads there are.  (lgkmcnt counts scalar loads too: a wait for n leaves at most n of either.)"""
    lines = [line.split(";")[0].strip() for line in body.split("\n")]
    lines = [line for line in lines if line and (line.endswith(":") or not line.startswith("."))]
    label = {line[:-1]: i for i, line in enumerate(lines) if line.endswith(":")}
    seen, at, todo = {}, {}, [(0, 0)]
    while todo:
        i, n = todo.pop()
        while i < len(lines) and seen.get(i, -1) < n:
            seen[i] = n
            op, _, args = lines[i].partition(" ")
            if op.startswith("ds_"):
                n = min(n + 1, 100)
            elif op == "s_waitcnt":
                counts = dict(re.findall(r"(vmcnt|expcnt|lgkmcnt)\((\d+)\)", args))
                assert counts, lines[i]
                n = min(n, int(counts.get("lgkmcnt", n)))
            elif op == "s_barrier":
                at[i] = max(at.get(i, 0), n)
            elif op.startswith("s_cbranch"):
                todo.append((label[args.strip()], n))
            elif op == "s_branch":
                i = label[args.strip()]
                continue
            else:
                assert op not in ("s_setpc_b64", "s_swappc_b64"), lines[i]     # (a call would not be followed)
                if op == "s_endpgm":
                    break
            i += 1
    count = lambda op: sum(line.startswith(op) for line in lines)
    return [at[i] for i in sorted(at)], count("s_barrier"), count("ds_read"), count("global_load_lds")


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    tmp = tmp_path_factory.mktemp("barriers")
    src, asm = tmp / "wide.hip", tmp / "wide.s"
    forms = [(t, "false") for t in TILES] + [(t, "true") for t in BY_LINE]
    src.write_text('#include "flat_wide_kernel.hpp"\nnamespace ann {\n' + "".join(
        f"template __global__ void flat_wide_kernel<F16, {t}, false, {by_line}>(const void *, int64_t, int, const void *, int, float *, int64_t, int, int, int, After);\n"
        for t, by_line in forms) + "}\n")
    subprocess.run([HIPCC, *FLAGS, "-I", CSRC, "--cuda-device-only", "-S", str(src), "-o", str(asm)], check=True, capture_output=True, text=True)
    bodies = re.findall(r"^_ZN3ann16flat_wide_kernel\w+:[^\n]*\n(.*?)^\.Lfunc_end", asm.read_text(), re.S | re.M)
    assert len(bodies) == len(forms)
    return dict(zip(forms, bodies))


@pytest.mark.parametrize("tile,by_line", [(t, "false") for t in TILES] + [(t, "true") for t in BY_LINE])
def test_no_reads_outstanding_at_a_barrier(kernels, tile, by_line):
    at, barriers, reads, loads = outstanding(kernels[tile, by_line])
    assert barriers and reads and loads and len(at) == barriers          # (all barriers are reached)
    assert at == [0] * barriers


@pytest.mark.parametrize("tile,by_line", [(t, "false") for t in TILES] + [(t, "true") for t in BY_LINE])
def test_no_register_in_scratch_memory(kernels, tile, by_line):
    """A wait for one that comes back is a wait for the stage loads that are on their way."""
    assert "scratch_" not in kernels[tile, by_line]


def test_an_outstanding_read_is_seen():
    body = "\tds_read_b128 v[0:3], v4\n\ts_cbranch_scc0 .LBB0_1\n\ts_waitcnt vmcnt(0) lgkmcnt(0)\n.LBB0_1:\n\ts_barrier\n\ts_endpgm\n"
    assert outstanding(body)[0] == [1]
    assert outstanding(body.replace("s_cbranch_scc0 .LBB0_1", "s_nop 0"))[0] == [0]
