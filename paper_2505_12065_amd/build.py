"""Build libann.so (gfx950) from csrc/*.hip with hipcc: one object per
translation unit, compiled in parallel, linked into the package directory; and _marshal.so,
the binding's native half, from csrc/marshal.cpp with the host compiler and torch's headers."""
from __future__ import annotations

import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OBJ = os.path.join(CSRC, "_build")
LIB = os.path.join(HERE, "libann.so")
MARSHAL = os.path.join(HERE, "_marshal.so")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
# -packed-fp32-ops is switched off on purpose: some packed fp32 forms have been
# seen to give wrong results on the test machines.
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Wall",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]


def _sources():
    return sorted(f for f in os.listdir(CSRC) if f.endswith(".hip"))


def _headers_mtime():
    hs = [os.path.join(CSRC, f) for f in os.listdir(CSRC) if f.endswith(".hpp")]
    hs.append(os.path.join(HERE, "..", "include", "ann.h"))
    return max(os.path.getmtime(h) for h in hs)


def _compile(src: str, force: bool) -> str:
    obj = os.path.join(OBJ, src[:-4] + ".o")
    spath = os.path.join(CSRC, src)
    if (not force and os.path.exists(obj)
            and os.path.getmtime(obj) > max(os.path.getmtime(spath), _headers_mtime())):
        return obj
    cmd = [HIPCC, *FLAGS, "-c", spath, "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    err = "\n".join(l for l in r.stderr.splitlines() if "packed-fp32-ops" not in l)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed on {src}:\n{err}")
    if err.strip():
        sys.stderr.write(err + "\n")
    return obj


def marshal_target() -> str:
    """What _marshal.so is built for: it has the layouts of one torch's and one Python's objects compiled into it."""
    import torch
    return f"torch {torch.__version__} python {sys.version_info[0]}.{sys.version_info[1]}"


def _build_marshal(force: bool) -> None:
    src = os.path.join(CSRC, "marshal.cpp")
    target, record = marshal_target(), os.path.join(OBJ, "marshal.target")
    if not force and os.path.exists(MARSHAL) and os.path.getmtime(MARSHAL) > max(os.path.getmtime(src), _headers_mtime()):
        if os.path.exists(record):
            with open(record) as f:
                if f.read() == target:
                    return
    import sysconfig
    import torch
    from torch.utils import cpp_extension
    include = [f"-isystem{p}" for p in cpp_extension.include_paths() + [sysconfig.get_paths()["include"]]]
    libs = os.path.join(os.path.dirname(torch.__file__), "lib")
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall",
                           f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}", f'-DANN_BUILT_FOR="{target}"', *include, src,
                           "-o", MARSHAL, f"-L{libs}", "-ltorch_python", "-ltorch_cpu", "-lc10"])
    with open(record, "w") as f:
        f.write(target)


def _try_marshal(force: bool) -> None:
    """The library does not need it: where it cannot be built, none is left and the binding marshals in Python."""
    try:
        _build_marshal(force)
    except (OSError, ImportError, subprocess.CalledProcessError) as e:
        if os.path.exists(MARSHAL):
            os.remove(MARSHAL)
        sys.stderr.write(f"_marshal.so was not built: {e}\n")


def build_library(force: bool = True, jobs: int = 8) -> str:
    os.makedirs(OBJ, exist_ok=True)
    with ThreadPoolExecutor(max_workers=jobs) as ex:
        marshal = ex.submit(_try_marshal, force)
        objs = list(ex.map(lambda s: _compile(s, force), _sources()))
        marshal.result()
    subprocess.check_call([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB, *objs])
    return LIB


if __name__ == "__main__":
    print(build_library(force="--incremental" not in sys.argv))
