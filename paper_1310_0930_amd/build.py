"""Build libpic.so (HIP for gfx950) in-tree with hipcc."""
import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libpic.so")
SOURCES = ["pic_api.hip", "k_push.hip", "k_sort.hip", "k_fdtd.hip", "k_diag.hip", "k_adjoint.hip",
           "k_window.hip"]
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-munsafe-fp-atomics",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-Wall", "-Wno-unused-function", "-I", os.path.join(HERE, "..", "include")]


# The push and the adjoint are compiled per dimension count, order and precision,
# and once more for their dispatch (one compiler takes 20 minutes for all the
# adjoint's; on 8 CPUs the parts take 5)
PARTS = [(src, (dims, order, real)) for src in ("k_adjoint.hip", "k_push.hip") for dims in (3, 2)
         for order in (4, 3, 2, 1) for real in ("double", "float")]
UNITS = PARTS + [(src, None) for src in SOURCES]


def _compile(unit, objdir, verbose):
    src, part = unit
    name, defs = os.path.splitext(src)[0], []
    if part:
        name += "_%d%d%s" % part
        defs = ["-DPIC_DIMS=%d" % part[0], "-DPIC_ORDER=%d" % part[1], "-DPIC_REAL=" + part[2]]
    obj = os.path.join(objdir, name + ".o")
    cmd = [HIPCC] + FLAGS + defs + ["-c", os.path.join(CSRC, src), "-o", obj]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    return obj


# LDS throughput probe (bench.py's LDS peaks; not part of the PIC step)
PROBE_LIB = os.path.join(HERE, "liblds_probe.so")
PROBE_SOURCES = ["lds_probe.hip"]


def _link(objs, out, verbose):
    cmd = [HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", out + ".tmp"] + objs
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    os.replace(out + ".tmp", out)


def build(verbose: bool = False, jobs: int = 8) -> str:
    objdir = os.path.join(HERE, "_build")
    os.makedirs(objdir, exist_ok=True)
    with ThreadPoolExecutor(max_workers=jobs) as ex:
        units = UNITS + [(src, None) for src in PROBE_SOURCES]
        objs = list(ex.map(lambda u: _compile(u, objdir, verbose), units))
    _link(objs[: len(UNITS)], LIB, verbose)
    _link(objs[len(UNITS):], PROBE_LIB, verbose)
    return LIB


if __name__ == "__main__":
    build(verbose="-v" in sys.argv)
