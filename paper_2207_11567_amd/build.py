"""Builds liblbm.so (the HIP/gfx950 library behind include/lbm.h) in-tree with hipcc.

Usage: python -m paper_2207_11567_amd.build   (or build() from Python).
Compiles every translation unit under csrc/ in parallel into _build/ and links the
shared library next to this file.  The step's instances, most of the work, are one object
per lattice, precision and number of scalars (generated units that instantiate
launch_one), which the dispatching units only refer to: about 2 minutes on 8 cores instead
of 5 with an object per precision.  Always recompiles.
"""
import concurrent.futures as cf
import os
import subprocess
import sys

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
BUILD = os.path.join(ROOT, "_build")
LIB = os.path.join(PKG, "liblbm.so")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
ARCH = "gfx950"

FLAGS = ["-std=c++17", "-O3", f"--offload-arch={ARCH}", "-fPIC",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-I", os.path.join(ROOT, "include")]

UNITS = ["lbm_capi.hip", "lbm_d2q9.hip", "lbm_d3q27.hip", "lbm_adjoint.hip"]

_ARGS = "(int, const StepArgs &, int, hipStream_t, const double *, const double *, const double *)"


def _instances():
    """Paths of the generated instance units, the longest compilations first; writes them and the
    header that declares them to the dispatching units to _build/."""
    combos = [(q, p, n) for n in (6, 2, 1, 0) for q in (27, 9) for p in (0, 2, 1)]
    head = f'#include "{CSRC}/lbm_launch.hpp"\n'

    def body(word):
        return "".join(f"{word} hipError_t launch_one<{q}, {p}, {n}>{_ARGS};\n" for q, p, n in combos)

    with open(os.path.join(BUILD, "instances.hpp"), "w") as f:
        f.write("#pragma once\n" + head + "namespace lbm {\n" + body("extern template") + "}\n")
    units = []
    for q, p, n in combos:
        units.append(os.path.join(BUILD, f"step_{q}_{p}_{n}.hip"))
        with open(units[-1], "w") as f:
            f.write(head + f"namespace lbm {{ template hipError_t launch_one<{q}, {p}, {n}>{_ARGS}; }}\n")
    return units


def _compile(src):
    obj = os.path.join(BUILD, os.path.basename(src).replace(".hip", ".o"))
    cmd = [HIPCC] + FLAGS + ["-c", src, "-o", obj]
    if os.path.basename(src) in ("lbm_d2q9.hip", "lbm_d3q27.hip"):
        cmd += ["-include", os.path.join(BUILD, "instances.hpp")]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed for {src}:\n{r.stderr}")
    return obj


def build(verbose=True):
    os.makedirs(BUILD, exist_ok=True)
    units = _instances() + [os.path.join(CSRC, u) for u in UNITS]
    workers = min(len(units), max(1, min(8, os.cpu_count() or 1)))
    with cf.ThreadPoolExecutor(workers) as ex:
        objs = list(ex.map(_compile, units))
    tmp = LIB + ".tmp"
    cmd = [HIPCC, "-shared", "-fPIC", f"--offload-arch={ARCH}", "-o", tmp] + objs
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed:\n{r.stderr}")
    os.replace(tmp, LIB)
    if verbose:
        print(f"built {LIB}")
    return LIB


if __name__ == "__main__":
    build()
    sys.exit(0)
