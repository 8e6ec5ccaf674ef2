"""Build libck.so (gfx950) from the HIP sources in csrc/ with hipcc.

Each translation unit is compiled separately (in parallel) and linked into
one shared library next to this file.  Packed FP32 instructions are disabled
for all device code.
"""
import concurrent.futures as cf
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libck.so")
BUILD = os.path.join(HERE, "_build")
SOURCES = ["mech.hip", "k_lane.hip", "k_wave.hip", "k_wide.hip", "k_coop.hip", "api.hip"]
ARCH = os.environ.get("CK_OFFLOAD_ARCH", "gfx950")

# -disable-machine-licm: keeps the backend from hoisting FP64 constants (the exp / log polynomial
# coefficients) and addresses out of the per-reaction loops into long-lived registers; in these
# kernels that hoisting costs far more in register spills and occupancy than it saves.
CFLAGS = ["-O3", "-std=c++17", "-fPIC", f"--offload-arch={ARCH}", "-Wall", "-Wno-unused-function",
          "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-mllvm", "-disable-machine-licm",
          "-I", os.path.join(HERE, "..", "include")]


def _compile(src, verbose):
    obj = os.path.join(BUILD, os.path.splitext(src)[0] + ".o")
    cmd = ["hipcc", "-c", os.path.join(CSRC, src), "-o", obj] + CFLAGS
    if verbose:
        print(" ".join(cmd), flush=True)
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed for {src}:\n{r.stdout}\n{r.stderr}")
    return obj, r.stderr


def build(verbose=False, jobs=None):
    os.makedirs(BUILD, exist_ok=True)
    jobs = jobs or min(len(SOURCES), int(os.environ.get("MAX_JOBS", "8")))
    with cf.ThreadPoolExecutor(jobs) as ex:
        res = list(ex.map(lambda s: _compile(s, verbose), SOURCES))
    objs = [o for o, _ in res]
    tmp = LIB + ".tmp"
    cmd = ["hipcc", "-shared", "-fPIC", f"--offload-arch={ARCH}", "-o", tmp] + objs
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
