"""Build the HIP library liblxw.so (gfx950) in-tree with hipcc."""
import os
import subprocess
import sys
import tempfile
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "liblxw.so")
KERNELS = os.path.join(CSRC, "lxw_kernels.hip")
SOURCES = [KERNELS, os.path.join(CSRC, "lxw_indicator.hip"), os.path.join(CSRC, "lxw_state.hip"),
           os.path.join(CSRC, "lxw_host.cpp")]
N_PARTS = 6  # element configurations: the step kernels are compiled once for each (LXW_PART)
HEADERS = [os.path.join(CSRC, "lxw_internal.hpp"), os.path.join(os.path.dirname(HERE), "include", "lxw.h")]

# Packed FP32 instructions are disabled for all device code (the compiler may otherwise form
# v_pk_* FP32 operations on its own).
FLAGS = ["-O3", "-std=c++17", "--offload-arch=gfx950", "-fPIC",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-Wall", "-Wno-unused-result"]


def build(verbose=False):
    """Compiles every source to an object, side by side, and links them (nothing is reused)."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    jobs = [(KERNELS, [f"-DLXW_PART={p}"]) for p in range(N_PARTS)] + [(s, []) for s in SOURCES if s != KERNELS]

    def run(cmd):
        if verbose:
            print(" ".join(cmd), flush=True)
        subprocess.check_call(cmd)

    with tempfile.TemporaryDirectory() as tmp:
        objs = [os.path.join(tmp, f"{k}.o") for k in range(len(jobs))]
        n = int(os.environ.get("MAX_JOBS", min(8, os.cpu_count() or 1)))
        with ThreadPoolExecutor(max_workers=max(1, n)) as ex:
            list(ex.map(lambda j: run([hipcc] + FLAGS + j[0][1] + ["-c", j[0][0], "-o", j[1]]), zip(jobs, objs)))
        run([hipcc, "--offload-arch=gfx950", "-fPIC", "-shared"] + objs + ["-o", LIB + ".tmp"])
    os.replace(LIB + ".tmp", LIB)
    return LIB


def stale():
    if not os.path.exists(LIB):
        return True
    t = os.path.getmtime(LIB)
    return any(os.path.getmtime(p) > t for p in SOURCES + HEADERS)


if __name__ == "__main__":
    build(verbose="-v" in sys.argv)
