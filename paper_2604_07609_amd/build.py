"""Compiles libblink.so (HIP, gfx950) in-tree. Run as `python -m paper_2604_07609_amd.build`."""
import glob
import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
LIB = os.path.join(HERE, "libblink.so")
CSRC = os.path.join(HERE, "csrc")
OBJ = os.path.join(HERE, "_build")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]


def sources():
    return [os.path.join(CSRC, "blink.hip")] + sorted(glob.glob(os.path.join(CSRC, "kernels", "*.hip")))


def run(cmd, verbose):
    if verbose:
        print(" ".join(cmd), flush=True)
    r = subprocess.run(cmd, capture_output=True, text=True)
    err = "\n".join(l for l in r.stderr.splitlines() if "packed-fp32-ops" not in l)
    if r.returncode != 0:
        raise RuntimeError("hipcc failed:\n" + r.stdout + err)
    if verbose and err.strip():
        print(err)


def build(verbose=True):
    """Compiles every source (the kernels in parallel) and links the library."""
    os.makedirs(OBJ, exist_ok=True)
    objs = {s: os.path.join(OBJ, os.path.splitext(os.path.basename(s))[0] + ".o") for s in sources()}
    with ThreadPoolExecutor(max_workers=min(8, os.cpu_count() or 1)) as pool:
        list(pool.map(lambda s: run([HIPCC] + FLAGS + ["-c", "-o", objs[s], s], verbose), objs))
    run([HIPCC] + FLAGS + ["-shared", "-o", LIB] + list(objs.values()) + ["-lpthread"], verbose)
    return LIB


if __name__ == "__main__":
    build()
    sys.exit(0)
