"""Builds the HIP library libhipckks.so in-tree for gfx950 with hipcc.

Every source under csrc/ is compiled to an object (in parallel) and linked
into paper_2603_22437_amd/libhipckks.so.  Run it as a script,
`python paper_2603_22437_amd/build.py` (importing it through the package would
first load the library it is about to rebuild).
"""
import concurrent.futures
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
OBJ = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libhipckks.so")
ARCH = os.environ.get("HCK_OFFLOAD_ARCH", "gfx950")

FLAGS = ["-O3", "-std=c++17", "-fPIC", f"--offload-arch={ARCH}",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-Wall", "-Wno-unused-function", "-I", os.path.join(ROOT, "include"), "-I", CSRC]


# compiled once per ring degree, with HCK_LOGN its log2 N
PER_RING = ("ks_fused.hip", "ntt.hip")
RINGS = range(11, 18)


def units():
    """(source, ring or None) of every object, the longest compilations first."""
    names = sorted(f for f in os.listdir(CSRC) if f.endswith((".hip", ".cpp")))
    return ([(f, r) for f in PER_RING for r in reversed(RINGS)] +
            [(f, None) for f in names if f not in PER_RING])


def _compile(unit) -> str:
    name, ring = unit
    src = os.path.join(CSRC, name)
    obj = os.path.join(OBJ, name + (f".{ring}" if ring else "") + ".o")
    lang = ["-x", "hip"] if src.endswith(".hip") else []
    ringed = [f"-DHCK_LOGN={ring}"] if ring else []
    cmd = ["hipcc", *lang, *FLAGS, *ringed, "-c", src, "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed on {src}:\n{r.stdout}\n{r.stderr}")
    return obj


def build(verbose: bool = False) -> str:
    os.makedirs(OBJ, exist_ok=True)
    with concurrent.futures.ThreadPoolExecutor(max_workers=8) as ex:
        objs = list(ex.map(_compile, units()))
    tmp = LIB + ".tmp"
    cmd = ["hipcc", f"--offload-arch={ARCH}", "-shared", "-fPIC", "-o", tmp, *objs,
           "-lpthread"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed:\n{r.stdout}\n{r.stderr}")
    os.replace(tmp, LIB)
    if verbose:
        print(LIB, flush=True)
    return LIB


if __name__ == "__main__":
    build(verbose=True)
    sys.exit(0)
