"""Build ``liboctaoctree.so`` for gfx950 with hipcc (in-tree).

Every HIP source is compiled with packed FP32 instructions disabled and with
hardware float atomics enabled, then linked into one shared library next to
this file.
"""
import concurrent.futures as cf
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
OUT = os.path.join(HERE, "liboctaoctree.so")
SOURCES = ["oo_bwd.hip", "oo_query_f32.hip", "oo_query_f16.hip", "oo_query_bf16.hip", "oo_fwd.hip", "oo_mlp.hip",
           "oo_bwd16.hip", "oo_pred.hip", "oo_api.cpp", "oo_sort.hip", "oo_optim.hip", "oo_disp.hip"]
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-munsafe-fp-atomics",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-result", "-Werror=unused-value",
    "-I", os.path.join(ROOT, "include"), "-I", CSRC,
]


def _compile(src, obj, verbose):
    lang = ["-x", "hip"] if src.endswith(".hip") else []
    cmd = [HIPCC] + FLAGS + lang + ["-c", os.path.join(CSRC, src), "-o", obj]
    if verbose:
        print(" ".join(cmd), flush=True)
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed for {src}:\n{r.stderr}")
    return r.stderr


def build(verbose=False):
    bdir = os.path.join(HERE, "_build")
    os.makedirs(bdir, exist_ok=True)
    objs = [os.path.join(bdir, os.path.splitext(s)[0] + ".o") for s in SOURCES]
    with cf.ThreadPoolExecutor(max_workers=len(SOURCES)) as ex:
        for warn in ex.map(lambda so: _compile(so[0], so[1], verbose), zip(SOURCES, objs)):
            if verbose and warn.strip():
                print(warn)
    cmd = [HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", OUT + ".tmp"] + objs
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    os.replace(OUT + ".tmp", OUT)
    return OUT


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
