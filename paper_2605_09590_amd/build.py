"""Build libpico.so (HIP for gfx950) in-tree with hipcc."""
from __future__ import annotations

import concurrent.futures as cf
import os
import shutil
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
OUT = os.path.join(HERE, "libpico.so")
SOURCES = ["cart1d.hip", "cart1d_bf16.hip", "cart1d_split1.hip", "cart1d_split2.hip", "cart1d_split3.hip",
           "gram.hip", "grid2d.hip", "grid2d_bf16.hip", "toeplitz.hip", "kb.hip", "cs.hip", "cs64.hip",
           "tv.hip", "cg.hip", "reduced.hip", "pico_abi.hip", "serve.hip", "tune.hip"]

# Packed FP32 instructions stay off: the build relies on scalar / float2 code
# only, and the compiler must not fuse it into v_pk_* forms.
HIPFLAGS = [
    "--offload-arch=gfx950", "-O3", "-fPIC", "-std=c++17",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-mcode-object-version=5", "-Wno-unused-command-line-argument",
]


def _hipcc() -> str:
    for cand in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", shutil.which("hipcc")):
        if cand and os.path.exists(cand):
            return cand
    raise RuntimeError("hipcc not found")


def _compile(hipcc: str, src: str, obj: str) -> None:
    cmd = [hipcc, *HIPFLAGS, "-I", os.path.join(ROOT, "include"), "-c", src, "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed for {src}:\n{r.stderr[-6000:]}")


def build(verbose: bool = False) -> str:
    """Compile every HIP source for gfx950 and link libpico.so; returns its path."""
    hipcc = _hipcc()
    bdir = os.path.join(HERE, "_build")
    os.makedirs(bdir, exist_ok=True)
    objs = []
    with cf.ThreadPoolExecutor(max_workers=min(len(SOURCES), os.cpu_count() or 1)) as ex:
        futs = []
        for s in SOURCES:
            obj = os.path.join(bdir, os.path.splitext(s)[0] + ".o")
            objs.append(obj)
            futs.append(ex.submit(_compile, hipcc, os.path.join(CSRC, s), obj))
        for f in futs:
            f.result()
    tmp = OUT + ".tmp"
    cmd = [hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", "-pthread", "-o", tmp, *objs]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed:\n{r.stderr[-4000:]}")
    os.replace(tmp, OUT)
    if verbose:
        print("built", OUT)
    return OUT


if __name__ == "__main__":
    build(verbose=True)
