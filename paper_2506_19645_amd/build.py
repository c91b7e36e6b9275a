"""Build libcaat.so (HIP, gfx950 only) in-tree with hipcc.  No torch, no JIT cache."""
from __future__ import annotations

import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OUT = os.path.join(HERE, "libcaat.so")
SOURCES = ["caat_api.hip", "caat_gemm.hip", "caat_gemm_tiles_256x256.hip", "caat_gemm_tiles_192x256.hip",
           "caat_gemm_tiles_256x192.hip", "caat_gemm_tiles_128x128.hip", "caat_gemm_tiles_small.hip",
           "caat_gemm_tiles_split.hip", "caat_gemm_pair_256x256.hip", "caat_gemm_pair_192x256.hip",
           "caat_gemm_pair_128x128.hip", "caat_gemm_pair_small.hip", "caat_gemm_stream.hip",
           "caat_stream.hip", "caat_attn.hip", "caat_decode_attn.hip"]
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Xclang", "-target-feature", "-Xclang",
         "-packed-fp32-ops", "-Wall", "-Wno-unused-function"]


def _compile(src: str) -> str:
    obj = os.path.join(CSRC, src.replace(".hip", ".o"))
    cmd = [HIPCC] + FLAGS + ["-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    err = "\n".join(l for l in r.stderr.splitlines() if "packed-fp32-ops" not in l)
    if r.returncode != 0:
        raise RuntimeError("hipcc failed for %s:\n%s" % (src, err))
    if err.strip():
        sys.stderr.write(err + "\n")
    return obj


def build(verbose: bool = True) -> str:
    with ThreadPoolExecutor(max_workers=8) as ex:
        objs = list(ex.map(_compile, SOURCES))
    r = subprocess.run([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", OUT] + objs,
                       capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("link failed:\n" + r.stderr)
    if verbose:
        print("built", OUT)
    return OUT


if __name__ == "__main__":
    build()
