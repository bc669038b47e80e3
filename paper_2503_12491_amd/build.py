"""Compile libcake.so for gfx950 with hipcc.  `python -m paper_2503_12491_amd.build`."""
from __future__ import annotations

import os
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
OBJ_DIR = os.path.join(ROOT, "_build")
LIB_PATH = os.path.join(PKG, "libcake.so")

SOURCES = ["cake_host.cpp", "window_scores.hip", "scores_stream.hip", "select_topk.hip", "compact_kv.hip", "decode_update.hip", "plan_evict.hip",
           "quantize_kv.hip", "pass_run.hip", "cascade_stage.hip"]
# the package's host module: Python and torch headers, no device code, linked to libcake.so beside it
HOST_SRC = os.path.join(CSRC, "host_module.cpp")
HOST_PATH = os.path.join(PKG, "_host.so")
# standalone issue-rate microbenchmark (not part of the library): `python -m paper_2503_12491_amd.build --microbench`
MICROBENCH_SRC = os.path.join(CSRC, "microbench", "issue_port.hip")
MICROBENCH_PATH = os.path.join(PKG, "issue_port_microbench")

COMMON = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    "-I", os.path.join(ROOT, "include"), "-I", CSRC,
    # packed fp32 VALU ops stay off for all device code
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function",
]


def _hipcc() -> str:
    for cand in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", "hipcc"):
        if cand and (os.path.isabs(cand) and os.path.exists(cand) or not os.path.isabs(cand)):
            return cand
    raise RuntimeError("hipcc not found")


def _compile(src: str, verbose: bool) -> str:
    obj = os.path.join(OBJ_DIR, os.path.splitext(src)[0] + ".o")
    cmd = [_hipcc(), *COMMON, "-c", os.path.join(CSRC, src), "-o", obj]
    if src.endswith(".cpp"):
        cmd += ["-ffp-contract=off"]   # host arithmetic of the allocator: no fused multiply-add
    res = subprocess.run(cmd, capture_output=True, text=True)
    noise = "is not a recognized feature for this target"
    err = "\n".join(l for l in res.stderr.splitlines() if noise not in l)
    if res.returncode != 0:
        raise RuntimeError(f"hipcc failed on {src}:\n{err}")
    if verbose and err.strip():
        print(err, file=sys.stderr)
    return obj


def _compile_host() -> str:
    import torch
    root = os.path.dirname(torch.__file__)
    obj = os.path.join(OBJ_DIR, "host_module.o")
    cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-c", HOST_SRC, "-o", obj, "-I", os.path.join(ROOT, "include"), "-I", CSRC,
           "-I", os.path.join(root, "include"), "-I", os.path.join(root, "include", "torch", "csrc", "api", "include"),
           "-I", sysconfig.get_paths()["include"], f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}"]
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError(f"g++ failed on host_module.cpp:\n{res.stderr}")
    return obj


def _link_host(obj: str) -> None:
    import torch
    lib = os.path.join(os.path.dirname(torch.__file__), "lib")
    cmd = ["g++", "-shared", "-o", HOST_PATH + ".tmp", obj, "-L", PKG, "-lcake", "-Wl,-rpath,$ORIGIN", "-L", lib,
           "-ltorch_python", "-ltorch", "-ltorch_cpu", "-lc10"]
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError(f"link of the host module failed:\n{res.stderr}")
    os.replace(HOST_PATH + ".tmp", HOST_PATH)


def build(verbose: bool = False) -> str:
    """Compile every source and link paper_2503_12491_amd/libcake.so and the host module.  Returns the library's path."""
    os.makedirs(OBJ_DIR, exist_ok=True)
    with ThreadPoolExecutor(max_workers=6) as ex:
        host = ex.submit(_compile_host)
        objs = list(ex.map(lambda s: _compile(s, verbose), SOURCES))
    cmd = [_hipcc(), "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB_PATH + ".tmp", *objs]
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError(f"link failed:\n{res.stderr}")
    os.replace(LIB_PATH + ".tmp", LIB_PATH)
    _link_host(host.result())
    return LIB_PATH


def build_microbench() -> str:
    """Compile the issue-rate microbenchmark into paper_2503_12491_amd/issue_port_microbench."""
    cmd = [_hipcc(), "--offload-arch=gfx950", "-O3", "-std=c++17", "-Xclang", "-target-feature", "-Xclang",
           "-packed-fp32-ops", MICROBENCH_SRC, "-o", MICROBENCH_PATH]
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError(f"hipcc failed on the microbenchmark:\n{res.stderr}")
    return MICROBENCH_PATH


if __name__ == "__main__":
    print(build(verbose=True))
    if "--microbench" in sys.argv[1:]:
        print(build_microbench())
