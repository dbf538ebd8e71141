"""Build libsdattn.so (the C ABI of include/sdattn.h) for gfx950 with hipcc.

Each csrc/*.hip file is compiled separately (in parallel) and linked into a
shared library in the package directory, where the binding loads it.  The
measurement kernels of include/sdattn_probes.h (csrc/probes.hip) go into a
library of their own, libsdattn_probes.so, which only the benchmark loads.
The binding's extension module (csrc/marshal.cpp) is built with g++.
"""
from __future__ import annotations

import concurrent.futures
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
BUILD = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libsdattn.so")
PROBES_LIB = os.path.join(HERE, "libsdattn_probes.so")
PROBE_SOURCES = ["probes.hip"]
MARSHAL = os.path.join(HERE, "_marshal.so")
ARCH = "gfx950"

SOURCES = ["attn_fwd.hip", "attn_fwd_bf16.hip", "attn_fwd_stats.hip", "attn_fwd_short.hip", "attn_fwd_generic.hip", "softmax_rows.hip",
           "twopass.hip", "linear.hip", "norm_act.hip", "winograd.hip",
           "sdattn_api.hip"]

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
CFLAGS = [
    f"--offload-arch={ARCH}", "-O3", "-std=c++17", "-fPIC",
    "-Wall", "-Wno-unused-function",
    "-I", os.path.join(ROOT, "include"), "-I", CSRC,
    # keep the compiler from emitting packed fp32 ops (v_pk_fma_f32 and friends)
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    # matrix-core results in ordinary VGPRs: the softmax reads them directly
    # instead of copying them out of accumulation registers
    "-mllvm", "-amdgpu-mfma-vgpr-form",
]

# Per-file additions.  The short-sequence kernel is latency-bound: its first 14
# argument dwords arrive preloaded in SGPRs instead of through scalar loads.
# The tiled kernel's maxima are of finite scores: without NaNs to honour each
# takes one instruction instead of two.  NaN and infinite inputs still have to come
# out as NaN or Inf: what tests for them does so on bits, and
# tests/test_attn_stream_gpu.py takes them through every path.
_NO_NANS = ["-fno-honor-nans"]
EXTRA_FLAGS = {
    "attn_fwd.hip": _NO_NANS, "attn_fwd_bf16.hip": _NO_NANS, "attn_fwd_stats.hip": _NO_NANS,
    "attn_fwd_short.hip": ["-mllvm", "-amdgpu-kernarg-preload-count=14"],
}


def _compile(src: str, verbose: bool) -> str:
    obj = os.path.join(BUILD, os.path.splitext(src)[0] + ".o")
    cmd = [HIPCC, *CFLAGS, *EXTRA_FLAGS.get(src, []), "-c", os.path.join(CSRC, src), "-o", obj]
    if verbose:
        print(" ".join(cmd), flush=True)
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        sys.stderr.write(r.stdout + r.stderr)
        raise RuntimeError(f"hipcc failed on {src}")
    warn = "\n".join(l for l in r.stderr.splitlines() if "packed-fp32-ops" not in l
                     and "warning: feature flag" not in l and l.strip())
    if warn and verbose:
        sys.stderr.write(warn + "\n")
    return obj


def _link(objs, lib, verbose):
    tmp = lib + ".tmp"
    cmd = [HIPCC, f"--offload-arch={ARCH}", "-shared", "-fPIC", "-o", tmp, *objs]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    os.replace(tmp, lib)


def _build_marshal(verbose: bool) -> None:
    """The binding's extension module (csrc/marshal.cpp), against this Python's torch."""
    import sysconfig

    import torch
    from torch.utils import cpp_extension
    tdir = os.path.join(os.path.dirname(torch.__file__), "lib")
    tmp = MARSHAL + ".tmp"
    cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-fvisibility=hidden", "-Wall",
           f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
           "-I", sysconfig.get_paths()["include"]]
    for inc in cpp_extension.include_paths():
        cmd += ["-isystem", inc]
    cmd += [os.path.join(CSRC, "marshal.cpp"), "-o", tmp, "-L", tdir, "-lc10", "-ltorch_cpu", "-ltorch_python"]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    os.replace(tmp, MARSHAL)


def build(verbose: bool = False) -> str:
    os.makedirs(BUILD, exist_ok=True)
    srcs = SOURCES + PROBE_SOURCES
    with concurrent.futures.ThreadPoolExecutor(max_workers=len(srcs) + 1) as ex:
        marshal = ex.submit(_build_marshal, verbose)
        objs = list(ex.map(lambda s: _compile(s, verbose), srcs))
        marshal.result()
    _link(objs[:len(SOURCES)], LIB, verbose)
    _link(objs[len(SOURCES):], PROBES_LIB, verbose)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
