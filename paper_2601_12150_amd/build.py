"""Builds libnsattn.so (hand-written HIP for gfx950) next to this file with hipcc, and _nsbind.so, the native
half of the binding (C++ on torch's headers), with g++."""
from __future__ import annotations

import os
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OBJ = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libnsattn.so")
BIND = os.path.join(HERE, "_nsbind.so")
SOURCES = ["ns_api.hip", "ns_attn_generic.hip", "ns_attn_sweep.hip", "ns_attn_block16.hip", "ns_attn_ragged.hip", "ns_gemm256.hip",
           "ns_gemm128.hip",
           "ns_cls.hip", "ns_topk.hip", "ns_vit.hip", "ns_static.hip"]
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-ffp-contract=off",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",   # keep packed-fp32 VALU ops out
         "-Wall", "-Wno-unused-function", "-Wno-inline-asm"]


def _compile(src: str, extra) -> str:
    obj = os.path.join(OBJ, src.replace(".hip", ".o"))
    cmd = [HIPCC, *FLAGS, *extra, "-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    out = "\n".join(ln for ln in r.stdout.splitlines() if "is not a recognized feature" not in ln)
    if r.returncode != 0:
        raise RuntimeError("hipcc failed for %s:\n%s" % (src, out))
    if out.strip():
        print(out)
    return obj


def _compile_binding() -> str:
    from torch.utils.cpp_extension import include_paths
    import torch
    obj = os.path.join(OBJ, "ns_bind.o")
    inc = [*include_paths(), sysconfig.get_paths()["include"]]
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-fPIC", "-D_GLIBCXX_USE_CXX11_ABI=%d" % torch._C._GLIBCXX_USE_CXX11_ABI,
                           *["-isystem" + i for i in inc], "-c", os.path.join(CSRC, "ns_bind.cpp"), "-o", obj])
    return obj


def _link_binding(obj: str) -> None:
    import torch
    tmp = BIND + ".tmp%d" % os.getpid()
    # (torch's libraries are in the process already when the module is imported; libnsattn.so lies beside it)
    subprocess.check_call(["g++", "-shared", "-o", tmp, obj, "-L" + os.path.join(os.path.dirname(torch.__file__), "lib"),
                           "-ltorch_python", "-ltorch", "-ltorch_cpu", "-lc10", "-L" + HERE, "-l:libnsattn.so",
                           "-Wl,-rpath,$ORIGIN"])
    os.replace(tmp, BIND)


def build(extra_flags=(), verbose: bool = True) -> str:
    """Compile every translation unit and link the shared library.  Always rebuilds."""
    os.makedirs(OBJ, exist_ok=True)
    with ThreadPoolExecutor(max_workers=min(8, len(SOURCES))) as ex:
        bind = ex.submit(_compile_binding)
        objs = list(ex.map(lambda s: _compile(s, list(extra_flags)), SOURCES))
        bind_obj = bind.result()
    tmp = LIB + ".tmp%d" % os.getpid()
    subprocess.check_call([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp, *objs])
    os.replace(tmp, LIB)
    _link_binding(bind_obj)
    if verbose:
        print("built", LIB)
    return LIB


if __name__ == "__main__":
    build(sys.argv[1:])
