"""Build the native parts in-tree: libhgrn2.so (the C-ABI library of hand-written gfx950 kernels, with
hipcc) and _host.so (the binding's native call path, plain C++ against torch's headers).

hipcc cross-compiles for gfx950 without a GPU.  Usage: ``python -m paper_2404_07904_amd.build``.
"""
from __future__ import annotations

import os
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OBJ = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libhgrn2.so")
HOST = os.path.join(HERE, "_host.so")
SOURCES = ["api.hip", "sweep.hip", "fwd_out.hip", "fwd_fused.hip", "bwd_grad.hip", "bwd_walk.hip", "step.hip", "hgrn1.hip", "varlen.hip", "domain.hip", "probe.hip", "proj.hip"]
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Wall", "-Wno-unused-function",
         # keep the compiler from forming packed-fp32 VALU instructions
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]


def _run(cmd, what: str) -> None:
    r = subprocess.run(cmd, capture_output=True, text=True)
    msgs = "\n".join(l for l in (r.stdout + r.stderr).splitlines()
                     if "packed-fp32-ops" not in l and l.strip())
    if r.returncode != 0:
        raise RuntimeError("compiling %s failed:\n%s" % (what, msgs))
    if msgs:
        sys.stderr.write(msgs + "\n")


def _compile(src: str, extra) -> str:
    obj = os.path.join(OBJ, src.replace(".hip", ".o"))
    _run(["hipcc", *FLAGS, *extra, "-c", os.path.join(CSRC, src), "-o", obj], src)
    return obj


def _compile_host() -> str:
    import torch
    root = os.path.dirname(torch.__file__)
    obj = os.path.join(OBJ, "host.o")
    inc = [os.path.join(root, "include"), os.path.join(root, "include", "torch", "csrc", "api", "include"),
           sysconfig.get_paths()["include"], "/opt/rocm/include"]
    _run(["g++", "-O2", "-std=c++17", "-fPIC", "-Wall", "-DUSE_ROCM", "-D__HIP_PLATFORM_AMD__",
          "-D_GLIBCXX_USE_CXX11_ABI=%d" % int(torch._C._GLIBCXX_USE_CXX11_ABI),
          *["-isystem" + d for d in inc], "-c", os.path.join(CSRC, "host.cpp"), "-o", obj], "host.cpp")
    return obj


def _link(out: str, cmd) -> None:
    tmp = out + ".tmp%d" % os.getpid()
    subprocess.check_call([*cmd, "-o", tmp])
    os.replace(tmp, out)


def build(extra_flags=(), jobs: int = 7) -> str:
    import torch
    os.makedirs(OBJ, exist_ok=True)
    with ThreadPoolExecutor(max_workers=jobs) as ex:
        host = ex.submit(_compile_host)
        objs = list(ex.map(lambda s: _compile(s, list(extra_flags)), SOURCES))
        host_obj = host.result()
    _link(LIB, ["hipcc", "--offload-arch=gfx950", "-shared", "-fPIC", "-Wl,-soname,libhgrn2.so", *objs])
    # (torch's libraries are loaded by the interpreter before _host.so is; libhgrn2.so lies next to it)
    _link(HOST, ["g++", "-shared", "-fPIC", host_obj, "-L" + HERE, "-lhgrn2", "-Wl,-rpath,$ORIGIN",
                 "-L" + os.path.join(os.path.dirname(torch.__file__), "lib"), "-ltorch_python", "-ltorch_cpu", "-ltorch_hip", "-lc10",
                 "-lc10_hip"])
    return LIB


if __name__ == "__main__":
    print(build(sys.argv[1:]))
