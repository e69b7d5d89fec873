"""Compile csrc/*.hip for gfx950 into paper_2604_12452_amd/liblca.so, and binding/bind.cpp into _lcabind.so beside it (in-tree, so they travel with
the tree)."""
from __future__ import annotations

import os
import subprocess
import sys
import warnings
from concurrent.futures import ThreadPoolExecutor

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
OBJ = os.path.join(PKG, "_build")
LIB = os.path.join(PKG, "liblca.so")
BIND_SRC = os.path.join(PKG, "binding", "bind.cpp")
BIND = os.path.join(PKG, "_lcabind.so")       # the binding's marshalling in native code (lca.py does without where it does not load)

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = [
    "-O3", "-std=c++17", "--offload-arch=gfx950", "-fPIC",
    "-I", os.path.join(ROOT, "include"), "-I", CSRC,
    # packed-fp32 instructions are kept out of the generated code on purpose
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function",
]


def sources():
    return sorted(os.path.join(CSRC, f) for f in os.listdir(CSRC) if f.endswith(".hip"))


def _compile(src: str, force: bool) -> str:
    obj = os.path.join(OBJ, os.path.basename(src) + ".o")
    deps = [src] + [os.path.join(CSRC, f) for f in os.listdir(CSRC) if f.endswith(".h")] + [os.path.join(ROOT, "include", "lca.h")]
    if not force and os.path.exists(obj) and all(os.path.getmtime(obj) >= os.path.getmtime(d) for d in deps):
        return obj
    subprocess.run([HIPCC, *FLAGS, "-c", src, "-o", obj], check=True)
    return obj


def _build_binding(force: bool) -> None:
    import sysconfig
    import torch
    from .lca import bind_tag
    tag = bind_tag()
    if not force and os.path.exists(BIND) and all(os.path.getmtime(BIND) >= os.path.getmtime(d) for d in (BIND_SRC, os.path.join(ROOT, "include", "lca.h"))):
        with open(BIND, "rb") as f:
            if tag.encode() + b"\0" in f.read():
                return
    base = os.path.dirname(torch.__file__)
    tmp = BIND + f".{os.getpid()}.tmp"
    subprocess.run(["g++", "-O2", "-std=c++17", "-shared", "-fPIC", "-Wall", f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
                    f'-DLCA_BUILT_FOR="{tag}"', "-I", os.path.join(ROOT, "include"), "-isystem", sysconfig.get_paths()["include"], "-isystem",
                    os.path.join(base, "include"), "-isystem", os.path.join(base, "include", "torch", "csrc", "api", "include"), BIND_SRC, "-o", tmp,
                    "-L", os.path.join(base, "lib"), "-ltorch_python", "-ltorch_cpu", "-lc10"], check=True)
    os.replace(tmp, BIND)


def build(force: bool = False, verbose: bool = True) -> str:
    """Build the library and, where torch, its headers and g++ are there, the binding's native part; without it calls are marshalled in Python."""
    os.makedirs(OBJ, exist_ok=True)
    with ThreadPoolExecutor(max_workers=min(8, len(sources()))) as ex:
        binding = ex.submit(_build_binding, force)
        objs = list(ex.map(lambda s: _compile(s, force), sources()))
    tmp = LIB + f".{os.getpid()}.tmp"
    subprocess.run([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp, *objs], check=True)
    os.replace(tmp, LIB)
    if verbose:
        print(f"built {LIB}")
    try:
        binding.result()
    except (ImportError, OSError, subprocess.CalledProcessError) as e:
        if os.path.exists(BIND):
            os.remove(BIND)                     # (of another source or torch)
        warnings.warn(f"{BIND} was not built, calls are marshalled in Python: {e}", RuntimeWarning)
    return LIB


if __name__ == "__main__":
    build(force="--force" in sys.argv)
