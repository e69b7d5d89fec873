"""Which kernels a call launches, seen on the CPU: the library's objects linked with tests/launch_trace.cpp instead of with
the HIP runtime.  Arguments are addresses that nothing reads."""
import ctypes
import os
import subprocess
import tempfile
from collections import namedtuple

from paper_2604_12452_amd import build, lca

Launch = namedtuple("Launch", "kernel grid block lds")
_lib = None


def _load():
    global _lib
    if _lib is None:
        objs = [os.path.join(build.OBJ, os.path.basename(s) + ".o") for s in build.sources()]
        if not all(os.path.exists(o) for o in objs):
            build.build(verbose=False)
        with tempfile.TemporaryDirectory() as tmp:
            so = os.path.join(tmp, "traced.so")
            here = os.path.dirname(os.path.abspath(__file__))
            subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-Wl,-Bsymbolic", "-o", so, os.path.join(here, "launch_trace.cpp"),
                            *objs], check=True)
            _lib = ctypes.CDLL(so)
        _lib.trace_mla_params.restype = ctypes.POINTER(ctypes.c_int32 * 28)
        _lib.trace_log.restype = _lib.lca_last_error.restype = ctypes.c_char_p
        lca.load()
        for name in lca.EXPORTS:
            getattr(_lib, name).argtypes = getattr(lca.load(), name).argtypes
    return _lib


def launches(name: str, desc, *rest):
    """The launches of entry point `name` with this descriptor; `rest`: its other arguments (a CacheLayout among them may be given as it
    is)."""
    lib = _load()
    lib.trace_reset()
    cd = desc.c()
    args = [ctypes.byref(a.c()) if isinstance(a, lca.CacheLayout) else a for a in rest]
    status = getattr(lib, name)(ctypes.byref(cd), *args)
    assert status == lca.OK, lib.lca_last_error().decode()
    return [Launch(k, int(g), int(b), int(s)) for k, g, b, s in (line.split("\t") for line in lib.trace_log().decode().splitlines())]


A = 0x10000          # an address: aligned, not NULL, never read
WS = (A, 1 << 40)    # workspace and a size that is enough for any descriptor


def prefill(desc, dense=False, up=False):
    if dense:
        return launches("dense_mla_attn", desc, A, A, A, A, None, *WS, None)
    if up:
        return launches("lca_prefill_attn_up", desc, *[A] * 7, None, *WS, None)
    return launches("lca_prefill_attn", desc, *[A] * 6, None, *WS, None)


def condense(desc):
    return launches("lca_condense", desc, *[A] * 6, None, *WS, None)


def decode(desc, q8=False):
    return launches("lca_decode_attn_q8", desc, None, *[A] * 7, *WS, None) if q8 else launches("lca_decode_attn", desc, *[A] * 6, *WS, None)


def cache_update(desc):
    return launches("lca_cache_update", desc, lca.CacheLayout(desc.m, desc.w + desc.g), *[A] * 6, *WS, None)


def mla_items(desc, **kw):
    """(query blocks per sequence, log2 of the query blocks an XCD takes at a time, log2 of the heads of a work item) of the MLA prefill launch:
    the numbers behind the descriptor's sizes in the kernel's parameter block."""
    prefill(desc, **kw)
    words = list(_load().trace_mla_params().contents)
    sizes = [desc.B, desc.L, desc.H, desc.S, desc.g, desc.w, desc.m, 0]
    (at,) = [i + len(sizes) for i in range(len(words) - len(sizes)) if words[i:i + len(sizes)] == sizes]
    return tuple(words[at:at + 3])
