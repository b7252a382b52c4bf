"""The form of the prefill kernel that a call takes: what the library's own
rule (csrc/prefill_form.hpp, compiled here by itself) says, and what a call
launched."""
import ctypes
import functools
import os
import re
import subprocess
import tempfile

import paper_2602_02071_amd as baps

CSRC = os.path.join(os.path.dirname(baps.__file__), "csrc")
CUS = 256
SETUPS = ("e2e", "default", "exp2", "even", "fp8", "lambda9")
SIZES = ((64, 64), (64, 128), (128, 64), (128, 128))            # head dimension and key block with several forms

_SRC = """#include "prefill_form.hpp"
extern "C" int form(int D, int block, long long Sq, long long Sk, long long group, long long heads, int causal, int fp8,
                    int alg1, int full_table, int ties_even, int ncu)
{
    const baps::PrefillForm f = baps::prefill_form(baps::PrefillShape{D, block, Sq, Sk, group, heads, causal != 0,
        fp8 != 0, alg1 != 0, full_table != 0, ties_even != 0, ncu});
    return 16 * f.nw + f.kw;
}
"""


@functools.lru_cache(maxsize=None)
def _rule():
    with tempfile.TemporaryDirectory() as d:
        src, lib = os.path.join(d, "form.cpp"), os.path.join(d, "form.so")
        with open(src, "w") as f:
            f.write(_SRC)
        subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-shared", "-fPIC", "-I", CSRC, "-o", lib, src],
                       check=True)
        fn = ctypes.CDLL(lib).form
    fn.argtypes = [ctypes.c_int] * 2 + [ctypes.c_longlong] * 4 + [ctypes.c_int] * 6
    return fn


def form_of(shape, block, setup="e2e", cus=CUS):
    """(waves, waves on the same rows) of a call without tile-level restart."""
    B, Hq, Hkv, Sq, Sk, D, causal = shape
    f = _rule()(D, block, Sq, Sk, Hq // Hkv, B * Hkv, int(causal), int(setup == "fp8"),
                int(setup not in ("default", "exp2")), int(setup == "lambda9"), int(setup == "even"), cus)
    return f // 16, f % 16


def forms(size, setup, causal):
    """The forms that the rule picks somewhere for a head dimension and key block."""
    out = [(4, 2), (8, 1)]
    if size == (128, 128):
        out.append((8, 2))
    elif setup in ("e2e", "fp8") and (size != (64, 64) or (setup == "fp8" and causal)):
        out.append((4, 1))
    return out


@functools.lru_cache(maxsize=None)
def shape_for(size, setup, causal, form):
    """The cheapest of a list of ragged shapes that takes a form."""
    cand = [(1, h, h, sq, max(sq, 333), size[0], causal)
            for h in (3, 5, 7, 16, 24, 40, 64, 86, 100, 130, 172, 200, 260, 300, 400, 540)
            for sq in (150, 300, 333, 700, 1024, 2048)]
    cand.sort(key=lambda s: s[1] * s[3] * s[4])
    for s in cand:
        if form_of(s, size[1], setup) == form:
            return s
    return None


def launched(fn):
    """fn()'s result and the names of the library's kernels that it launched."""
    import torch
    torch.cuda.synchronize()
    with torch.profiler.profile(activities=[torch.profiler.ProfilerActivity.CUDA]) as prof:
        out = fn()
        torch.cuda.synchronize()
    return out, [e.name for e in prof.events() if "baps::" in e.name]


def launched_form(names):
    """(D, block, waves, waves on the same rows) of the one prefill kernel among names."""
    keys = [re.search(r"baps_attn_fwd_kernel<(\d+), (\d+), (\d+), (\d+),", n) for n in names]
    keys = [tuple(int(x) for x in m.groups()) for m in keys if m]
    assert len(keys) == 1, names
    return keys[0]
