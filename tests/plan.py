"""The host rule that plans a forward (csrc/dma_plan.hpp, plain C++), compiled with the host compiler for the tests: which
kernel a call runs on, without a GPU."""
import ctypes
import functools
import os
import subprocess
import tempfile

from paper_2604_03950_amd import build as B

SHIM = r"""
#include "dma_plan.hpp"
static dma::AttnArgs args(const int* p)
{
    dma::AttnArgs a = {};
    a.B = p[0]; a.Hq = p[1]; a.Hkv = p[2]; a.S = p[3]; a.D = p[4]; a.tile = p[4]; a.causal = p[5]; a.lo_fmt = p[6]; a.per_token = p[7];
    return a;
}
extern "C" float longest_list(const int* p, int rows, int heads_item, int slots, float step, float item)
{
    return dma::longest_list(args(p), rows, heads_item, slots, step, item);
}
extern "C" int key_split(const int* p, int cus) { return dma::key_split(args(p), cus); }
"""


@functools.cache
def library():
    with tempfile.TemporaryDirectory() as d:
        so = os.path.join(d, "plan.so")
        subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-shared", "-fPIC", "-I", B.CSRC, "-x", "c++", "-", "-o", so],
                       input=SHIM, text=True, check=True)
        lib = ctypes.CDLL(so)
    lib.longest_list.restype = ctypes.c_float
    lib.longest_list.argtypes = [ctypes.POINTER(ctypes.c_int), ctypes.c_int, ctypes.c_int, ctypes.c_int, ctypes.c_float, ctypes.c_float]
    return lib


def problem(B, Hq, Hkv, S, D=128, causal=True, lo=2, per_token=False):
    """lo: product-path id of the low format (dma_device.hpp)."""
    return (ctypes.c_int * 8)(B, Hq, Hkv, S, D, int(causal), lo, int(per_token))


def key_split(p, cus=256):
    """Waves that share 32 query rows: 1, 2 or 4."""
    return library().key_split(p, cus)
