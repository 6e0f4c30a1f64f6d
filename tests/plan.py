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
    a.B = p[0]; a.Hq = p[1]; a.Hkv = p[2]; a.S = p[3]; a.D = p[4]; a.tile = p[4]; a.causal = p[5]; a.lo_fmt = p[6]; a.per_token = p[7]; a.hi_fmt = p[8];
    return a;
}
extern "C" void dealt_load(const int* p, int rows, int heads_item, int cus, int resident, float step, float item, float* out)
{
    const dma::Load l = dma::dealt_load(args(p), rows, heads_item, cus, resident, step, item);
    out[0] = l.longest;
    out[1] = l.cu;
}
extern "C" int key_split(const int* p, int cus, const int* resident) { return dma::key_split(args(p), cus, resident[0], resident[1], resident[2]); }
extern "C" int unsplit_item(const int* p, int cus) { return (int)dma::unsplit_item(args(p), cus); }
"""


@functools.cache
def library():
    with tempfile.TemporaryDirectory() as d:
        so = os.path.join(d, "plan.so")
        subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-shared", "-fPIC", "-I", B.CSRC, "-x", "c++", "-", "-o", so],
                       input=SHIM, text=True, check=True)
        lib = ctypes.CDLL(so)
    lib.dealt_load.argtypes = [ctypes.POINTER(ctypes.c_int)] + 4 * [ctypes.c_int] + 2 * [ctypes.c_float] + [ctypes.POINTER(ctypes.c_float)]
    return lib


def problem(B, Hq, Hkv, S, D=128, causal=True, lo=2, per_token=False):
    """lo: product-path id of the low format (dma_device.hpp); the high one is 3 (key_split: its own)."""
    return (ctypes.c_int * 9)(B, Hq, Hkv, S, D, int(causal), lo, int(per_token), 3)


def dealt_load(p, rows, heads_item, cus, resident, step, item):
    """(longest list of a workgroup, work of a compute unit)."""
    out = (ctypes.c_float * 2)()
    library().dealt_load(p, rows, heads_item, cus, resident, step, item, out)
    return tuple(out)


def resident(D, lo, hi, per_token=False):
    """Workgroups per CU of the unsplit kernel and of the ones that split keys over two and four waves (lo, hi: product-path
    ids): what the launch asks the runtime for, here as the compiler reports it (test_isa.py holds it against the generated code)."""
    if D == 128:
        return 1, 1, 1                     # more than half of a CU's LDS each
    if lo != hi and hi != 1:               # the decoded 8-bit keys beside the MXFP4 ones: 42 KB of LDS
        return 3, 3, 3
    return (3 if per_token and lo > 2 else 4), 4, 4


def key_split(p, hi=3, cus=256):
    """Waves that share 32 query rows: 1, 2 or 4."""
    p[8] = hi
    return library().key_split(p, cus, (ctypes.c_int * 3)(*resident(p[4], p[6], hi, bool(p[7]))))


ONE_TILE, TWO_TILES, TWO_HEADS = range(3)


def unsplit_item(p, cus=256):
    """What an unsplit item holds: one logical tile, two in a row of a head, or the same tile of two heads."""
    return library().unsplit_item(p, cus)
