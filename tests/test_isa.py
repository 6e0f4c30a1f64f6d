"""Checks on the generated gfx950 code (no GPU needed: hipcc cross-compiles).

The packed-bf16 FP4 convert of the K staging takes its four source dwords out of one 128-bit load tuple.  One shape of
that code made the compiler name the tuple's first register in all four converts (wrong codes, caught by the parity
tests at the time); this test pins the generated code: every group of four converts into one destination reads four
different source registers.  (The compiler is the image's; the check guards edits of the source.)
The same listing must hold no packed binary32 arithmetic: the library is built with those forms switched off.
"""
import functools
import os
import re
import subprocess
import tempfile

import pytest

import plan
from paper_2604_03950_amd import build as B


@functools.cache
def listing(lo, hi):
    """Generated code of one pair of formats."""
    flags = [f for f in B.HIPCC_FLAGS if f != "-fPIC"]
    with tempfile.TemporaryDirectory() as d:
        out = os.path.join(d, "inst.s")
        subprocess.run(["hipcc"] + flags + [f"-DDMA_LO={lo}", f"-DDMA_HI={hi}", "-S", "--cuda-device-only", "-o", out,
                                            os.path.join(B.CSRC, "dma_attn_inst.hip")],
                       check=True, stdout=subprocess.DEVNULL, stderr=subprocess.DEVNULL)
        return open(out).read()


def resources(lo, hi, kernel):
    """What the instances of a kernel hold, by their template arguments."""
    counts = {}
    for block in re.split(r"(?=- \.agpr_count)", listing(lo, hi)):
        name = re.search(rf"\.name:\s+(_ZN3dma\d+{kernel}I\S+)", block)
        if name:
            key = tuple(int(n) for n in re.findall(r"L[ib](\d+)E", name.group(1)))
            counts[key] = {f: int(re.search(rf"\.{f}:\s+(\d+)", block).group(1))
                           for f in ("vgpr_count", "vgpr_spill_count", "sgpr_spill_count", "group_segment_fixed_size", "max_flat_workgroup_size")}
    return counts


@pytest.mark.parametrize("lo,hi", [(2, 3), (2, 1), (2, 4), (2, 2)])      # every pair whose low format is MXFP4
def test_fp4_convert_groups_read_four_registers(lo, hi):
    text = listing(lo, hi)
    # the build flags keep the packed binary32 add / multiply / fused multiply-add forms out of the generated code
    assert not re.search(r"\bv_pk_(add|mul|fma)_f32\b", text)
    lines = [ln.strip() for ln in text.splitlines() if "v_cvt_scalef32_pk_fp4_bf16" in ln]
    assert len(lines) >= 16 and len(lines) % 4 == 0
    # The four converts into one destination dword fill its bytes in order (op_sel of the destination byte); the
    # scheduler may interleave the groups of different destinations, so the groups are collected per destination.
    want_sel = ["", "[0,0,1,0]", "[0,0,0,1]", "[0,0,1,1]"]
    open_groups, n_groups = {}, 0
    for ln in lines:
        ops = ln.split()
        dst, src = ops[1].rstrip(","), ops[2].rstrip(",")
        sel = re.search(r"op_sel:(\[[0-9,]+\])", ln).group(1) if "op_sel" in ln else ""
        grp = open_groups.setdefault(dst, [])
        assert sel == want_sel[len(grp)], (dst, grp, ln)     # the next byte of this destination, nothing else
        grp.append(src)
        if len(grp) == 4:
            assert len(set(grp)) == 4, (dst, grp)            # four different source registers
            del open_groups[dst]
            n_groups += 1
    assert not open_groups and n_groups == len(lines) // 4


def test_instances_keep_their_registers():
    """What the instances of the default pair hold in registers.  A value that lives through the tile loops for the sake of a
    rare shape (the filled-up tile of an odd number of tiles) is paid for by every length: in spilled scalar registers, which
    are moved to and from vector lanes, and in vector registers.  The limits on the general instances with two tiles
    per workgroup lie between the counts with one bound per wave (0, 0, 2 and 3 spilled SGPRs) and with a flag and a
    second test beside it (7, 7, 10 and 11)."""
    # (D, tile, tiles per workgroup, low, high, general, per-token scale, MX-format P V)
    for key, c in resources(2, 3, "dma_attn_fwd_kernel").items():
        D, _, tpw, _, _, general, per_token, pv_mx = key
        spilled = 21 if per_token else 6 if general and pv_mx else 3 if general else 0
        assert c["sgpr_spill_count"] <= spilled, (key, c)
        # only the MX-format P V spills vector registers
        assert c["vgpr_spill_count"] <= (16 if pv_mx else 0), (key, c)
        if D == 128 and tpw == 2 and not pv_mx:
            assert c["vgpr_count"] <= (250 if per_token else 238), (key, c)
    # (D, tile, waves per 32 query rows, low, high, per-token scale)
    for key, c in resources(2, 3, "dma_attn_split_kernel").items():
        D, _, waves, _, _, per_token = key
        assert c["sgpr_spill_count"] <= (15 if per_token else 0) and c["vgpr_spill_count"] == 0, (key, c)
        assert c["vgpr_count"] <= ({2: 225, 4: 214}[waves] if D == 128 else 134), (key, c)


@pytest.mark.parametrize("lo,hi", B.ATTN_PAIRS)
def test_instances(lo, hi):
    """What a pair is built as: the workgroups of the forward kernels that share a CU (512 registers per lane and SIMD in steps
    of 8, 160 KB of LDS in steps of 1280 bytes), which the tests of the split rule have in a table; and no instance that no call
    reaches."""
    def fits(c):
        waves = c["max_flat_workgroup_size"] // 64
        return min(512 // (-(-c["vgpr_count"] // 8) * 8) * 4 // waves, 160 * 1024 // (-(-c["group_segment_fixed_size"] // 1280) * 1280))

    seen = 0
    for (D, _, tpw, _, _, general, per_token, pv_mx), c in resources(lo, hi, "dma_attn_fwd_kernel").items():
        if tpw == 2 and not pv_mx:
            assert fits(c) == plan.resident(D, lo, hi, per_token)[0], (D, general, per_token, c)
            seen += 1
    for (D, _, ks, _, _, per_token), c in resources(lo, hi, "dma_attn_split_kernel").items():
        assert fits(c) == plan.resident(D, lo, hi, per_token)[{2: 1, 4: 2}[ks]], (D, ks, per_token, c)
        seen += 1
    assert seen >= 7
    # the pairs on the native FP8 MFMA refuse the Step-2 scale, unquantized operands have none: no instances for either
    scaled = [k for k in resources(lo, hi, "dma_attn_fwd_kernel") if k[6]] + [k for k in resources(lo, hi, "dma_attn_split_kernel") if k[5]]
    assert bool(scaled) == (lo != 0 and hi != 1), scaled


@pytest.mark.parametrize("lo,hi", [(2, 3), (2, 4), (3, 3), (4, 4)])      # every pair with keys decoded from 8 bits
def test_no_matrix_instruction_while_converts_saturate(lo, hi):
    """MODE.FP16_OVFL ends with the keys' converts to 8 bits: in it the matrix instructions turn NaN and infinities into numbers.  No
    other convert or 16-bit arithmetic may move in but the converts back to bf16, which the mode leaves alone."""
    on = sections = 0
    for ln in listing(lo, hi).splitlines():
        m = re.match(r"\s+s_setreg_imm32_b32 hwreg\(HW_REG_MODE, 23, 1\), ([01])", ln)
        if m:
            assert int(m.group(1)) != on, ln
            on = int(m.group(1))
            sections += on
        if on:
            assert not re.match(r"\s+(v_mfma|s_cbranch|s_branch|s_endpgm|s_barrier|v_\w+_f16|v_cvt_(?!scalef32_pk_((fp8|bf8)_bf16|bf16_(fp8|bf8))))", ln), ln
        assert on or not re.match(r"\s+v_cvt_scalef32_pk_(fp8|bf8)_bf16", ln), ln
    assert on == 0 and sections
