"""The forward for many work items against the oracle: small problems, repeated over the batch until the split rule (plan.py)
leaves the keys of a tile to one wave, as it does at the sizes where the oracle can only follow sampled rows.  Every row of the
first repetition is compared at the bar of the other cases, and every repetition has to agree with the first bit for bit:
what a row's result is made of does not depend on the item's place in the schedule."""
import numpy as np
import pytest
import torch

import parity
import plan
from paper_2604_03950_amd import workloads as wl

PATH = {"bf16": 0, "e4m3": 3, "e2m1": 2, "e5m2": 4}
# D, low, high, band, options (of the binding; gran: granularity of the Step-2 scale)
FORMS = [(D,) + form for D in (128, 64) for form in (
    ("e2m1", "e4m3", 2, {}),
    ("e2m1", "e4m3", 0, {}),
    ("e2m1", "e4m3", 1, dict(sink_tiles=2)),
    ("e2m1", "e4m3", 2, dict(causal=False)),
    ("e2m1", "e4m3", 1, dict(causal=False, sink_tiles=1)),
    ("e2m1", "e4m3", 1, dict(per_token_scale=True)),
    ("e2m1", "e4m3", 1, dict(per_token_scale=True, gran="tensor")),
    ("e2m1", "e4m3", 2, dict(per_token_scale=True, gran="block", causal=False)),
    ("e2m1", "e4m3", 1, dict(pv_mx=True)),
    ("e2m1", "e4m3", 1, dict(pv_mx=True, causal=False)),
    ("e2m1", "e5m2", 1, {}),
    ("e2m1", "e2m1", 0, {}),
    ("e4m3", "e4m3", 0, {}),
    ("e4m3", "e4m3", 0, dict(causal=False, per_token_scale=True)),
    ("e5m2", "e5m2", 0, {}),
    ("bf16", "bf16", 0, {}),
    ("bf16", "bf16", 0, dict(causal=False)),
    ("e2m1", "e4m3", 2, dict(fp8_mfma=True)),
    ("e4m3", "e4m3", 0, dict(fp8_mfma=True)),
)]
# heads, kv heads, tiles (the last one whole or not), what an item holds, items at most (or as many as the split rule wants).
# Two tiles in a row of one head: an odd number of tiles is filled up with one past the end.
SHAPES = [(3, 3, 3, True, plan.TWO_TILES, 0), (1, 1, 4, True, plan.TWO_TILES, 0), (3, 1, 4, False, plan.TWO_TILES, 0),
          (1, 1, 5, False, plan.TWO_TILES, 0), (4, 2, 3, False, plan.TWO_HEADS, 0), (2, 1, 1, False, plan.TWO_HEADS, 0),
          (4, 1, 4, True, plan.TWO_HEADS, 0), (4, 2, 1, True, plan.ONE_TILE, 256), (2, 1, 1, False, plan.ONE_TILE, 256),
          (3, 1, 1, False, plan.ONE_TILE, 256), (4, 2, 3, False, plan.TWO_TILES, 256)]

@pytest.mark.gpu
@pytest.mark.parametrize("form", range(len(FORMS)))
def test_unsplit_against_the_oracle(oracle, form):
    from paper_2604_03950_amd import binding as dma
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    D, lo, hi, band, options = FORMS[form]
    kw = dict(options)
    gran = kw.pop("gran", "token")
    fp8 = kw.get("fp8_mfma", False)
    scaled, causal = kw.get("per_token_scale", False), kw.get("causal", True)
    gpu_fmt = {"bf16": dma.FMT_BF16, "e4m3": dma.FMT_MXFP8_E4M3, "e2m1": dma.FMT_MXFP4_E2M1, "e5m2": dma.FMT_MXFP8_E5M2}
    ref_fmt = {"bf16": oracle.FMT_BF16, "e4m3": oracle.FMT_E4M3, "e2m1": oracle.FMT_E2M1, "e5m2": oracle.FMT_E5M2}
    for case, (Hq, Hkv, tiles, whole, item, few) in enumerate(SHAPES):
        S = tiles * D - (0 if whole else 37)
        reps = few // (Hq * -(-tiles // 2)) or 3 * 256 // (Hq * -(-tiles // 2)) + 1
        if case % 2:                                             # with and without a share of the heads per XCD
            reps += -1 if few else -reps % 8
        if few and tiles > 1 and not (D == 128 and causal):
            continue
        path = [1 if fp8 and f == "e4m3" else PATH[f] for f in (lo, hi)]
        p = plan.problem(reps, Hq, Hkv, S, D, causal, path[0], scaled)
        assert plan.unsplit_item(p) == item and (kw.get("pv_mx") or plan.key_split(p, path[1]) == 1)
        w = wl.small_variant(wl.CONFIGS["prefill_8k" if D == 128 else "tiny"], S=S, Hq=Hq, Hkv=Hkv, seed=100 * form + case)
        bits = wl.generate(w)
        what = f"D={D} Hq={Hq} Hkv={Hkv} S={S} x{reps} {lo}/{hi} band={band} {options}"
        print(what, flush=True)
        q, k, v = (dma.bits_to_bf16_tensor(b).repeat(reps, 1, 1, 1) for b in bits)
        amax = None
        if scaled and gran != "token":
            gid = dma.GRAN_BLOCK if gran == "block" else dma.GRAN_TENSOR
            amax = (dma.dma_mx_group_amax(q, True, gid, D), dma.dma_mx_group_amax(k, False, gid, D))
        out = torch.full((reps, Hq, S, D), float("nan"), dtype=torch.float32, device="cuda")         # unwritten rows stay NaN
        dma.dma_attn_fwd(q, k, v, diag_band_tiles=band, lo_fmt=gpu_fmt[lo], hi_fmt=gpu_fmt[hi], tile=D, group_amax=amax, out=out, **kw)
        assert torch.isfinite(out).all(), what
        assert torch.equal(out, out[:1].expand_as(out)), what
        rows = oracle.all_rows(1, Hq, S)
        okw = dict(tile=D, band=band, hi_fmt=ref_fmt[hi], lo_fmt=ref_fmt[lo], sink=kw.get("sink_tiles", 0), causal=causal,
                   per_token=gran if scaled else False, pv_mx=kw.get("pv_mx", False))
        want = oracle.dma_attn_rows(*bits, rows, **okw)
        got = out[0].cpu().numpy()[rows[:, 1], rows[:, 2]].astype(np.float64)
        if fp8:                                                  # the bar of the native FP8 MFMA (it cuts small products)
            assert np.linalg.norm(got - want) / np.linalg.norm(want) < 2e-2, what
        else:
            parity.compare(got, want, rows, "    result", oracle, bits, okw, max_abs=2e-3, rel_l2=1e-3)
