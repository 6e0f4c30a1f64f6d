"""What this library is timed on: the calls that a program using it makes, over the sizes it makes them at.

``listed()`` names fixed cases, ``draw(rng)`` gives further ones of the same ranges; a case is a plain dict.  Two kinds:

``attn``   one attention forward of a prefill (``dma_attn_fwd``), with the group maxima it needs where the scale of
           Alg. 2 Step 2 has a coarser granularity than the row.  Sequence lengths run from a short prompt to the 32k
           context of the benchmark, whole tiles and ragged ones, with the head counts of the repository's workloads
           (32/32, 32/8, 40/8) and those of a program that keeps a share of the heads on each GPU (8/2, 4/1).
``quant``  the standalone MX quantizer on a Q or K tensor (``dma_mx_quantize``, ``_dual``, ``_token``), from a short
           prompt's keys to the queries of the 8k prefill and beyond.

Inputs follow ``paper_2604_03950_amd/workloads.py``: N(0, 1) with 2 % of the Q / K channels scaled by 10 .. 20, or
Student-t with three degrees of freedom, drawn on the GPU from the seed.
"""
import math

import torch

from paper_2604_03950_amd import binding

FORMATS = {"bf16": binding.FMT_BF16, "e4m3": binding.FMT_MXFP8_E4M3, "e5m2": binding.FMT_MXFP8_E5M2,
           "e2m1": binding.FMT_MXFP4_E2M1}
GRANULARITIES = {"block": binding.GRAN_BLOCK, "tensor": binding.GRAN_TENSOR}


def attn(B, Hq, Hkv, S, D=128, band=2, lo="e2m1", hi="e4m3", causal=True, sink=0, scale="none", values="outliers"):
    """scale: Alg. 2 Step 2 off ("none"), per "token", per "block" (one tile of one head) or per "tensor"."""
    return {"kind": "attn", "B": B, "Hq": Hq, "Hkv": Hkv, "S": S, "D": D, "band": band, "lo": lo, "hi": hi,
            "causal": causal, "sink": sink, "scale": scale, "values": values}


def quant(heads, S, D=128, fmt="dual", query=False, token=False):
    return {"kind": "quant", "heads": heads, "S": S, "D": D, "fmt": fmt, "query": query, "token": token}


def listed():
    cases = [
        # the smallest configuration of the repository (two heads, D = 64): one call is launch latency
        dict(attn(1, 2, 2, 256, D=64, band=1), name="tiny_d64"),
        # a short question to a model with 32 query heads on 8 kv heads; ragged, as prompts are
        dict(attn(1, 32, 8, 613), name="short_prompt"),
        # the short end of long-document prompts (2.5k tokens), same heads, ragged
        dict(attn(1, 32, 8, 2500), name="prompt_2500"),
        # the share of one of eight GPUs in an 8k prefill: few heads, a long sequence
        dict(attn(1, 4, 1, 8192), name="head_shard_8k"),
        # the benchmark's prefill
        dict(attn(1, 32, 32, 8192), name="prefill_8k"),
        # many moderate contexts at once
        dict(attn(8, 32, 32, 4096), name="batched_4k"),
        # the benchmark's long context: the largest
        dict(attn(1, 32, 8, 32768), name="gqa_32k"),
        # every tile in MXFP8 on heavy-tailed values: the accurate setting of the precision comparison
        dict(attn(1, 40, 8, 16384, band=0, lo="e4m3", hi="e4m3", values="student"), name="all_mxfp8_16k"),
        # encoder-style attention with the sink window, ragged
        dict(attn(2, 32, 8, 3000, causal=False, sink=1), name="bidirectional_3000"),
        # the Step-2 scale shared by a whole tensor: group maxima of Q and K, then the forward
        dict(attn(1, 32, 8, 4096, scale="tensor"), name="tensor_scale_4k"),
        # both copies of the 8k prefill's queries from one read
        dict(quant(32, 8192, query=True), name="quantize_dual_8k"),
        # the keys of a short prompt to 4 bits
        dict(quant(8, 613, fmt="e2m1"), name="quantize_short"),
    ]
    return cases


LARGEST_FLOPS = 4.0 * 128 * 32 * 32768 * 32769 / 2
LARGEST_ELEMENTS = 32 * 32768 * 128


def _length(rng, low, high):
    s = int(round(math.exp(rng.uniform(math.log(low), math.log(high)))))
    # a third of the programs pad to whole tiles, the others pass the prompt as it is
    return max(128, s // 128 * 128) if rng.random() < 1 / 3 else s


def draw(rng):
    if rng.random() < 0.2:
        D = rng.choice([64, 128, 128, 256])
        heads = rng.choice([1, 2, 8, 32, 40, 64])
        S = min(_length(rng, 200, 32768), LARGEST_ELEMENTS // (heads * D))
        fmt = rng.choice(["dual", "dual", "e2m1", "e4m3", "e5m2"])
        return quant(heads, S, D, fmt, query=rng.random() < 0.5, token=fmt != "dual" and rng.random() < 0.25)
    D = 64 if rng.random() < 0.2 else 128
    Hq, Hkv = rng.choice([(32, 32), (32, 8), (32, 8), (40, 8), (16, 8), (8, 2), (4, 1)])
    S = _length(rng, 130, 32768 if D == 128 else 8192)
    B = rng.choice([1, 1, 1, 2, 3, 8])
    option = rng.choice(["plain"] * 9 + ["bf16", "e4m3", "e2m1", "e5m2", "sink", "bidirectional", "token", "block", "tensor"])
    band = rng.choice([1, 2, 2, 2, 4, 8])
    values = rng.choice(["outliers", "outliers", "student"])
    case = attn(B, Hq, Hkv, S, D, band, values=values)
    if option in ("bf16", "e4m3", "e2m1"):
        case.update(lo=option, hi=option, band=0)
    elif option == "e5m2":
        case.update(hi="e5m2")
    elif option == "sink":
        case.update(sink=rng.choice([1, 2]))
    elif option == "bidirectional":
        case.update(causal=False)
    elif option in ("token", "block", "tensor"):
        case.update(scale=option)
    # the slower options at no more than the cost of the largest listed case
    budget = LARGEST_FLOPS * (0.5 if option in ("bf16", "e4m3", "token", "block", "tensor") or D == 64 else 0.9)
    while work(case)["flops"] > budget:
        if case["B"] > 1:
            case["B"] = case["B"] // 2
        else:
            case["S"] = int(case["S"] * 0.8)
    return case


def _values(gen, shape, kind):
    """bf16 on the GPU, and the same shape's values before any channel is scaled."""
    x = torch.randn(shape, generator=gen, device="cuda", dtype=torch.float32)
    if kind == "student":
        # Student-t with three degrees of freedom at unit variance: normal / sqrt(chi2_3 / 3) / sqrt(3)
        chi2 = sum(torch.randn(shape, generator=gen, device="cuda", dtype=torch.float32).square_() for _ in range(3))
        x /= chi2.clamp_min_(1e-6).sqrt_()
    return x


def _scale_channels(gen, D):
    """Per-channel factors: 2 % of the channels (rounded up) times 10 .. 20."""
    n = math.ceil(0.02 * D)
    f = torch.ones(D, device="cuda")
    f[torch.randperm(D, generator=gen, device="cuda")[:n]] = 10 + 10 * torch.rand(n, generator=gen, device="cuda")
    return f


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    D = case["D"]
    if case["kind"] == "quant":
        x = _values(gen, (case["heads"], case["S"], D), "outliers") * _scale_channels(gen, D)
        return {"case": case, "x": x.to(torch.bfloat16)}
    B, Hq, Hkv, S = case["B"], case["Hq"], case["Hkv"], case["S"]
    q = _values(gen, (B, Hq, S, D), case["values"])
    k = _values(gen, (B, Hkv, S, D), case["values"])
    if case["values"] == "outliers":
        group = Hq // Hkv
        for h in range(Hkv):
            f = _scale_channels(gen, D)
            q[:, h * group:(h + 1) * group] *= f
            k[:, h] *= f
    v = _values(gen, (B, Hkv, S, D), case["values"])
    return {"case": case, "q": q.to(torch.bfloat16), "k": k.to(torch.bfloat16), "v": v.to(torch.bfloat16)}


def run(state):
    case = state["case"]
    if case["kind"] == "quant":
        if case["fmt"] == "dual":
            return binding.dma_mx_quantize_dual(state["x"], case["query"])
        call = binding.dma_mx_quantize_token if case["token"] else binding.dma_mx_quantize
        return call(state["x"], FORMATS[case["fmt"]], case["query"])
    q, k, v = state["q"], state["k"], state["v"]
    tile = 64 if case["D"] == 64 else None                      # the logical tile that goes with the head dimension
    amax = None
    if case["scale"] in GRANULARITIES:
        gran = GRANULARITIES[case["scale"]]
        amax = (binding.dma_mx_group_amax(q, True, gran, tile or 128), binding.dma_mx_group_amax(k, False, gran, tile or 128))
    out = binding.dma_attn_fwd(q, k, v, diag_band_tiles=case["band"], hi_fmt=FORMATS[case["hi"]], lo_fmt=FORMATS[case["lo"]],
                               causal=case["causal"], tile=tile, sink_tiles=case["sink"],
                               per_token_scale=case["scale"] != "none", group_amax=amax)
    return (out,) if amax is None else (out, *amax)


def work(case):
    D, S = case["D"], case["S"]
    if case["kind"] == "quant":
        elements = case["heads"] * S * D
        bits = {"e2m1": 4, "e4m3": 8, "e5m2": 8, "dual": 12}[case["fmt"]]
        scales = (2 if case["fmt"] == "dual" else 1) * elements // 32
        tokens = 4 * case["heads"] * S if case["token"] else 0
        return {"bytes": 2 * elements + bits * elements // 8 + scales + tokens, "flops": 2 * elements}
    B, Hq, Hkv = case["B"], case["Hq"], case["Hkv"]
    pairs = S * (S + 1) // 2 if case["causal"] else S * S       # (query, key) pairs of one head
    group_maxima = 4 * B * (Hq + Hkv) * S if case["scale"] in GRANULARITIES else 0
    return {"bytes": B * S * D * (Hq * (2 + 4) + 2 * Hkv * 2) + group_maxima, "flops": 4 * D * pairs * B * Hq}


def tolerance(case):
    if case["kind"] == "quant":
        return "exact"                                          # codes and scales have one right answer
    # A probability on a rounding midpoint of bf16 goes either way with the last bit of its binary32 score, and then
    # moves its row by up to 2^-8.  The same forward with the MX blocks of Q and K permuted along D (score products
    # summed in another order) differs by at most 5e-5 and 8e-3 over the listed cases and 24 drawn ones; four times that.
    return {"rel": 2e-4, "max": 3e-2}
