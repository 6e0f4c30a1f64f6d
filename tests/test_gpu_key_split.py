"""A forward with few work items runs on the kernel that splits the keys of a tile over waves; the same problem repeated over a
large batch runs on the unsplit one.  Both form the same probabilities, so they may differ by the order of the binary32 sums
over the keys only: every entry of every repetition is compared, over the formats, masks, windows, scales and lengths that
the split accepts (edges of tiles and of the halves of a tile; odd tile counts; workgroups with a second item).  Which kernel
a call runs on comes from the rule itself (plan.py): every form meets every split that its head dimension has."""
import pytest
import torch

import plan

F = {"bf16": 0, "e4m3": 1, "e2m1": 2, "e5m2": 3}

# D, lo, hi, band, options
FORMS = [
    (128, "e2m1", "e4m3", 2, {}),
    (128, "e2m1", "e4m3", 1, dict(sink_tiles=2)),
    (128, "e2m1", "e4m3", 2, dict(causal=False)),
    (128, "e2m1", "e4m3", 1, dict(causal=False, sink_tiles=1)),
    (128, "e2m1", "e4m3", 2, dict(per_token_scale=True)),
    (128, "e2m1", "e4m3", 2, dict(per_token_scale=True, gran=3)),
    (128, "e2m1", "e4m3", 1, dict(per_token_scale=True, gran=2, causal=False)),
    (128, "e2m1", "e5m2", 9, {}),
    (128, "e2m1", "e4m3", 2, dict(fp8_mfma=True)),
    (128, "e2m1", "e2m1", 0, {}),
    (128, "e4m3", "e4m3", 0, {}),
    (128, "e4m3", "e4m3", 0, dict(causal=False, per_token_scale=True)),
    (128, "e5m2", "e5m2", 0, {}),
    (128, "bf16", "bf16", 0, {}),
    (128, "bf16", "bf16", 0, dict(causal=False)),
    (128, "e4m3", "e4m3", 0, dict(fp8_mfma=True)),
    (128, "e2m1", "e2m1", 0, dict(per_token_scale=True)),
    (128, "e2m1", "e5m2", 1, dict(per_token_scale=True)),
    (128, "e5m2", "e5m2", 0, dict(per_token_scale=True)),
    (64, "e2m1", "e4m3", 1, {}),
    (64, "e2m1", "e4m3", 2, dict(causal=False, sink_tiles=1)),
    (64, "e2m1", "e4m3", 2, dict(per_token_scale=True, gran=3)),
    (64, "e4m3", "e4m3", 0, dict(per_token_scale=True)),
    (64, "bf16", "bf16", 0, {}),
    (64, "e2m1", "e4m3", 2, dict(per_token_scale=True)),
    (64, "e2m1", "e5m2", 1, {}),
    (64, "e2m1", "e2m1", 0, {}),
    (64, "e4m3", "e4m3", 0, dict(fp8_mfma=True)),
]
# heads, kv heads, length: 2 heads take four waves at D = 128, 32 heads two (at S = 613 four with the mask)
SHAPES = {128: [(2, 1, 129), (2, 2, 257), (2, 1, 448), (2, 1, 1100), (32, 8, 613), (32, 8, 1100)],
          64: [(2, 1, 65), (2, 2, 161), (4, 1, 700), (32, 8, 1600)]}


@pytest.mark.gpu
@pytest.mark.parametrize("form", range(len(FORMS)))
def test_split_matches_unsplit(form):
    from paper_2604_03950_amd import binding as dma
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    D, lo, hi, band, options = FORMS[form]
    path = {"bf16": 0, "e4m3": 1 if options.get("fp8_mfma") else 3, "e2m1": 2, "e5m2": 4}
    scaled = bool(options.get("per_token_scale"))
    split = lambda B, Hq, Hkv, S: plan.key_split(
        plan.problem(B, Hq, Hkv, S, D, options.get("causal", True), path[lo], scaled), path[hi])
    splits, second_item = set(), set()             # ... and the ones that dealt a workgroup a second item
    for case, (Hq, Hkv, S) in enumerate(SHAPES[D]):
        waves = split(1, Hq, Hkv, S)
        if waves == 1:
            continue
        splits.add(waves)
        if Hq * -(-S // (256 // waves if D == 128 else 64)) > 256 * plan.resident(D, path[lo], path[hi], scaled)[waves // 2]:
            second_item.add(waves)
        g = torch.Generator(device="cuda").manual_seed(100 * form + case)
        draw = lambda h: torch.randn((1, h, S, D), generator=g, device="cuda")
        q, k, v = draw(Hq), draw(Hkv), draw(Hkv)
        q[..., 5] *= 12
        k[..., 5] *= 15
        q, k, v = (t.to(torch.bfloat16) for t in (q, k, v))
        kw = dict(options)
        gran = kw.pop("gran", None)
        tile = 64 if D == 64 else None

        def forward(q, k, v):
            amax = None
            if gran is not None:
                amax = (dma.dma_mx_group_amax(q, True, gran, tile or 128), dma.dma_mx_group_amax(k, False, gran, tile or 128))
            return dma.dma_attn_fwd(q, k, v, diag_band_tiles=band, lo_fmt=F[lo], hi_fmt=F[hi], tile=tile, group_amax=amax, **kw)

        one = forward(q, k, v)
        pairs = Hq * ((S + 2 * D - 1) // (2 * D))
        reps = 3 * 256 // pairs + 1
        assert split(reps, Hq, Hkv, S) == 1
        many = forward(*(t.repeat(reps, 1, 1, 1) for t in (q, k, v)))
        assert torch.isfinite(one).all()
        # each side is within (additions + 8) units of 2^-24 of the exact sums, relative to the largest |v|
        bound = 2 * (S + 8) * 2.0 ** -24 * float(v.float().abs().max())
        diff = (many - one).abs().amax()
        assert float(diff) <= bound, (FORMS[form], Hq, S, float(diff), bound)
        if S > 2 * D:
            # the two kernels add in different orders: equal bits everywhere would mean that only one of them ran
            assert not torch.equal(many[0], one[0]), (FORMS[form], Hq, S)
    assert splits == ({2, 4} if D == 128 else {2}), splits
    if options.get("causal", True) and (D == 128 or plan.resident(64, path[lo], path[hi], scaled)[1] == 3):
        assert second_item == splits, second_item
