"""What the forward makes of the keys on their way to LDS, against the oracle's quantizer: quantizing is idempotent, so the
forward on K and on the oracle's decoded K must agree bit for bit.  The keys cover what a staging can get wrong: block
maxima on both sides of the largest element (1.75 of a binade, where the element is clamped), every bf16 mantissa and
sign, ties, zeros and zero blocks, elements that underflow, blocks of very different scale next to each other."""
import numpy as np
import pytest
import torch

import plan

FMTS = {"e4m3": 1, "e2m1": 2, "e5m2": 3}


def keys(rng, S, D):
    """bf16 patterns [1, 2, S, D]."""
    mant = rng.integers(0, 128, (2, S, D))
    expo = 127 - rng.geometric(0.35, (2, S, D)) + np.repeat(rng.integers(-5, 2, (2, S, D // 32)), 32, axis=-1)
    bits = ((rng.integers(0, 2, (2, S, D)) << 15) | (expo << 7) | mant).astype(np.uint16)
    blocks = bits.reshape(2, S, D // 32, 32)
    top = blocks[..., 0]                                                   # block maxima with every mantissa in turn
    top[...] = (top & 0x8000) | ((127 + 2) << 7) | (np.arange(top.size).reshape(top.shape) % 128)
    blocks[:, ::7, 0] = 0                                                  # zero blocks, and negative zeros
    blocks[:, ::7, 0, 1] = 0x8000
    blocks[:, 1::9, -1] &= 0x807F                                          # subnormal bf16 only
    return blocks.reshape(1, 2, S, D)


@pytest.mark.gpu
@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("fmt", ["e4m3", "e5m2", "e2m1"])
@pytest.mark.parametrize("reps", [1, 400])          # few items (keys split over waves) and many
def test_forward_sees_the_oracles_keys(oracle, D, fmt, reps):
    from paper_2604_03950_amd import binding as dma
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    f = {"e4m3": oracle.FMT_E4M3, "e5m2": oracle.FMT_E5M2, "e2m1": oracle.FMT_E2M1}[fmt]
    S = 3 * D + 37
    rng = np.random.default_rng(D)
    k = keys(rng, S, D)
    codes, scales = oracle.mx_quantize(k.reshape(-1, D), f, False)
    decoded = np.asarray(oracle.mx_dequantize(codes, scales, f)).astype(np.float32)
    seen = (decoded.view(np.uint32) >> 16).astype(np.uint16).reshape(k.shape)
    assert np.array_equal((seen.astype(np.uint32) << 16).view(np.float32).reshape(decoded.shape), decoded)      # a bf16 each
    g = torch.Generator(device="cuda").manual_seed(D)
    q = torch.randn((1, 4, S, D), generator=g, device="cuda").to(torch.bfloat16)
    v = torch.randn((1, 2, S, D), generator=g, device="cuda").to(torch.bfloat16)

    def forward(bits):
        kd = dma.bits_to_bf16_tensor(bits)
        q_, k_, v_ = (t.repeat(reps, 1, 1, 1) for t in (q, kd, v))
        return dma.dma_attn_fwd(q_, k_, v_, diag_band_tiles=0, lo_fmt=FMTS[fmt], hi_fmt=FMTS[fmt], tile=64 if D == 64 else None)

    a, b = forward(k), forward(seen)
    assert torch.isfinite(a).all()
    assert torch.equal(a, b)
    assert not torch.equal(a, forward(k ^ 0x8000))      # the keys matter at all


PATHS = {"e4m3": 3, "e2m1": 2, "e5m2": 4}            # product-path ids of the plan


@pytest.mark.gpu
@pytest.mark.parametrize("D,reps,split", [(64, 1, 2), (64, 400, 1), (128, 1, 4), (128, 24, 2), (128, 400, 1)])
@pytest.mark.parametrize("lo,hi", [("e4m3", "e4m3"), ("e5m2", "e5m2"), ("e2m1", "e4m3"), ("e2m1", "e5m2")])
def test_infinities_and_nans(D, reps, split, lo, hi):
    """The keys' converts to 8 bits saturate in a mode in which the matrix instructions would lose infinities and NaN: neither may
    show.  A NaN among E4M3 or E5M2 keys, and an infinity among E4M3 ones, gives the key scores of NaN; an infinity among E5M2
    keys is one in the scores too; a NaN among the values reaches every row that sees it; rows before the key and the other
    head are untouched.  Every split of the keys; the pairs of one format walk tiles 0 to 4 of their last query tiles in main
    steps, where the next tile's converts come right behind the score or P V products, the others walk band steps."""
    from paper_2604_03950_amd import binding as dma
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    N = 8
    S = (N - 1) * D + 37
    assert plan.key_split(plan.problem(reps, 2, 2, S, D, lo=PATHS[lo]), PATHS[hi]) == split
    g = torch.Generator(device="cuda").manual_seed(D)
    q, k, v = (torch.randn((1, 2, S, D), generator=g, device="cuda").to(torch.bfloat16) for _ in range(3))

    def forward(k, v):
        out = dma.dma_attn_fwd(*(t.repeat(reps, 1, 1, 1) for t in (q, k, v)), diag_band_tiles=N, lo_fmt=FMTS[lo], hi_fmt=FMTS[hi],
                               tile=64 if D == 64 else None)                  # the band covers every tile
        assert torch.equal(out.nan_to_num(), out[:1].nan_to_num().expand_as(out))
        return out[0]

    plain = forward(k, v)
    assert torch.isfinite(plain).all()
    rows = torch.arange(S, device="cuda")
    for at in (11, D + 11, 2 * D + 40, (N - 2) * D + 11):
        for value in (float("nan"), float("inf"), float("-inf")):
            for column in (*range(0, 32, 2), 31, D - 7, D - 1):                # every dword of a block
                bad = k.clone()
                bad[:, 0, at, column] = value
                out = forward(bad, v)
                assert torch.equal(out[0, :at], plain[0, :at]) and torch.equal(out[1], plain[1]), (at, value, column)
                if hi == "e4m3" or value != value:
                    assert out[0, at:].isnan().all(), (at, value, column)
                    continue
                # The score is an infinity of the sign of the query's element: a row is NaN, or has no weight left for the
                # key, which 2^100 in its place gives as well.  (An element well below its block's maximum may round to 0.)
                sign = q[0, 0, :, column].float() * (1 if value > 0 else -1)
                up, down = (rows >= at) & (sign > 0.1), (rows >= at) & (sign < -0.1)
                bad[:, 0, at, column] = 2.0 ** 100 * (1 if value > 0 else -1)
                assert out[0, up].isnan().all() and up.any(), (at, value, column)
                assert torch.equal(out[0, down], forward(bad, v)[0, down]) and down.any(), (at, value, column)
        for column in (0, D - 1):
            bad = v.clone()
            bad[:, 0, at, column] = float("nan")
            out = forward(k, bad)
            seen = torch.arange(D, device="cuda") == column
            assert out[0, at:, seen].isnan().all() and torch.equal(out[0, :, ~seen], plain[0, :, ~seen]) and torch.equal(out[1], plain[1])
            tile = at // D * D                                                # within it a masked key's weight is 0, and 0 x NaN a NaN
            assert torch.equal(out[0, :tile], plain[0, :tile])
