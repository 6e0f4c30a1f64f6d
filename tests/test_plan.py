"""The plan of a forward against a plain reading of the schedule the kernels walk (no GPU needed)."""
import random

import pytest

import plan


def dealt(B, Hq, Hkv, NG, heads_item, slots, cost):
    """Sum of cost(group) over the items of every workgroup, dealt as the kernels deal them: ranked heaviest first within
    blocks of query heads, to the workgroups (of one XCD where the kv heads divide over eight) forwards and backwards in turn."""
    items = B * (Hq // heads_item) * NG
    blocks = min(items, slots)
    units, group = B * Hkv, Hq // Hkv // heads_item
    by_xcd = units % 8 == 0 and blocks % 8 == 0
    workers = blocks // 8 if by_xcd else blocks
    heads = (units // 8 if by_xcd else units) * group
    block = next((hb for hb in range(group, heads, group) if heads % hb == 0 and hb * NG % (2 * workers) == 0), heads)
    load = [0.0] * workers
    for pos in range(heads * NG):
        r, at = divmod(pos, workers)
        load[workers - 1 - at if r % 2 else at] += cost(NG - 1 - pos % (block * NG) // block)
    return load


def items_of(S, tile, rows, causal):
    N = -(-S // tile)
    tiles = lambda grp: min(((grp + 1) * rows - 1) // tile + 1, N) if causal else N
    return -(-S // rows), tiles


def test_dealt_load():
    """The longest list is the longest over all workgroups, not only the first and the last: those two miss it wherever the last
    round is partial or a run of items of one length ends inside a round.  The work of a CU: an even share of everything with
    the mask, the lists of as many workgroups as the fullest CU holds without it."""
    rng = random.Random(1)
    cases = [(1, 40, 8, 487, 128, True, 64, 1, 256, 1), (2, 40, 8, 618, 128, True, 128, 1, 256, 1), (2, 40, 8, 650, 64, True, 64, 1, 256, 2)]
    for _ in range(400):
        D = rng.choice([64, 128])
        Hkv, group = rng.choice([1, 2, 3, 5, 8, 16]), rng.choice([1, 2, 3, 4, 5])
        pair = group % 2 == 0 and rng.random() < 0.5
        rows = D if pair else rng.choice([D // 2, D, 2 * D])
        cases.append((rng.choice([1, 1, 2, 8]), Hkv * group, Hkv, rng.randrange(D + 1, 3000), D, rng.random() < 0.7, rows, 2 if pair else 1,
                      rng.choice([1, 7, 64, 256]), rng.choice([1, 2, 3, 4])))
    ends_miss = 0
    for B, Hq, Hkv, S, D, causal, rows, heads_item, cus, resident in cases:
        NG, tiles = items_of(S, D, rows, causal)
        load = dealt(B, Hq, Hkv, NG, heads_item, cus * resident, lambda grp: 1.5 + 0.5 * tiles(grp))        # exact in binary32
        what = (B, Hq, Hkv, S, D, causal, rows, heads_item, cus, resident)
        longest, cu = plan.dealt_load(plan.problem(B, Hq, Hkv, S, D, causal), rows, heads_item, cus, resident, 0.5, 1.5)
        assert longest == max(load), what
        total = sum(1.5 + 0.5 * tiles(grp) for grp in range(NG)) * B * (Hq // heads_item)
        blocks = min(B * (Hq // heads_item) * NG, cus * resident)
        assert cu == pytest.approx(total / cus if causal else total / blocks * -(-blocks // cus), rel=1e-6), what
        ends_miss += max(load[0], load[-1]) < max(load)
    assert ends_miss >= 10                     # the cases do hold lists that neither end has


def test_split_by_the_longest_list():
    """40 / 8 heads, S = 487: by the first and the last workgroup four waves looked shorter (4.86 steps) than two (4.98);
    a workgroup in the middle has 5.39."""
    assert plan.key_split(plan.problem(1, 40, 8, 487)) == 2


@pytest.mark.parametrize("B,Hq,Hkv,S,causal,lo,hi,split", [
    (8, 2, 1, 4290, True, 2, 3, 1),          # 64.5 us unsplit, 72.8 split
    (3, 5, 1, 4565, True, 3, 3, 1),          # 77.8, 87.0
    (1, 8, 2, 2600, False, 2, 3, 1),         # 40.9, 43.0
    (1, 4, 1, 3700, True, 2, 3, 2),
    (1, 2, 2, 256, True, 2, 3, 2),
])
def test_split_at_the_occupancy_of_the_launch(B, Hq, Hkv, S, causal, lo, hi, split):
    """D = 64: three or four workgroups share a CU.  Counted as two, the rule split calls that the split makes slower."""
    assert plan.key_split(plan.problem(B, Hq, Hkv, S, 64, causal, lo), hi) == split


@pytest.mark.parametrize("B,Hq,Hkv,S,D,lo,hi,split", [
    (1, 40, 8, 400, 128, 2, 2, 4),           # us with two waves and four: 15.1, 13.5
    (1, 40, 8, 400, 128, 3, 3, 4),           # 17.0, 14.0
    (1, 40, 8, 400, 128, 4, 4, 4),           # 17.0, 14.1
    (1, 40, 8, 400, 128, 1, 1, 4),           # 15.9, 13.8
    (1, 40, 8, 400, 128, 0, 0, 2),           # 14.6, 15.3: no query operands to make
    (1, 32, 8, 822, 128, 2, 2, 4),           # 18.6, 17.1
    (1, 32, 8, 822, 128, 2, 3, 2),           # 20.1, 20.5
    (3, 8, 2, 1199, 128, 3, 3, 4),           # 27.3, 24.7
    (3, 8, 2, 1199, 128, 2, 3, 2),           # 25.5, 26.0
    (1, 8, 1, 4387, 128, 3, 3, 4),           # 0.93 of the time with two
    (1, 32, 8, 1800, 64, 0, 0, 2),           # two waves and unsplit: 28.0, 31.6
    (45, 5, 1, 298, 64, 2, 2, 1),            # 13.8, 11.9: more than two items per compute unit
    (16, 16, 16, 292, 64, 2, 2, 1),          # 14.7, 12.4
    (8, 32, 8, 267, 64, 0, 0, 1),            # 14.2, 12.4
    (1, 4, 1, 3700, 128, 2, 3, 4),
    (1, 32, 8, 2600, 128, 2, 3, 1),
])
def test_split_costs(B, Hq, Hkv, S, D, lo, hi, split):
    """Problems close to where the choice turns, as timed."""
    assert plan.key_split(plan.problem(B, Hq, Hkv, S, D, lo=lo), hi) == split


@pytest.mark.parametrize("B,Hq,Hkv,S,lo,hi", [
    (1, 40, 8, 400, 3, 3),                   # us with two waves and four: 17.6, 18.1
    (1, 32, 8, 822, 3, 3),                   # 25.3, 25.9
    (1, 32, 8, 822, 2, 3),                   # 24.0, 26.5
])
def test_split_costs_with_the_step_2_scale(B, Hq, Hkv, S, lo, hi):
    """Its query operands are made by every wave for itself: an item of four waves costs what it did."""
    assert plan.key_split(plan.problem(B, Hq, Hkv, S, 128, True, lo, True), hi) == 2


@pytest.mark.parametrize("B,Hq,Hkv,S,D,item", [
    (1, 32, 8, 128, 128, plan.ONE_TILE),     # us alone and in pairs, all MXFP8: 9.6, 11.2
    (8, 32, 8, 128, 128, plan.ONE_TILE),
    (9, 32, 8, 128, 128, plan.TWO_HEADS),    # more heads than compute units
    (64, 32, 8, 100, 128, plan.TWO_HEADS),   # 67.0, 47.0
    (1, 4, 4, 1, 64, plan.ONE_TILE),
    (100, 9, 3, 64, 64, plan.ONE_TILE),      # no pairs
    (64, 40, 8, 300, 128, plan.TWO_TILES),
    (64, 32, 8, 300, 128, plan.TWO_HEADS),
    (1, 128, 32, 269, 128, plan.TWO_TILES),  # 16.0 us, with a tile of two heads 18.0
    (8, 12, 3, 318, 128, plan.TWO_TILES),    # 18.9, 21.0
    (1, 129, 43, 269, 128, plan.TWO_TILES),  # no pairs
    (1, 132, 33, 269, 128, plan.TWO_HEADS),  # more items than compute units
    (1, 128, 32, 256, 128, plan.TWO_HEADS),
    (1, 128, 32, 150, 64, plan.TWO_HEADS),
])
def test_unsplit_item(B, Hq, Hkv, S, D, item):
    assert plan.unsplit_item(plan.problem(B, Hq, Hkv, S, D)) == item
    if item == plan.TWO_TILES and Hq // Hkv % 2 == 0:
        assert plan.unsplit_item(plan.problem(B, Hq, Hkv, S, D, causal=False)) == plan.TWO_HEADS


@pytest.mark.parametrize("B,Hq,Hkv,S,lo,hi,per_token,split", [
    (4, 48, 16, 192, 3, 3, True, 1),         # us unsplit and split: 11.3, 12.5
    (11, 16, 2, 256, 0, 0, False, 1),        # 9.8, 10.3
    (1, 4, 1, 3700, 2, 3, True, 2),
])
def test_split_without_the_mask_at_d64(B, Hq, Hkv, S, lo, hi, per_token, split):
    assert plan.key_split(plan.problem(B, Hq, Hkv, S, 64, False, lo, per_token), hi) == split
