"""Attention items dealt by the rows' lengths (dealt_size, dealt_splits, dealt_range of cf_plan_arith.h, compiled for the host): at
most one item per member, at most 64 splits a row, splits that meet and cover every row, whatever the last bits of the device's reciprocals."""
import random

import pytest

import plan_arith

ULPS = (-2, -1, 0, 1, 2)


def check(lens, team_size, tps, gain, pairmap, ulps):
    d = plan_arith.deal(lens, team_size, tps, gain, pairmap, ulps)
    if not d.items:
        return d
    what = (lens, team_size, tps, gain, pairmap, ulps, d.items, d.size, d.splits)
    assert len(lens) <= d.items <= team_size and tps - d.size >= gain and all(1 <= n <= 64 for n in d.splits), what
    for length, row in zip(lens, d.ranges):
        assert row[0][0] == 0 and row[-1][1] == length and all(0 <= t0 <= t1 <= length for t0, t1 in row), what
        assert all(a[1] == b[0] for a, b in zip(row, row[1:])), what
    return d


@pytest.mark.parametrize("ulps", ULPS)
@pytest.mark.parametrize("rows", [1, 2, 8, 16])
def test_long_rows_with_as_many_members_as_rows(rows, ulps):
    """The only candidate that can fit is the longest row, where the quotient of 2 len - 1 and len may come out as 2 from 2^20 on."""
    rng = random.Random(rows)
    lengths = [2 ** k + e for k in range(18, 24) for e in (-1, 0, 1)] + [rng.randint(2 ** 20, 2 ** 24 - 400) for _ in range(300)]
    for longest in lengths:
        for rest in ([longest] * (rows - 1), [1] * (rows - 1), [rng.randint(0, longest) for _ in range(rows - 1)]):
            check([longest] + rest, rows, 2 ** 24 - 1, plan_arith.ragged_gain(64), 0, ulps)
            check(rest + [longest], rows + 1, 2 ** 24 - 1, plan_arith.ragged_gain(64), 1, ulps)


@pytest.mark.parametrize("ulps", ULPS)
def test_items_of_any_lengths(ulps):
    rng = random.Random(7 + ulps)
    dealt = 0
    for _ in range(6000):
        rows, top = rng.randint(1, 16), int(2 ** rng.uniform(6, 24)) - 1
        team_size = rng.randint(rows, rng.choice([rows, rows + 2, 32, 64, 256]) if rows < 32 else rows)
        lens = [int(top * rng.choice([0, rng.random(), rng.random() ** 6, 1])) for _ in range(rows)]
        splits = 1
        while splits < 64 and rows * splits * 2 <= team_size:
            splits *= 2
        d = check(lens, team_size, max(1, -(-top // splits)), plan_arith.ragged_gain(rng.choice([64, 128])), rng.randint(0, 1), ulps)
        dealt += d.items > 0
    assert dealt > 500


@pytest.mark.parametrize("head_dim", [64, 128])
def test_dealt_from_the_gain_on(head_dim):
    gain = plan_arith.ragged_gain(head_dim)
    lens = [8192, 170, 170, 170]
    size = plan_arith.deal(lens, 32, 10 ** 6, gain).size
    assert size > 0 and check(lens, 32, size + gain, gain, 1, 0).size == size
    assert check(lens, 32, size + gain - 1, gain, 1, 0).items == 0
