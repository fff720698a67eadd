"""The kernels' arithmetic as the host compiler sees it: divisions without an integer division, by plan constants (qdiv: the high
half of a product with ceil(2^31 / d)) and by divisors of a workgroup (fdiv: with a reciprocal that may be an ulp or two off), and
the shares of the hidden units that the FFN block's workgroups own."""
import ctypes

import numpy as np
import pytest

import plan_arith

DIVISORS = sorted(set(list(range(1, 70)) + [127, 128, 129, 255, 256, 341, 512, 824, 1000, 1023, 1024, 2048, 4095, 8192]))


def _ints(n):
    n = np.ascontiguousarray(n, dtype=np.int32)
    return n.ctypes.data_as(ctypes.POINTER(ctypes.c_int)), len(n), n


@pytest.mark.parametrize("d", DIVISORS)
def test_qdiv(d):
    n = np.unique(np.concatenate([np.arange(4096), np.arange(1, 40) * d - 1, np.arange(40) * d, [65535, min(2 ** 31 // d - 1, 2 ** 20)]]))
    p, count, keep = _ints(n[n.astype(np.int64) * d < 2 ** 31])
    assert plan_arith.load().pa_qdiv_differs(p, count, d) == -1


@pytest.mark.parametrize("d", DIVISORS)
def test_fdiv(d):
    k = np.unique(np.concatenate([np.arange(0, 2 ** 20, 977), np.arange(2 ** 20 // d + 1) * d, np.arange(1, 2 ** 20 // d + 1) * d - 1]))
    p, count, keep = _ints(k[k < 2 ** 20])
    for ulps in (-2, -1, 0, 1, 2):
        assert plan_arith.load().pa_fdiv_differs(p, count, d, ulps) == -1, ulps


@pytest.mark.parametrize("uneven", [0, 1])
def test_shares_of_the_hidden_units(uneven):
    """What neighbours own covers every unit once, the even one owns as many as the odd one or more, nobody owns none or more than the
    room that is made for it (the stride of its sums in LDS)."""
    lib = plan_arith.load()
    for W in (8, 16, 200, 256, 304) + (() if uneven else (1, 7, 255)):
        for F in list(range(W, 3 * W + 1)) + [10 * W + 7, 11008, 14336, 28672, 40001, 850432]:
            if F < W:
                continue
            first = [lib.pa_first_unit(w, F, W, uneven) for w in range(W + 1)]
            share = [b - a for a, b in zip(first, first[1:])]
            assert first[0] == 0 and first[-1] == F and min(share) >= 1 and max(share) <= lib.pa_most_units(F, W, uneven)
            if uneven:
                assert all(share[w] >= share[w + 1] for w in range(0, W, 2))


def test_shares_are_uneven_where_the_larger_one_fits():
    """Whole rounds of the eight dies, and the LDS of the largest batch tile on both sides of the limit.  What equal shares fit is never
    refused for the uneven ones."""
    lib = plan_arith.load()
    assert [lib.pa_uneven_shares(4096, 11008, w, 1) for w in (256, 252, 255, 8, 4, 304)] == [1, 0, 0, 1, 0, 1]
    sides = set()
    for d_model, tile in ((8, 1), (8, 4), (512, 2), (4096, 1), (4104, 4), (8192, 2)):
        for units in range(1, 20000, 7):
            F = 256 * units
            if F * d_model * 2 > 0x7fffffff or lib.pa_lds_bytes(d_model, tile, units) > lib.pa_lds_limit():
                break
            uneven = lib.pa_uneven_shares(d_model, F, 256, tile)
            most = lib.pa_most_units(F, 256, uneven)
            assert lib.pa_lds_bytes(d_model, tile, most) <= lib.pa_lds_limit()
            assert uneven or lib.pa_lds_bytes(d_model, tile, lib.pa_most_units(F, 256, 1)) > lib.pa_lds_limit()
            sides.add((tile, uneven))
    assert sides >= {(1, 0), (1, 1), (2, 1), (4, 0), (4, 1)}, sides
