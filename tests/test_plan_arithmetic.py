"""The divisions the fused kernel does without an integer division, emulated: by plan constants (qdiv: the high half of a product
with ceil(2^31 / d)) and by divisors of a workgroup (fdiv: with a reciprocal that may be an ulp or two off)."""
import numpy as np
import pytest

DIVISORS = sorted(set(list(range(1, 70)) + [127, 128, 129, 255, 256, 341, 512, 824, 1000, 1023, 1024, 2048, 4095, 8192]))


@pytest.mark.parametrize("d", DIVISORS)
def test_qdiv(d):
    m = (0x80000000 + d - 1) // d
    n = np.unique(np.concatenate([np.arange(4096), np.arange(1, 40) * d - 1, np.arange(40) * d, [65535, min(2 ** 31 // d - 1, 2 ** 20)]])).astype(np.uint64)
    n = n[n * d < 2 ** 31]
    assert np.array_equal((2 * n * np.uint64(m)) >> np.uint64(32), n // np.uint64(d))


@pytest.mark.parametrize("d", DIVISORS)
def test_fdiv(d):
    k = np.unique(np.concatenate([np.arange(0, 2 ** 20, 977), np.arange(2 ** 20 // d + 1) * d, np.arange(1, 2 ** 20 // d + 1) * d - 1]))
    k = k[k < 2 ** 20].astype(np.int64)
    r = np.float32(1.0) / np.float32(d)
    for ulps in (-2, -1, 0, 1, 2):
        rr = r
        for _ in range(abs(ulps)):
            rr = np.nextafter(rr, np.float32(np.inf if ulps > 0 else 0), dtype=np.float32)
        got = ((k.astype(np.float32) + np.float32(0.5)) * rr).astype(np.int64)
        assert np.array_equal(got, k // d), ulps


def test_uneven_shares_of_the_hidden_units():
    """FFN kernels: what neighbours own covers every unit once, the even one owns as many as the odd one or more, nobody owns none
    or more than the host makes room for."""
    def even_units(pair):
        return (pair * 524 + 512) >> 10

    def first_unit(w, F, W):
        p0 = (w & ~1) * F // W
        return p0 + even_units((w + 1) * F // W - p0) if w & 1 else p0

    for W in (8, 16, 200, 256, 304):
        for F in list(range(W, 3 * W + 1)) + [10 * W + 7, 11008, 14336, 28672, 40001]:
            if F < W:
                continue
            first = [first_unit(w, F, W) for w in range(W + 1)]
            share = [b - a for a, b in zip(first, first[1:])]
            most = max(even_units((F + W // 2 - 1) // (W // 2)), -(-F // W))
            assert first[0] == 0 and first[-1] == F and min(share) >= 1 and max(share) <= most
            assert all(share[w] >= share[w + 1] for w in range(0, W, 2))
