"""The candidate prefilter's packed comparison, restated on the CPU and
checked against the comparisons axis by axis: three 20-bit levels in one
64-bit word, 21 bits apart, compared by one subtraction with guard bits."""

import numpy as np
import pytest

BITS, STRIDE = 20, 21
QMAX = (1 << BITS) - 1
GUARD = np.uint64((1 << BITS) * (1 + (1 << STRIDE) + (1 << (2 * STRIDE))))


def pack(levels):
    """(n, 3) levels of 0..QMAX in one word each."""
    w = np.zeros(levels.shape[0], dtype=np.uint64)
    for d in range(3):
        w |= levels[:, d].astype(np.uint64) << np.uint64(STRIDE * d)
    return w


def all_ge(x, y):
    """x >= y in every field, by the subtraction."""
    return (((x | GUARD) - y) & GUARD) == GUARD


@pytest.mark.parametrize("seed", [0, 1])
def test_packed_comparison(seed):
    rng = np.random.default_rng(seed)
    n = 200_000
    x = rng.integers(0, QMAX + 1, size=(n, 3))
    # equal, neighbouring, extreme and unrelated levels, axis by axis
    kind = rng.integers(0, 6, size=(n, 3))
    y = np.select([kind == 0, kind == 1, kind == 2, kind == 3, kind == 4],
                  [x, np.minimum(x + 1, QMAX), np.maximum(x - 1, 0), np.zeros_like(x), np.full_like(x, QMAX)],
                  rng.integers(0, QMAX + 1, size=(n, 3)))
    assert np.array_equal(all_ge(pack(x), pack(y)), (x >= y).all(1))
    assert np.array_equal(all_ge(pack(y), pack(x)), (y >= x).all(1))


def test_decisions_are_those_of_the_levels():
    """Pass, fail and undecided from packed thresholds (lp = la + 1, cp =
    ec - 1) are those of the four comparisons per axis."""
    rng = np.random.default_rng(2)
    n = 200_000
    ea = rng.integers(0, 40, size=(n, 3))
    la = ea - (rng.random((n, 3)) < 0.3)
    ec = ea + rng.integers(1, 30, size=(n, 3))
    ql, qh = rng.integers(0, 60, size=(n, 3)), rng.integers(0, 60, size=(n, 3))
    fail = ((qh < ea) | (ql > ec)).any(1)
    passed = ((qh > la) & (ql < ec)).all(1)
    P, H, L = pack, pack(qh), pack(ql)
    got_pass = all_ge(H, P(la + 1)) & all_ge(P(ec - 1), L)
    got_meet = all_ge(H, P(ea)) & all_ge(P(ec), L)
    assert np.array_equal(got_pass, passed)
    assert np.array_equal(~got_meet, fail)
    assert not (got_pass & ~got_meet).any()
