"""CPU: the per-element cut's bisection over keys (the selection kernel's
bounds and steps, written out in integers) ends and finds the threshold of the
plain rule for sets with ties, neighbours one bit apart, zeros and single
values."""

import random
import struct

import pytest


def bits(x):
    return struct.unpack("<Q", struct.pack("<d", x))[0]


def val(k):
    return struct.unpack("<d", struct.pack("<Q", k))[0]


def search(keys, feasible, small_bound, B):
    """The loop of the kernel; feasible(k): the sum of the values below key k fits."""
    last_upto = lambda most: max([0] + [k for k in keys if k <= most])  # noqa: E731
    first_from = lambda least: min([2 ** 64 - 1] + [k for k in keys if k >= least])  # noqa: E731
    small = last_upto(bits(small_bound))
    lo = small if small else first_from(0)
    over = first_from(bits(B) + 1)
    hi = (over if over != 2 ** 64 - 1 else last_upto(0x7FF0000000000000)) + 1
    for step in range(400):
        mid = lo + 1 + ((hi - lo - 1) >> 1)
        up = first_from(mid)
        if up < hi:
            if feasible(up):
                lo = up
            else:
                hi = mid
        else:
            dn = last_upto(mid - 1)
            if dn <= lo:
                return lo, step
            hi = dn + 1
    raise AssertionError("the search does not end")


@pytest.mark.parametrize("seed", range(200))
def test_search_ends_at_the_threshold(seed):
    r = random.Random(seed)
    n = r.choice([1, 2, 3, 8, 64, 512])
    kind = seed % 5
    if kind == 0:
        vals = [2.0 ** r.uniform(-60, 2) for _ in range(n)]
    elif kind == 1:
        base = bits(2.0 ** r.uniform(-3, 3))
        vals = [val(base + r.randrange(3)) for _ in range(n)]  # neighbours and ties
    elif kind == 2:
        vals = [r.choice([0.0, 1.0, 2.0]) for _ in range(n)]
    elif kind == 3:
        vals = [val(bits(1.0) + i) for i in range(n)]
    else:
        vals = [r.choice([5e-324, 1e-300, 1e-10, 1.0]) for _ in range(n)]
    keys = [bits(v) for v in vals]
    for B in (0.0, sum(vals) * 1e-6, sum(vals) * 0.3, sum(vals) * 0.999, max(vals), min(vals)):
        feasible = lambda k: sum(sorted(v for v, q in zip(vals, keys) if q < k)) <= B  # noqa: E731,B023
        if feasible(0x7FF0000000000000):
            continue  # everything fits: the kernel does not search
        tau, steps = search(keys, feasible, B / (2.0 * max(n, 64)), B)
        assert tau == max(k for k in keys if feasible(k))
        assert steps <= 130
