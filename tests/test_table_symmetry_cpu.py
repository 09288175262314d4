"""CPU: the bit-exact mirror symmetry of the FP64 tables that the fixed-order
contractions rely on (they read half of the entries and take the mirrored ones
from them by sign)."""

import numpy as np
import pytest

from paper_2407_20731_amd import isr


@pytest.mark.parametrize("order", range(1, 16))
def test_tables_mirror_bit_for_bit(order):
    n = order + 1
    T = isr.gll_tables(order)
    A, V = T["A"], T["V"]
    bits = lambda a: np.ascontiguousarray(a).view(np.uint64)  # noqa: E731
    sign = np.where(np.arange(n) % 2 == 0, 1.0, -1.0)
    half = np.arange(n) < n // 2  # the middle entry of an odd n is read itself
    # A[p][n-1-i] = (-1)^p A[p][i]
    assert np.array_equal(bits(A[:, ::-1][:, half]), bits((sign[:, None] * A)[:, half]))
    # V[n-1-i][k] = (-1)^k V[i][k]
    assert np.array_equal(bits(V[::-1][half]), bits((V * sign[None, :])[half]))
