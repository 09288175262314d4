"""The per-element cut's search in the selection kernel itself, on elements whose
energies are hard sets: neighbours a few bits apart, ties, few distinct values
with zeros, consecutive floats, three hundred orders of magnitude, single values;
bit for bit against the oracle's threshold of every element."""

import numpy as np
import pytest
import torch

from oracle import elemcut as P
from oracle.tables import gll_tables
from paper_2407_20731_amd import isr

pytestmark = pytest.mark.gpu


def _sets(rng, n3):
    one = np.array([1.0])
    consecutive = (one.view(np.int64) + np.arange(n3)).view(np.float64)
    few = rng.choice([0.0, 1.0, 2.0], n3)
    few[0] = 1.0
    single = np.zeros(n3)
    single[rng.integers(n3)] = 3.0
    return [2.0 ** rng.uniform(-60, 2, n3), 2.0 ** rng.uniform(-3, 3) * (1.0 + rng.integers(0, 3, n3) * 2.0 ** -51), few,
            consecutive, rng.choice([5e-324, 1e-300, 1e-10, 1.0], n3), np.full(n3, 0.7), single, np.zeros(n3),
            2.0 ** rng.uniform(-900, -840, n3), np.where(np.arange(n3) == 5, 1.0, 1e-12)]


@pytest.mark.parametrize("order", [1, 2, 3, 5, 7, 8, 11, 15])
@pytest.mark.parametrize("tol", [0.0, 1e-8, 1e-3, 0.3 ** 0.5, 0.999 ** 0.5, 1.5])
def test_hard_sets(order, tol):
    T, n = gll_tables(order), order + 1
    rng = np.random.default_rng(order)
    x = np.array([s for _ in range(2) for s in _sets(rng, n ** 3)])
    coef = rng.choice([-1.0, 1.0], x.shape) * np.sqrt(x)
    nodal = np.einsum("kr,jq,ip,erqp->ekji", T.V, T.V, T.V, coef.reshape(-1, n, n, n) / np.sqrt(np.asarray(T.g3)),
                      optimize=True)
    # the sets as modal energies, and as squares of nodal values
    u = np.ascontiguousarray(np.stack([nodal, coef.reshape(-1, n, n, n)]))
    ref = P.compress_elemcut(u, order, tol)
    with isr.Context(device=0) as ctx:
        blob = ctx.compress_elemcut(torch.from_numpy(u).cuda(), order, tol)
        arr = blob.arrays()
        for c, r in enumerate(ref):
            h = arr.comps[c]
            assert (h["U2"], h["dropped"], h["err2"], h["kept"]) == (r.U2, r.dropped, r.err2, r.kept), c
            assert np.array_equal(arr.bitmap[c], r.bitmap) and np.array_equal(arr.elem_ptr[c], r.elem_ptr), c
            assert np.array_equal(arr.values[c].view(np.uint64), r.values.view(np.uint64)), c
        blob.free()
