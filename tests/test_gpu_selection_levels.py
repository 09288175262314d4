"""Threshold selection where its levels can go wrong: boundary sub-bins of a
few, of about the narrowing and sort limits, and of more members than the sort
takes; ties across the cut; thresholds decided at the first and the last
fraction bits; bit for bit against the oracle."""

import numpy as np
import pytest
import torch

import oracle
from paper_2407_20731_amd import isr
from oracle.tables import gll_tables

pytestmark = pytest.mark.gpu


def _field(order, n_elem, coef):
    """Nodal field whose Legendre coefficients are coef[e, r, q, p]."""
    V = gll_tables(order).V
    return np.ascontiguousarray(np.einsum("kr,jq,ip,erqp->ekji", V, V, V, coef, optimize=True))[None]


@pytest.mark.parametrize("kind,n_elem", [("few", 8), ("sort_limit", 16), ("cap", 24), ("ties", 24), ("close", 24), ("binade", 40),
                                         ("two_values", 40)])
@pytest.mark.parametrize("prec", ["fp64"])
def test_selection_levels(kind, n_elem, prec):
    order, n = 7, 8
    rng = np.random.default_rng(n_elem)
    T = gll_tables(order)
    g = np.asarray(T.g3)
    m = n_elem * n ** 3
    x = {
        "few": lambda: 2.0 ** rng.uniform(-30, 0, m),
        "sort_limit": lambda: 1.0 + rng.random(m) * 2.0 ** -7,
        "cap": lambda: 1.0 + rng.random(m) * 2.0 ** -9,
        "ties": lambda: np.where(rng.random(m) < 0.7, 1.0, 2.0 ** rng.uniform(-3, 3, m)),
        "close": lambda: 1.0 + rng.integers(0, 3, m) * 2.0 ** -20,
        "binade": lambda: 2.0 ** rng.uniform(0, 1, m),
        "two_values": lambda: rng.choice([1.0, 1.0 + 2.0 ** -44], m),
    }[kind]()
    coef = (rng.choice([-1.0, 1.0], m) * np.sqrt(x)).reshape(n_elem, n, n, n) / np.sqrt(g)
    u = _field(order, n_elem, coef)
    with isr.Context(device=0) as ctx:
        for tol in (0.05, 0.4, 0.8):
            ref = oracle.compress(u, order, tol, keep_arrays=True).comps[0]
            blob = ctx.compress(torch.from_numpy(u).cuda(), order, tol, prec)
            s = blob.stats
            assert (s["tau"][0], s["kept"][0], s["dropped"][0], s["norm2"][0], s["err2"][0]) == (
                ref.tau, ref.kept, ref.dropped, ref.U2, ref.err2), tol
            assert np.array_equal(blob.arrays().bitmap[0], ref.bitmap), tol
            blob.free()
