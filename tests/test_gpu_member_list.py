"""Selection where more than half of a small component's energies share the
threshold's sub-bin: their list holds every value of the component (or as many
as are sorted at once, if that is less); bit for bit against the oracle."""

import numpy as np
import pytest
import torch

import oracle
from oracle.tables import gll_tables
from paper_2407_20731_amd import isr

pytestmark = pytest.mark.gpu


def _field(order, x, seed):
    """Nodal field [1, E, n, n, n] whose coefficients have the energies x[e]."""
    T, n = gll_tables(order), order + 1
    sign = np.random.default_rng(seed).choice([-1.0, 1.0], x.shape)
    coef = (sign * np.sqrt(x)).reshape(-1, n, n, n) / np.sqrt(np.asarray(T.g3).reshape(n, n, n))
    return np.ascontiguousarray(np.einsum("kr,jq,ip,erqp->ekji", T.V, T.V, T.V, coef, optimize=True))[None]


# 512 to 8,191 values: below, at and above the limit of what is sorted (4,096)
@pytest.mark.parametrize("order,n_elem", [(1, 64), (3, 65), (7, 1), (7, 8), (7, 15), (8, 1), (9, 1), (9, 5), (11, 4), (15, 1)])
@pytest.mark.parametrize("kind", ["sub_bin", "equal"])
def test_most_energies_in_one_sub_bin(order, n_elem, kind):
    m = n_elem * (order + 1) ** 3
    rng = np.random.default_rng(m)
    # one 1/256 of a binade, some of its eight parts; or as good as one value
    x = 1.0 + 2.0 ** -7 + rng.uniform(0.3, 0.9, m) * 2.0 ** -8 if kind == "sub_bin" else np.full(m, 1.01)
    u = _field(order, x, m)
    with isr.Context(device=0) as ctx:
        for tol in (0.05, 0.4, 0.8):
            ref = oracle.compress(u, order, tol, keep_arrays=True).comps[0]
            blob = ctx.compress(torch.from_numpy(u).cuda(), order, tol, "fp64")
            s = blob.stats
            assert (s["tau"][0], s["kept"][0], s["dropped"][0], s["norm2"][0], s["err2"][0]) == (
                ref.tau, ref.kept, ref.dropped, ref.U2, ref.err2), tol
            assert np.array_equal(blob.arrays().bitmap[0], ref.bitmap), tol
            blob.free()
