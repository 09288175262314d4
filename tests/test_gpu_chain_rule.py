"""Which small requests take the selection chain in one workgroup per component:
white noise at a loose tolerance, whose candidate list holds most values, is not
slower at 1,000 elements than at 4,000 (which take separate launches); and both
sides of every line of the rule, bit for bit against the oracle."""

import time

import numpy as np
import pytest
import torch

import oracle
from paper_2407_20731_amd import isr

pytestmark = pytest.mark.gpu


def _white(n_elem, order, ncomp):
    n = order + 1
    return np.random.default_rng(n_elem).standard_normal((ncomp, n_elem, n, n, n))


@pytest.mark.parametrize("precision", ["fp64", "fp32", "bf16"])
@pytest.mark.parametrize("order,n_elem", [(7, 1000), (9, 500)])
def test_long_lists_take_separate_launches(order, n_elem, precision):
    best = {}
    with isr.Context(device=0) as ctx:
        for E in (n_elem, 4 * n_elem):
            u = torch.from_numpy(_white(E, order, 3)).cuda()
            for _ in range(7):
                torch.cuda.synchronize()
                t = time.perf_counter()
                ctx.compress(u, order, 0.5, precision).free()
                torch.cuda.synchronize()
                best[E] = min(best.get(E, 1.0), time.perf_counter() - t)
    assert best[n_elem] < best[4 * n_elem], best


# 2^17 and 2^18 values are 256 and 512 elements at N = 7; N = 3: the limit on
# elements comes first
@pytest.mark.parametrize("order,n_elem", [(7, 255), (7, 256), (7, 512), (7, 513), (3, 1024), (3, 1025)])
@pytest.mark.parametrize("tol", [1e-2, 1.1e-2])
def test_both_sides_of_the_line(order, n_elem, tol):
    u = _white(n_elem, order, 2)
    ref = oracle.compress(u, order, tol, keep_arrays=True)
    with isr.Context(device=0) as ctx:
        blob = ctx.compress(torch.from_numpy(u).cuda(), order, tol, "fp64")
        s, arr = blob.stats, blob.arrays()
        for c, r in enumerate(ref.comps):
            got = (s["norm2"][c], s["tau"][c], s["dropped"][c], s["err2"][c], s["kept"][c])
            assert got == (r.U2, r.tau, r.dropped, r.err2, r.kept), c
            assert np.array_equal(arr.bitmap[c], r.bitmap) and np.array_equal(arr.elem_ptr[c], r.elem_ptr), c
        blob.free()
