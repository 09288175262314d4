"""The smallest budget of the per-element cut: the worst-case blob, the
coefficients, the thresholds and the error bins, and next to nothing beside
them; also where a budget repair computes the coefficients again."""

import pytest
import torch

import synth
from oracle import elemcut as P
from paper_2407_20731_amd import isr

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("order,n_elem,ncomp", [(1, 60000, 3), (3, 20011, 1), (5, 20000, 3), (9, 5003, 2)])
def test_smallest_budget(order, n_elem, ncomp):
    n3 = (order + 1) ** 3
    values = ncomp * n_elem * n3 * 8
    blob = values + ncomp * (n_elem * ((n3 + 63) // 64) * 8 + (n_elem + 1) * 8)
    scratch = values + ncomp * n_elem * 8 + ncomp * 2048 * 24
    u = torch.from_numpy(synth.field(n_elem, order, ncomp=ncomp)).cuda()
    with isr.Context(device=0, budget_bytes=blob + scratch + (16 << 10)) as ctx:
        tight = ctx.compress_elemcut(u, order, 1e-3).to_bytes()
    with isr.Context(device=0) as ctx:
        assert ctx.compress_elemcut(u, order, 1e-3).to_bytes() == tight


@pytest.mark.parametrize("order,repairs", [(4, False), (7, True), (10, True)])
def test_repair(order, repairs):
    # bounds at the rounding of the transforms, where the first cut's error exceeds them
    u, iters = synth.field(3, order, ncomp=2, noise=0.0), 0
    with isr.Context(device=0) as ctx:
        for tol in (1e-14, 1e-15, 3e-16):
            ref = P.compress_elemcut(u, order, tol)
            blob = ctx.compress_elemcut(torch.from_numpy(u).cuda(), order, tol)
            iters += blob.stats["repair_iters"]
            for h, r in zip(blob.arrays().comps, ref):
                assert (h["U2"], h["dropped"], h["err2"], h["kept"]) == (r.U2, r.dropped, r.err2, r.kept), tol
            blob.free()
    assert (iters > 0) == repairs
