"""A NaN in a large field is bad input at the first attempt: no second one with
lists for every value, which a tight budget would refuse for want of memory."""

import pytest
import torch

import synth
from paper_2407_20731_amd import isr

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("order,precision", [(2, "fp64"), (5, "fp64"), (7, "fp64"), (7, "fp32"), (7, "bf16"), (5, "bf16"),
                                             (9, "fp64"), (9, "bf16"), (12, "fp64")])
def test_nan_is_refused_as_input(order, precision):
    n3 = (order + 1) ** 3
    n_elem = (1 << 23) // n3
    # worst-case blob, first attempt's lists (2^20 candidates), histograms; lists for every
    # value would take 100 MB more
    blob = n_elem * ((8 if precision == "fp64" else 4) * n3 + 8 * ((n3 + 63) // 64) + 8)
    u = synth.field(n_elem, order, ncomp=1)
    u[0, n_elem // 3].flat[n3 // 2] = float("nan")
    d = torch.from_numpy(u).cuda()
    with isr.Context(device=0, budget_bytes=blob + (48 << 20)) as ctx:
        with pytest.raises(isr.IsrError) as e:
            ctx.compress(d, order, 1e-3, precision)
        assert e.value.code == isr.EINVAL
        # the same field without it fits
        u[0, n_elem // 3].flat[n3 // 2] = 0.25
        d.copy_(torch.from_numpy(u))
        ctx.compress(d, order, 1e-3, precision).free()
