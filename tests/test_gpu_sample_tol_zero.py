"""tol = 0: the threshold is the smallest energy of the component.  A field of
fewer than 2,048 tiles is sampled whole, so the window holds that energy
wherever it lies."""

import pytest
import torch

import synth
from paper_2407_20731_amd import isr

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("order,n_elem,precision", [(5, 1900, "fp64"), (6, 2000, "fp64"), (3, 7000, "fp64"),
                                                    (7, 2047, "bf16"), (5, 7000, "bf16"), (9, 1500, "fp32")])
def test_window_holds_the_smallest_energy(order, n_elem, precision):
    base = torch.from_numpy(synth.field(n_elem, order)).cuda()
    with isr.Context(device=0) as ctx:
        for small in (1, n_elem // 2 + 1, n_elem - 2):
            u = base.clone()
            u[:, small] *= 2.0 ** -40
            blob = ctx.compress(u, order, 0.0, precision)
            assert blob.stats["path"] == 1, small
            blob.free()
