"""The sampled window of the low orders, whose tiles hold few values: requests
whose threshold a sample of 256 tiles missed are decided on the streaming path."""

import pytest
import torch

import synth
from paper_2407_20731_amd import isr

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["fp64", "fp32", "bf16"])
def test_window_holds_the_threshold(precision):
    u = torch.from_numpy(synth.field(30011, 1, seed=1, noise=0.0)).cuda()
    with isr.Context(device=0) as ctx:
        blob = ctx.compress(u, 1, 1e-4, precision)
        assert blob.stats["path"] == 1
        blob.free()
