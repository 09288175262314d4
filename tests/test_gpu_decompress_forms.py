"""Decompression of the orders that the wave-tile kernel serves, in both output
types: ragged tiles, whole tiles, dense and empty elements, an output that is
only 8-byte aligned, quantisation codes; against the oracle's inverse."""

import numpy as np
import pytest
import torch

import oracle
import synth
from paper_2407_20731_amd import isr

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("order,n_elem", [(1, 1), (1, 33), (2, 15), (3, 9), (4, 5), (5, 3), (6, 2), (7, 1), (7, 130)])
@pytest.mark.parametrize("tol", [-1.0, 1e-2])
def test_fp64_blob_both_output_types(order, n_elem, tol):
    u = synth.field(n_elem, order, ncomp=2, seed=order + n_elem)
    u[1, n_elem // 2] = 0.0  # an element without kept values
    ref = oracle.compress(u, order, tol, keep_arrays=True)
    with isr.Context(device=0) as ctx:
        blob = ctx.compress(torch.from_numpy(u).cuda(), order, tol, "fp64")
        n = order + 1
        # one double past a fresh allocation: 8-byte aligned only
        for dtype, np_t in ((torch.float64, np.float64), (torch.float32, np.float32)):
            per = 8 // dtype.itemsize
            raw = torch.full((u.size + 2 * per,), 7.0, dtype=dtype, device="cuda")
            out = raw[per:per + u.size].view(2, n_elem, n, n, n)
            ctx.decompress(blob, out=out)
            torch.cuda.synchronize()
            for c, rc in enumerate(ref.comps):
                # the FP64 inverse bit for bit; FP32 output is its rounding
                assert np.array_equal(out[c].cpu().numpy(), rc.recon.astype(np_t))
            assert (raw[:per] == 7.0).all() and (raw[per + u.size:] == 7.0).all()
        blob.free()


@pytest.mark.parametrize("prec", ["fp32", "bf16"])
@pytest.mark.parametrize("order,n_elem", [(1, 33), (4, 9), (6, 3), (7, 1), (7, 65)])
def test_wave_tile_blob_both_output_types(order, n_elem, prec):
    u = synth.field(n_elem, order, ncomp=2, seed=3 * order + n_elem)
    with isr.Context(device=0) as ctx:
        ctx.set_tile(order, prec, 0)
        blob = ctx.compress(torch.from_numpy(u).cuda(), order, 1e-3, prec)
        d64 = ctx.decompress(blob)
        d32 = ctx.decompress(blob, dtype=torch.float32)
        torch.cuda.synchronize()
        # the transform's values are FP32: both outputs hold the same numbers
        assert torch.equal(d64.float(), d32) and torch.equal(d32.double(), d64)
        for c in range(2):
            err = np.sqrt(((d64[c].cpu().numpy() - u[c]) ** 2).mean() / (u[c] ** 2).mean())
            assert err < 1e-2  # unweighted norm: the bound is 1e-3 in the mass-weighted one
        blob.free()


@pytest.mark.parametrize("order,n_elem", [(3, 9), (7, 65)])
def test_quantised_blob_to_fp32(order, n_elem):
    u = synth.field(n_elem, order, ncomp=1, seed=7)
    with isr.Context(device=0) as ctx:
        blob = ctx.compress_quantized(torch.from_numpy(u).cuda(), order, 1e-3)
        d64 = ctx.decompress(blob)
        d32 = ctx.decompress(blob, dtype=torch.float32)
        torch.cuda.synchronize()
        assert torch.equal(d64.float(), d32)
        blob.free()


@pytest.mark.parametrize("prec", ["fp32", "bf16"])
@pytest.mark.parametrize("order,tile,n_elem", [(1, 64, 65), (2, 16, 17), (4, 8, 3), (5, 4, 9), (6, 3, 4), (8, 1, 2), (9, 2, 5),
                                               (10, 1, 3)])
@pytest.mark.parametrize("tol", [-1.0, 1e-2])
def test_dense_tile_blob_both_output_types(order, tile, n_elem, tol, prec):
    u = synth.field(n_elem, order, ncomp=2, seed=5 * order + n_elem)
    u[1, n_elem // 2] = 0.0
    n = order + 1
    with isr.Context(device=0) as ctx:
        ctx.set_tile(order, prec, tile)
        blob = ctx.compress(torch.from_numpy(u).cuda(), order, tol, prec)
        d64 = ctx.decompress(blob)
        raw = torch.full((u.size + 4,), 7.0, dtype=torch.float32, device="cuda")
        d32 = raw[2:2 + u.size].view(2, n_elem, n, n, n)  # 8-byte aligned only
        ctx.decompress(blob, out=d32)
        torch.cuda.synchronize()
        assert torch.equal(d64.float(), d32) and torch.equal(d32.double(), d64)
        assert (raw[:2] == 7.0).all() and (raw[2 + u.size:] == 7.0).all()
        # the oracle's inverse of the kept values; the transform error of the
        # BF16 split is about 2^-16 of the coefficients' scale, FP32's 2^-24
        arr = blob.arrays()
        T = oracle.tables.gll_tables(order)
        coef = np.zeros((2, n_elem, n ** 3))
        for c in range(2):
            bits = np.unpackbits(arr.bitmap[c].view(np.uint8).reshape(n_elem, -1), axis=1, bitorder="little")
            coef[c][bits[:, :n ** 3].astype(bool)] = arr.values[c]
        x = coef.reshape(2, n_elem, n, n, n)
        full = np.einsum("kr,jq,ip,cerqp->cekji", T.V, T.V, T.V, x, optimize=True)
        scale = np.einsum("kr,jq,ip,cerqp->cekji", abs(T.V), abs(T.V), abs(T.V), abs(x), optimize=True).max()
        assert np.abs(d64.cpu().numpy() - full).max() <= (2.0 ** -12 if prec == "bf16" else 2.0 ** -20) * scale
        blob.free()
