"""The workloads that the library's speed is measured on.

Every case is a whole use of the public binding (`paper_2407_20731_amd.isr`):
a snapshot (or several) resident in HBM goes through one of the compression
calls, and its reconstruction comes back.  Sizes are those of bench.py and of
the tests, or ragged ones near them.  `listed` names the cases, `draw` gives
further ones of the same ranges, `prepare` makes what a program has in hand
before the call, `run` is one pass, `work` what the pass cannot do without,
and `exact` its result in plain 64-bit torch arithmetic.

A case is a dict of
  op     "snapshot"  isr_compress, then isr_decompress of the blob
         "elemcut"   isr_compress_elemcut, then isr_decompress
         "quantized" isr_compress_quantized, then isr_decompress
         "writer"    isr_compress, the blob's bytes to the host, a blob made
                     from those bytes again, isr_decompress of that one
         "batch"     isr_compress_batch, then isr_decompress of every blob
         "serving"   isr_submit of every snapshot, isr_poll and
                     isr_decompress of each in turn
  sizes  the snapshots, "order:elements" each
  prec   "fp64", "fp32" or "bf16" (fp64 results are reconstructed to FP64,
         the others to FP32)
  tol    relative L2 bound
  jac    with per-element Jacobians
"""

import math

import numpy as np
import torch

from paper_2407_20731_amd import isr

NCOMP = 3
SHARE = 0.5  # of the error budget spent on quantisation
N_MODES, KMAX, NOISE = 64, 4.0, 1e-6


def _case(name, op, sizes, prec, tol=1e-3, jac=False):
    return {"name": name, "op": op, "sizes": sizes, "prec": prec, "tol": tol, "jac": jac}


def listed():
    return [
        # one rank's share of a strongly scaled run: launches and latency
        _case("n7_bf16_64", "snapshot", "7:64", "bf16"),
        # the 8^3 box
        _case("n7_fp32_512", "snapshot", "7:512", "fp32"),
        # the headline snapshot (805 MB) on the fast path
        _case("n7_bf16_65536", "snapshot", "7:65536", "bf16"),
        # the same snapshot where bit-reproducible results are wanted
        _case("n7_fp64_65536", "snapshot", "7:65536", "fp64"),
        # a lower order on a mesh of unequal cells
        _case("n5_fp32_jac_50001", "snapshot", "5:50001", "fp32", jac=True),
        # a higher order, a large snapshot
        _case("n9_bf16_32768", "snapshot", "9:32768", "bf16"),
        # a higher order in FP64, a ragged element count, a tight bound
        _case("n9_fp64_4097", "snapshot", "9:4097", "fp64", tol=1e-5),
        # the snapshots that a run has kept, reduced together
        _case("batch_bf16_8", "batch", "5:4096 7:50000 9:8191 7:12000 5:30001 9:20000 7:6007 5:100000", "bf16"),
        # requests of a running simulation, several resident at once
        _case("serving_fp32_10", "serving",
              "7:20000 5:7001 9:12007 7:1000 5:54000 9:3333 7:33000 5:20000 9:20000 7:9001", "fp32"),
        # every element within the bound by itself
        _case("elemcut_n7_8192", "elemcut", "7:8192", "fp64"),
        # kept coefficients as integer codes
        _case("quantized_n7_10007", "quantized", "7:10007", "fp64"),
        # a checkpoint written and read back
        _case("writer_n7_fp64_4096", "writer", "7:4096", "fp64"),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(["snapshot"] * 6 + ["batch", "serving", "elemcut", "quantized", "writer"])
    tol = rng.choice([1e-2, 1e-3, 1e-3])
    jac = False
    if op in ("batch", "serving"):
        prec = rng.choice(["fp32", "bf16"])
        sizes = []
        for _ in range(rng.randint(3, 8)):
            order = rng.choice([5, 7, 9])
            sizes.append("%d:%d" % (order, _log_uniform(rng, 1000, {5: 50000, 7: 25000, 9: 12000}[order])))
        sizes = " ".join(sizes)
    else:
        order = rng.choice([5, 7, 7, 9, 3, 4, 6, 8, 10, 11, 12])
        if op == "snapshot":
            prec = rng.choice(["fp64", "fp32", "bf16"])
            most = 25e6 if prec == "fp64" or order > 7 else 100e6  # values
            if prec != "bf16":
                tol = rng.choice([1e-2, 1e-3, 1e-4])
            jac = rng.random() < 0.25
        else:
            prec, most = "fp64", 10e6
        sizes = "%d:%d" % (order, _log_uniform(rng, 64, most / (NCOMP * (order + 1) ** 3)))
    return {"op": op, "sizes": sizes, "prec": prec, "tol": tol, "jac": jac}


def _snapshots(case):
    return [tuple(int(x) for x in s.split(":")) for s in case["sizes"].split()]


# ---- inputs ----------------------------------------------------------------


def _nodes(order):
    """Gauss-Lobatto-Legendre points and weights."""
    leg = np.polynomial.legendre.Legendre.basis(order)
    x = np.concatenate(([-1.0], np.sort(leg.deriv().roots().real), [1.0])) if order > 1 else np.array([-1.0, 1.0])
    return x, 2.0 / (order * (order + 1) * leg(x) ** 2)


def _field(order, n_elem, seed, device="cuda"):
    """A velocity snapshot [3, E, n, n, n]: a divergence-free sum of 64 Fourier
    modes with a k^-5/3 amplitude spectrum at the GLL points of cubes of edge
    2 pi / 8, each component of unit RMS, plus noise of 1e-6."""
    rng = np.random.default_rng(seed)
    k = rng.integers(-4, 5, size=(16 * N_MODES, 3))
    k2 = (k * k).sum(1)
    k = k[(k2 > 0) & (k2 <= KMAX * KMAX)][:N_MODES].astype(np.float64)
    norm = np.sqrt((k * k).sum(1))
    phase = rng.uniform(0.0, 2.0 * math.pi, len(k))
    d = rng.standard_normal((len(k), 3))
    d -= (d * k).sum(1, keepdims=True) * k / (norm * norm)[:, None]
    d /= np.sqrt((d * d).sum(1, keepdims=True))
    nx = max(1, math.ceil(n_elem ** (1.0 / 3.0) - 1e-9))
    nz = math.ceil(n_elem / (nx * nx))
    n, (x, _), h = order + 1, _nodes(order), math.pi / 4.0

    def waves(axis, blocks):
        at = ((np.arange(blocks)[:, None] + 0.5 * (x + 1.0)) * h).ravel()
        return torch.from_numpy(np.exp(1j * k[:, axis, None] * at)).to(device)

    ex, ey, ez = waves(0, nx), waves(1, nx), waves(2, nz)
    u = torch.empty((NCOMP, n_elem, n, n, n), dtype=torch.float64, device=device)
    for c in range(NCOMP):
        a = torch.from_numpy(norm ** (-5.0 / 3.0) * d[:, c] * np.exp(1j * phase)).to(device)
        for z0 in range(0, nz, 8):  # layers of blocks, to bound the products held
            z1 = min(nz, z0 + 8)
            zy = ((a[:, None] * ez[:, z0 * n:z1 * n])[:, :, None] * ey[:, None, :]).reshape(len(k), -1).t().contiguous()
            g = zy.real.contiguous() @ ex.real.contiguous() - zy.imag.contiguous() @ ex.imag.contiguous()
            g = g.reshape(z1 - z0, n, nx, n, nx, n).permute(0, 2, 4, 1, 3, 5).reshape(-1, n, n, n)
            e0, e1 = z0 * nx * nx, min(n_elem, z1 * nx * nx)
            if e1 > e0:
                u[c, e0:e1] = g[:e1 - e0]
        u[c] /= torch.sqrt(torch.mean(u[c] * u[c]))
    gen = torch.Generator(device=device)
    gen.manual_seed(seed)
    u += NOISE * torch.randn(u.shape, generator=gen, dtype=torch.float64, device=device)
    return u


def _jacobians(n_elem, seed, device="cuda"):
    gen = torch.Generator(device=device)
    gen.manual_seed(seed + 77)
    return 0.5 + torch.rand(n_elem, generator=gen, dtype=torch.float64, device=device)


_context = []


def _ctx():
    """The one library context that a program keeps."""
    if not _context:
        _context.append(isr.Context(device=0))
    return _context[0]


def prepare(case, seed):
    dtype = torch.float64 if case["prec"] == "fp64" else torch.float32
    fields = [_field(o, e, seed + 1000 * i) for i, (o, e) in enumerate(_snapshots(case))]
    values = sum(u.numel() for u in fields)
    return {
        "file": np.zeros(4096 + 10 * values, dtype=np.uint8) if case["op"] == "writer" else None,
        "case": case, "ctx": _ctx(), "orders": [o for o, _ in _snapshots(case)], "fields": fields,
        "jac": _jacobians(fields[0].shape[1], seed) if case["jac"] else None,
        "out": [torch.empty(u.shape, dtype=dtype, device=u.device) for u in fields],
    }


# ---- one pass --------------------------------------------------------------


def _result(ctx, blob, out):
    ctx.decompress(blob, out=out)
    s = blob.stats
    res = {"field": out, "kept": np.array(s["kept"], dtype=np.int64)}
    res.update((k, np.array(s[k])) for k in ("norm2", "rel_err"))
    if not math.isnan(s["tau"][0]):  # the per-element cut has no component threshold
        res["tau"] = np.array(s["tau"])
    return res


def run(state):
    case, ctx = state["case"], state["ctx"]
    op, prec, tol = case["op"], case["prec"], case["tol"]
    fields, orders, outs = state["fields"], state["orders"], state["out"]
    if op == "batch":
        blobs = ctx.compress_batch([(u, o, tol) for u, o in zip(fields, orders)], prec)
        res = [_result(ctx, b, out) for b, out in zip(blobs, outs)]
        for b in blobs:
            b.free()
        return res
    if op == "serving":
        ids = [ctx.submit(u, o, tol, prec) for u, o in zip(fields, orders)]
        res = []
        for i, out in zip(ids, outs):
            blob = ctx.poll(i, wait_ms=-1)
            res.append(_result(ctx, blob, out))
            blob.free()
        return res
    u, order, out = fields[0], orders[0], outs[0]
    if op == "elemcut":
        blob = ctx.compress_elemcut(u, order, tol, jac=state["jac"])
    elif op == "quantized":
        blob = ctx.compress_quantized(u, order, tol, SHARE)
    else:
        blob = ctx.compress(u, order, tol, prec, jac=state["jac"])
    if op == "writer":
        written = blob.to_bytes()
        state["file"][:len(written)] = np.frombuffer(written, dtype=np.uint8)
        again = ctx.blob_from_bytes(written)
        ctx.decompress(again, out=out)
        again.free()
        res = {"field": out, "file": state["file"], "length": len(written)}
    else:
        res = _result(ctx, blob, out)
    blob.free()
    return res


def work(case):
    """The field read once, the reconstruction written once, and between them
    one forward transform and one inverse; the blob (a few per cent of the
    field) is left out except where it goes to the host."""
    values = [NCOMP * e * (o + 1) ** 3 for o, e in _snapshots(case)]
    nbytes = sum(values) * (16 if case["prec"] == "fp64" else 12)
    flops = sum(v * 6 * (2 * o + 1) for v, (o, _) in zip(values, _snapshots(case)))
    return {"bytes": nbytes, "flops": flops}


# ---- the result in plain 64-bit arithmetic ---------------------------------


def _along(m, u):
    """m applied along each of the three node axes of u [E, n, n, n]."""
    e, n = u.shape[0], u.shape[1]
    for _ in range(3):  # contract the last axis, then bring the next one there
        u = (u.reshape(-1, n) @ m.t()).reshape(e, n, n, n).permute(0, 3, 1, 2).contiguous()
    return u


def _kept_above(e, budget):
    """Mask of the energies e [rows, m] kept per row when the smallest are
    dropped while their sum stays within the row's budget, and that sum."""
    v, _ = torch.sort(e, dim=1)
    s = torch.cumsum(v, dim=1)
    below = s - v  # sum of the energies before each one
    fits = below <= budget[:, None]
    last = (fits.sum(dim=1, keepdim=True) - 1).clamp(min=0)
    tau = torch.gather(v, 1, last)
    all_fit = s[:, -1:] <= budget[:, None]
    tau = torch.where(all_fit, torch.full_like(tau, math.inf), tau)
    kept = e >= tau
    return kept, tau[:, 0], (e * ~kept).sum(dim=1)


def _exact_one(case, order, u, jac):
    n, tol = order + 1, case["tol"]
    x, w = _nodes(order)
    vander = np.polynomial.legendre.legvander(x, order)
    gamma = 2.0 / (2.0 * np.arange(n) + 1.0)
    gamma[-1] = 2.0 / order
    dev = u.device
    to = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(dev)  # noqa: E731
    v, a = to(vander), to(np.linalg.inv(vander))
    w3 = to(w[:, None, None] * w[None, :, None] * w[None, None, :])
    g3 = to(gamma[:, None, None] * gamma[None, :, None] * gamma[None, None, :])
    j = torch.ones(u.shape[1], dtype=torch.float64, device=dev) if jac is None else jac
    field, stats = torch.empty_like(u), {"norm2": [], "tau": [], "rel_err": []}
    for c in range(u.shape[0]):
        coef = _along(a, u[c])
        e = (coef * coef * g3 * j[:, None, None, None]).reshape(u.shape[1], -1)
        elem2 = (u[c] * u[c] * w3).sum(dim=(1, 2, 3)) * j
        u2 = elem2.sum()
        if case["op"] == "elemcut":
            kept, tau, dropped = _kept_above(e, tol * tol * elem2)
        else:
            share = SHARE if case["op"] == "quantized" else 0.0
            kept, tau, dropped = _kept_above(e.reshape(1, -1), (tol * tol * u2 * (1.0 - share)).reshape(1))
        kept = kept.reshape(coef.shape)
        if case["op"] == "quantized":
            step = 2.0 * torch.sqrt((tol * tol * u2 - dropped[0]) / kept.sum()) * (1.0 - 2.0 ** -20)
            root = torch.sqrt(g3)
            coef = torch.round(coef * root / step) * step / root
        field[c] = _along(v, coef * kept)
        err2 = ((u[c] - field[c]) ** 2 * w3).sum(dim=(1, 2, 3)) @ j
        stats["norm2"].append(float(u2))
        stats["tau"].append(float(tau[0]))
        stats["rel_err"].append(float(torch.sqrt(err2 / u2)))
    return field, stats


def exact(case, seed):
    res = []
    for i, (order, n_elem) in enumerate(_snapshots(case)):
        u = _field(order, n_elem, seed + 1000 * i)
        field, stats = _exact_one(case, order, u, _jacobians(n_elem, seed) if case["jac"] else None)
        if case["op"] == "writer":
            res.append({"field": field})
        else:
            if case["op"] == "elemcut":
                del stats["tau"]
            res.append({"field": field, **{k: np.array(v) for k, v in stats.items()}})
    return res if case["op"] in ("batch", "serving") else res[0]
