"""Performance cases of the ST-HOSVD library: what its users run, by size, type and option.

A case is a flat dict: the operation (``op``), the tensor (``dims``, mode 1 fastest, and the planted
multilinear ranks, both as "AxBxC" texts; ``rho``, ``noise``), its storage ``dtype``, and the options
of the call (``eps`` or fixed ranks, ``gram`` and ``ttm`` arithmetic).  Tensors are planted Tucker
models with decaying cores plus noise, as the data that the method compresses has.  Every operation
goes through ``paper_1510_06689_amd.tucker``; a program that compresses a series of snapshots of one
shape keeps a ``Compressor`` (or a captured ``BatchCompressor``) and calls it for each, so these are
in the state.
"""
import math

import numpy as np
import torch

from paper_1510_06689_amd import tucker

DEVICE = "cuda:0"


def _case(name, op, dims, ranks, dtype="float64", gram="fp64", ttm="fp64", rho=0.7, noise=1e-5, eps=1e-4, fixed=False, sweeps=0, sizes=""):
    c = {"op": op, "dims": dims, "ranks": ranks, "dtype": dtype, "gram": gram, "ttm": ttm, "rho": rho, "noise": noise, "eps": eps, "fixed": fixed, "sweeps": sweeps,
         "sizes": sizes}
    return dict(c, name=name) if name else c


def listed():
    return [
        # the smallest call: one 32^3 block, all launches and read-backs
        _case("small_f64", "compress", "32x32x32", "4x5x6", rho=1.0, noise=1e-6),
        # an ordinary 3-way volume of odd extents; one mode above 256
        _case("volume_f64", "compress", "301x187x211", "14x11x17"),
        # an ordinary 5-way tensor of odd extents in single precision, mixed arithmetic; one mode above 128
        _case("ragged_mixed", "compress", "131x77x90x21x5", "13x12x11x6x3", dtype="float32", gram="split_bf16", ttm="bf16x3"),
        # the large combustion-shaped tensor, 17.2 GB in double precision
        _case("combustion128_f64", "compress", "128x128x128x32x32", "16x16x16x8x8"),
        # the same stored in single precision (8.6 GB), mixed arithmetic
        _case("combustion128_mixed", "compress", "128x128x128x32x32", "16x16x16x8x8", dtype="float32", gram="split_bf16", ttm="bf16x3"),
        # the paper's mode-order shape with its fixed ranks: wide modes, two of them kept at rank 100
        _case("paper250_f64", "compress", "25x250x250x250", "10x10x100x100", rho=0.98, fixed=True),
        # single-precision data whose tolerance asks for double-precision arithmetic, at high ranks
        _case("f32_fp64_highrank", "compress", "128x128x128x48", "64x56x48x20", dtype="float32", rho=0.95, noise=1e-6, eps=1e-5),
        # a tolerance near the square root of the unit roundoff: singular values from a QR instead of a Gram
        _case("qr_f64", "compress", "128x128x128x16", "16x16x16x8", gram="qr", noise=1e-8, eps=1e-7),
        # uneven problems compressed together, a captured graph replayed
        _case("batch12_mixed", "batch", "", "12x12x12x6", dtype="float32", gram="split_bf16", ttm="bf16x3", rho=0.6,
              sizes="24,31,38,44,52,59,64,70,77,83,90,96"),
        # Alg. 2 from the ST-HOSVD start, two sweeps on data with 5% noise
        _case("hooi_f64", "hooi", "100x100x100x50", "10x10x10x10", noise=0.05, fixed=True, sweeps=2),
        # decompression of the large single-precision tensor
        _case("reconstruct_f32", "reconstruct", "128x128x128x32x32", "16x16x16x8x8", dtype="float32", ttm="bf16x3"),
        # decompression in double precision at odd extents, and its error metrics against the data
        _case("verify_f64", "verify", "121x83x67x29", "14x11x17x9"),
    ]


def _sizes(rng, ndim, elements, most):
    """ndim extents whose product is near `elements`, each between 4 and `most`, uneven and often odd."""
    w = [rng.uniform(0.6, 1.4) for _ in range(ndim)]
    s = sum(w)
    return [max(4, min(most, round(elements ** (v / s)))) for v in w]


def draw(rng):
    kind = rng.choice(["compress_f64", "compress_f64", "mixed", "mixed", "f32_fp64", "fixed", "qr", "batch", "hooi", "reconstruct", "verify"])
    if kind == "batch":
        count = rng.randint(5, 12)
        return _case("", "batch", "", "12x12x12x6", dtype="float32", gram="split_bf16", ttm="bf16x3", rho=0.6,
                     sizes=",".join(str(rng.randint(24, 96)) for _ in range(count)))
    ndim = rng.choice([3, 3, 4, 4, 5])
    top = {"qr": 3e7, "hooi": 6e7, "mixed": 4e8}.get(kind, 2e8)
    dims = _sizes(rng, ndim, math.exp(rng.uniform(math.log(3e4), math.log(top))), 128 if kind == "qr" else 400)
    high = kind in ("f32_fp64", "fixed") and rng.random() < 0.5
    ranks = [max(2, min(64 if high else 20, int(d * rng.uniform(0.2, 0.5) if high else d * rng.uniform(0.08, 0.3)))) for d in dims]
    for n in range(ndim):  # an unfolding's rank is at most the product of the other ranks
        ranks[n] = max(1, min(ranks[n], math.prod(ranks) // ranks[n] // 2))
    rho = round(max(0.7, 0.003 ** (1 / max(1, max(ranks) - 1))), 3)
    d, r = "x".join(map(str, dims)), "x".join(map(str, ranks))
    if kind == "compress_f64":
        return _case("", "compress", d, r, rho=rho)
    if kind == "mixed":
        return _case("", "compress", d, r, dtype="float32", gram="split_bf16", ttm="bf16x3", rho=rho)
    if kind == "f32_fp64":
        return _case("", "compress", d, r, dtype="float32", rho=rho, noise=1e-6, eps=1e-5)
    if kind == "fixed":
        return _case("", "compress", d, r, rho=rho, fixed=True)
    if kind == "qr":
        return _case("", "compress", d, r, gram="qr", rho=rho, noise=1e-8, eps=1e-7)
    if kind == "hooi":
        return _case("", "hooi", d, r, rho=rho, noise=0.05, fixed=True, sweeps=2)
    if kind == "reconstruct":
        f32 = rng.random() < 0.5
        return _case("", "reconstruct", d, r, dtype="float32" if f32 else "float64", ttm="bf16x3" if f32 else "fp64", rho=rho)
    return _case("", "verify", d, r, rho=rho)


# ----------------------------------------------------------------- inputs

def _ints(text):
    return [int(v) for v in text.split("x")]


def _batch_dims(case):
    """s x s x s x 16 for each size, and the planted ranks capped by the extents."""
    top = _ints(case["ranks"])
    dims = [[int(s)] * 3 + [16] for s in case["sizes"].split(",")]
    return [(d, [min(r, k) for r, k in zip(top, d)]) for d in dims]


def _model(dims, ranks, rho, gen):
    """A core (N-way, C order of the reversed modes) with decaying entries and smooth orthonormal factors."""
    factors = []
    for i, r in zip(dims, ranks):
        a = torch.cos(math.pi * (torch.arange(i, dtype=torch.float64, device=DEVICE)[:, None] + 0.5) * torch.arange(r, dtype=torch.float64, device=DEVICE) / i)
        q, t = torch.linalg.qr(a + 0.1 / math.sqrt(i) * torch.randn(i, r, generator=gen, dtype=torch.float64, device=DEVICE))
        factors.append(q * torch.sign(torch.diagonal(t)))
    core = torch.randn(ranks[::-1], generator=gen, dtype=torch.float64, device=DEVICE)
    for n, r in enumerate(ranks):
        core *= (rho ** torch.arange(r, dtype=torch.float64, device=DEVICE)).view([-1 if k == len(ranks) - 1 - n else 1 for k in range(len(ranks))])
    return core, factors


def _times(x, mode, m):
    """x (C order of the reversed modes) times the K x J matrix m in `mode`, in the same order of axes."""
    lead, j = x.shape[: x.dim() - 1 - mode], x.shape[x.dim() - 1 - mode]
    tail = x.shape[x.dim() - mode:]
    z = torch.matmul(x.reshape(-1, j), m.t()) if mode == 0 else torch.matmul(m, x.reshape(-1, j, math.prod(tail)))
    return z.reshape(lead + (m.shape[0],) + tail)


def _expand(core, factors):
    x = core
    for n in sorted(range(len(factors)), key=lambda k: factors[k].shape[0] / factors[k].shape[1]):
        x = _times(x, n, factors[n])
    return x


def _planted(dims, ranks, case, gen):
    core, factors = _model(dims, ranks, case["rho"], gen)
    x = _expand(core, factors)
    sigma = case["noise"] * float(core.norm()) / math.sqrt(x.numel())
    for part in x.view(x.shape[0], -1).split(max(1, (1 << 28) * x.shape[0] // x.numel())):
        part.add_(torch.randn(part.shape, generator=gen, dtype=torch.float64, device=DEVICE), alpha=sigma)
    return x if case["dtype"] == "float64" else x.to(torch.float32)


def _fortran(x):
    """The logical (I_1, ..., I_N) view, mode 1 fastest in memory."""
    return x.permute(*reversed(range(x.dim())))


def _inputs(case, seed):
    """Plain tensors (C order of the reversed modes), from the seed alone."""
    gen = torch.Generator(device=DEVICE)
    gen.manual_seed(seed)
    if case["op"] == "batch":
        return [_planted(d, r, case, gen) for d, r in _batch_dims(case)]
    dims, ranks = _ints(case["dims"]), _ints(case["ranks"])
    if case["op"] in ("reconstruct", "verify"):
        core, factors = _model(dims, ranks, case["rho"], gen)
        x = None
        if case["op"] == "verify":  # the data that the model was computed from
            x = _expand(core, factors)
            x.add_(torch.randn(x.shape, generator=gen, dtype=torch.float64, device=DEVICE), alpha=case["noise"] * float(core.norm()) / math.sqrt(x.numel()))
        return core if case["dtype"] == "float64" else core.to(torch.float32), factors, x
    return _planted(dims, ranks, case, gen)


def prepare(case, seed):
    state = {"case": case}
    made = _inputs(case, seed)
    if case["op"] == "batch":
        state["batch"] = tucker.BatchCompressor([_fortran(x) for x in made], case["eps"], ttm_precision=case["ttm"])
        state["batch"].capture()
    elif case["op"] in ("reconstruct", "verify"):
        core, factors, x = made
        state.update(core=_fortran(core), factors=[u.t().contiguous().t() for u in factors], x=None if x is None else _fortran(x))
    else:
        state["x"] = _fortran(made)
        state["compressor"] = tucker.Compressor(_ints(case["dims"]), made.dtype, DEVICE, case["eps"], ranks=_ints(case["ranks"]) if case["fixed"] else None,
                                                gram_precision=case["gram"], ttm_precision=case["ttm"])
    return state


def _answer(t):
    return {"core": t.core, "factors": t.factors, "eigvals": t.eigvals, "ranks": np.array(t.ranks), "energies": np.array([t.norm2, *t.discarded])}


def run(state):
    case = state["case"]
    if case["op"] == "compress":
        state["compressor"].run(state["x"])
        return _answer(state["compressor"].result())
    if case["op"] == "hooi":
        fits = state["compressor"].run_hooi(state["x"], max_sweeps=case["sweeps"], tol=-1.0)
        t = state["compressor"].result()
        return {"core": t.core, "factors": t.factors, "fits": np.array([t.norm2, *fits])}
    if case["op"] == "batch":
        state["batch"].replay()
        state["batch"].finish()
        got = state["batch"].results()
        return {"cores": [t.core for t in got], "factors": [t.factors for t in got], "ranks": np.array([t.ranks for t in got]),
                "energies": np.array([[t.norm2, *t.discarded] for t in got])}
    xhat = tucker.reconstruct(state["core"], state["factors"], precision=case["ttm"])
    if case["op"] == "reconstruct":
        return xhat
    return {"xhat": xhat, "metrics": np.array(tucker.error_metrics(state["x"], xhat))}


# ------------------------------------------------------------------- work

def _sthosvd_flops(dims, ranks, qr=False):
    """Gram (its distinct entries; for the QR path the Householder QR) and product of every mode."""
    cur, flops = list(dims), 0.0
    for n, r in enumerate(ranks):
        size = math.prod(cur)
        flops += (2.0 * size * cur[n] if qr else (cur[n] + 1.0) * size) + 2.0 * r * size
        cur[n] = r
    return flops


def work(case):
    b = 8 if case["dtype"] == "float64" else 4
    if case["op"] == "batch":
        each = _batch_dims(case)
        return {"bytes": sum(b * (math.prod(d) + math.prod(r)) + 8 * sum(i * k for i, k in zip(d, r)) for d, r in each), "flops": sum(_sthosvd_flops(d, r) for d, r in each)}
    dims, ranks = _ints(case["dims"]), _ints(case["ranks"])
    full, core, fac = math.prod(dims), math.prod(ranks), 8 * sum(i * r for i, r in zip(dims, ranks))
    if case["op"] in ("reconstruct", "verify"):
        cur, flops = list(ranks), 0.0
        for n in sorted(range(len(dims)), key=lambda k: dims[k] / ranks[k]):
            flops += 2.0 * math.prod(cur) * dims[n]
            cur[n] = dims[n]
        more = full if case["op"] == "verify" else 0
        return {"bytes": b * (full + core + more) + fac, "flops": flops + 5.0 * more}
    flops = _sthosvd_flops(dims, ranks, case["gram"] == "qr")
    for _ in range(case["sweeps"]):
        for n in range(len(dims)):
            cur = list(dims)
            for m in range(len(dims)):
                if m != n:
                    flops += 2.0 * ranks[m] * math.prod(cur)
                    cur[m] = ranks[m]
            flops += (dims[n] + 1.0) * math.prod(cur)
    return {"bytes": b * (full + core) + fac, "flops": flops}


# ----------------------------------------------------- the same in 64 bits

def _rows(x, mode):
    """The mode's unfolding, J x (all other indices), of x in C order of the reversed modes."""
    return x.movedim(x.dim() - 1 - mode, 0).reshape(x.shape[x.dim() - 1 - mode], -1)


def _spectrum(y, mode, qr=False):
    """Squared singular values, descending, and left singular vectors of the unfolding, each with its largest entry positive."""
    a = _rows(y, mode)
    if qr:
        v, s, _ = np.linalg.svd(np.linalg.qr(a.t().cpu().numpy(), mode="r").T)
        lam = np.zeros(a.shape[0])
        lam[: s.size] = s * s
    else:
        lam, v = np.linalg.eigh(torch.matmul(a, a.t()).cpu().numpy())
        lam, v = lam[::-1].copy(), v[:, ::-1]
    v = v * np.sign(v[np.argmax(np.abs(v), axis=0), np.arange(v.shape[1])])
    return lam, v


def _exact_sthosvd(x, case, ranks):
    n2, n = float((x * x).sum()), x.dim()
    y, factors, spectra, found, lost = x, [], [], [], []
    for mode in range(n):
        lam, v = _spectrum(y, mode, case["gram"] == "qr")
        tail = np.append(np.cumsum(np.maximum(lam, 0)[::-1])[::-1], 0.0)
        r = ranks[mode] if case["fixed"] else max(1, int(np.argmax(tail <= case["eps"] ** 2 * n2 / n)))
        u = torch.from_numpy(np.ascontiguousarray(v[:, :r])).to(DEVICE)
        y = _times(y, mode, u.t())
        factors.append(u)
        spectra.append(torch.from_numpy(lam))
        found.append(r)
        lost.append(float(tail[r]))
    return {"core": _fortran(y), "factors": factors, "eigvals": spectra, "ranks": np.array(found), "energies": np.array([n2, *lost])}


def exact(case, seed):
    made = _inputs(case, seed)
    if case["op"] == "batch":
        got = [_exact_sthosvd(x.double(), case, None) for x in made]
        return {"cores": [t["core"] for t in got], "factors": [t["factors"] for t in got], "ranks": np.array([t["ranks"] for t in got]),
                "energies": np.array([t["energies"] for t in got])}
    if case["op"] in ("reconstruct", "verify"):
        core, factors, x = made
        xhat = _expand(core.double(), factors)
        if case["op"] == "reconstruct":
            return _fortran(xhat)
        d = x - xhat
        return {"xhat": _fortran(xhat), "metrics": np.array([float((d * d).sum()), float(d.abs().max()), float((x * x).sum())])}
    x = made.double()
    t = _exact_sthosvd(x, case, _ints(case["ranks"]))
    if case["op"] == "compress":
        return t
    n, fits = x.dim(), [t["energies"][0], t["energies"][0] - float((t["core"] ** 2).sum())]
    for _ in range(case["sweeps"]):
        for mode in range(n):
            y = x
            for m in range(n):
                if m != mode:
                    y = _times(y, m, t["factors"][m].t())
            _, v = _spectrum(y, mode)
            t["factors"][mode] = torch.from_numpy(np.ascontiguousarray(v[:, : t["ranks"][mode]])).to(DEVICE)
        core = _times(y, n - 1, t["factors"][n - 1].t())
        fits.append(t["energies"][0] - float((core ** 2).sum()))
    return {"core": _fortran(core), "factors": t["factors"], "fits": np.array(fits)}
