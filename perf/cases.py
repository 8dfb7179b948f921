"""Timed cases of the library: what its users have it do, through the Python entry points.

A case is a dict of plain values.  ``listed()`` names the standing ones, ``draw(rng)``
gives another case of the same ranges.  ``prepare(case, seed)`` makes the inputs on the
GPU, ``run(state)`` is one pass, ``work(case)`` the bytes and operations a pass cannot
do without, and ``exact(case, seed)`` the outputs of plain float64 torch for the same
inputs (None in the place of an output without such a value).

Kinds of case:

* ``fit``    one curve: ``fit`` (power or Chebyshev basis, float64 or compensated sums)
* ``resid``  one curve and the table of its errors: ``fit`` then ``residuals(store=True)``
* ``qr``     one curve through the orthogonal factorisation: ``fit_qr``
* ``batch``  many curves in one call: ``fit_batched`` (with or without a plan)
* ``qrb``    many curves through the factorisation: ``fit_qr_batched``
* ``grad``   a differentiable batch inside a training step: ``lsefit`` and its backward
"""
import math

import numpy as np
import torch

import paper_1512_08017_amd as lf

DEV = "cuda"
CHUNK = 1 << 24                      # points made (or summed) at a time
DT = {"f32": torch.float32, "f64": torch.float64}


def listed():
    return [
        # a few thousand measurements, one call: a calibration or a trend line in a
        # program that waits for it; launches and host time are all there is
        _fit("fit_small_f64", 4_097, 3, "f64"),
        # a million float64 readings and a straight line
        _fit("fit_linear_f64", 1_000_000, 1, "f64", lo=0.0, hi=10.0, noise=0.5),
        # x far from zero: time stamps or frequencies in a narrow window, degree 5
        _fit("fit_quintic_f32", 10_000_000, 5, "f32", lo=1000.0, hi=1001.0, noise=1e-4),
        # the benchmark: a cubic through 1e8 float32 points
        _fit("fit_cubic_f32", 100_000_000, 3, "f32", noise=0.01),
        # the compensated float32 sums with their refinement pass, an odd size
        _fit("fit_cubic_f32c", 30_000_001, 3, "f32", noise=0.01, precision="f32c"),
        # a smooth curve that no low degree describes: Chebyshev basis, range from the data
        _fit("fit_runge_cheb", 100_000_000, 12, "f32", noise=1e-3, basis="chebyshev"),
        # the orthogonal route, chosen where the normal equations are not trusted
        dict(_fit("qr_quintic_f32", 10_000_000, 5, "f32", noise=1e-4), kind="qr"),
        # the table of fitted errors: every residual written back
        dict(_fit("resid_cubic_f64", 10_000_000, 3, "f64", noise=0.1), kind="resid"),
        # many curves of very different lengths, the largest job
        _batch("batch_ragged_f32", 65_536, 16, 65_536, 3, "f32", lo=-5.0, hi=5.0, noise=0.1),
        # many short curves: pixels, sensors, windows of a signal
        _batch("batch_short_f32", 65_536, 16, 256, 3, "f32", lo=-5.0, hi=5.0, noise=0.1),
        # a training step through the fit: forward and backward
        dict(_batch("grad_batch_f32", 4_096, 4_096, 4_096, 2, "f32", noise=0.05, mixed=False), kind="grad"),
        # the same in float64 on a small batch, as in a test or a small model
        dict(_batch("grad_small_f64", 100, 50, 2_000, 3, "f64", noise=0.05, mixed=False), kind="grad"),
    ]


def _fit(name, n, degree, dtype, lo=-1.0, hi=1.0, noise=0.1, precision="f64", basis="monomial", solver="gepp",
         given=False):
    return {"name": name, "kind": "fit", "n": n, "degree": degree, "dtype": dtype, "lo": lo, "hi": hi,
            "noise": noise, "precision": precision, "basis": basis, "solver": solver, "given": given}


def _batch(name, fits, shortest, longest, degree, dtype, lo=-1.0, hi=1.0, noise=0.1, mixed=True, precision="f64",
           basis="monomial", solver="gepp", given=False, plan=False):
    return {"name": name, "kind": "batch", "fits": fits, "shortest": shortest, "longest": longest, "degree": degree,
            "dtype": dtype, "lo": lo, "hi": hi, "noise": noise, "mixed": mixed, "precision": precision,
            "basis": basis, "solver": solver, "given": given, "plan": plan}


def _log_int(rng, lo, hi):
    """An integer spread over the logarithm of [lo, hi]."""
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["fit", "fit", "fit", "cheb", "resid", "qr", "batch", "batch", "batch", "qrb", "grad", "grad"])
    dtype = rng.choice(["f32", "f32", "f64"])
    solver = rng.choice(["gepp", "gepp", "gepp", "cholesky"])
    given = rng.random() < 0.25
    if kind in ("fit", "cheb", "resid", "qr"):
        top = 100_000_000 if kind == "fit" else 50_000_000
        n = _log_int(rng, 1_000, top) // (2 if dtype == "f64" else 1) + 1
        degree = rng.randint(1, 5) if rng.random() < 0.8 else rng.randint(6, 8)
        # away from [-1, 1] only low degrees: higher powers of t lose the comparison to their conditioning
        lo, hi = rng.choice([(-1.0, 1.0), (0.0, 10.0), (1000.0, 1001.0)]) if degree <= 3 else (-1.0, 1.0)
        c = _fit("", n, degree, dtype, lo=lo, hi=hi, noise=rng.choice([1e-3, 0.05, 0.5]), solver=solver, given=given)
        if kind == "fit" and dtype == "f32" and rng.random() < 0.3:
            c["precision"] = "f32c"
        if kind == "cheb":
            c.update(basis="chebyshev", degree=rng.randint(4, 16), lo=-1.0, hi=1.0)
        if kind in ("resid", "qr"):
            c.update(kind=kind, solver="gepp")
        if kind == "qr" and c["lo"] > 100:
            c.update(lo=0.0, hi=10.0)   # float32 x of a narrow window far from zero repeat, which rounds differently
    else:
        # mean length of log-uniform lengths is (hi - lo) / ln(hi / lo); the total stays below the largest listed one
        shortest = _log_int(rng, 16, 1_024)
        longest = shortest if rng.random() < 0.3 else _log_int(rng, shortest, 65_536)
        most = 2.0e8 if dtype == "f32" else 1.0e8
        mean = shortest if longest == shortest else (longest - shortest) / math.log(longest / shortest)
        fits = _log_int(rng, 16, max(32, min(65_536, int(most / mean))))
        c = _batch("", fits, shortest, longest, rng.randint(1, 3), dtype, lo=-1.0, hi=1.0, noise=0.1, solver=solver,
                   given=given)
        if kind == "batch":
            c["plan"] = rng.random() < 0.25
            what = rng.random()
            if what < 0.2 and dtype == "f32":
                c["precision"] = "f32c"
            elif what < 0.4:
                c.update(basis="chebyshev", degree=rng.randint(2, 8) if shortest >= 64 else 3)
        elif kind == "qrb":
            c.update(kind="qrb", solver="gepp")
        else:
            c.update(kind="grad", mixed=False)
    del c["name"]
    return c


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
def _lengths(case, seed):
    """Log-uniform lengths: the same multiset for every seed (so that a case is a fixed
    amount of work), in an order of the seed's own."""
    r = np.random.default_rng([case["fits"], case["shortest"], case["longest"]])
    u = r.uniform(math.log(case["shortest"]), math.log(case["longest"] + 1e-9), case["fits"])
    n = np.clip(np.floor(np.exp(u)), case["shortest"], case["longest"]).astype(np.int64)
    if seed is not None:
        np.random.default_rng(seed).shuffle(n)
    return n


def _points(case):
    return case["n"] if "n" in case else int(_lengths(case, None).sum())


def _horner(coef, u):
    """sum_k coef[..., k] u^k over the last axis of coef (one polynomial, or one per point)."""
    out = torch.zeros_like(u)
    for k in range(coef.shape[-1] - 1, -1, -1):
        out = out * u + coef[..., k]
    return out


def _single_data(case, seed):
    g = torch.Generator(device=DEV).manual_seed(seed)
    n, dt, lo, hi = case["n"], DT[case["dtype"]], case["lo"], case["hi"]
    mid = 0.5 * (lo + hi) if lo > 100 else 0.0
    coef = torch.randn(case["degree"] + 1, generator=g, device=DEV, dtype=torch.float64)
    x = torch.empty(n, dtype=dt, device=DEV)
    y = torch.empty(n, dtype=dt, device=DEV)
    for a in range(0, n, CHUNK):
        b = min(n, a + CHUNK)
        u = torch.rand(b - a, generator=g, device=DEV, dtype=torch.float64) * (hi - lo) + lo
        e = torch.randn(b - a, generator=g, device=DEV, dtype=torch.float32)
        x[a:b] = u
        f = 1.0 / (1.0 + 25.0 * u * u) if case["basis"] == "chebyshev" else _horner(coef, u - mid)
        y[a:b] = f + case["noise"] * e
    return x, y


def _batch_data(case, seed):
    g = torch.Generator(device=DEV).manual_seed(seed)
    n = _lengths(case, seed)
    fits, dt, top = case["fits"], DT[case["dtype"]], case["degree"]
    off = np.zeros(fits + 1, dtype=np.int64)
    np.cumsum(n, out=off[1:])
    offsets = torch.from_numpy(off).to(DEV)
    if case["mixed"]:
        degrees = torch.randint(1, top + 1, (fits,), generator=g, device=DEV).to(torch.int32)
    else:
        degrees = torch.full((fits,), top, dtype=torch.int32, device=DEV)
    coef = torch.randn(fits, top + 1, generator=g, device=DEV, dtype=torch.float64)
    coef = coef * (torch.arange(top + 1, device=DEV)[None, :] <= degrees[:, None])
    total = int(off[-1])
    x = torch.empty(total, dtype=dt, device=DEV)
    y = torch.empty(total, dtype=dt, device=DEV)
    for a in range(0, total, CHUNK):
        b = min(total, a + CHUNK)
        u = torch.rand(b - a, generator=g, device=DEV, dtype=torch.float64) * (case["hi"] - case["lo"]) + case["lo"]
        e = torch.randn(b - a, generator=g, device=DEV, dtype=torch.float32)
        f = torch.searchsorted(offsets, torch.arange(a, b, device=DEV), right=True) - 1
        x[a:b] = u
        y[a:b] = _horner(coef[f], u) + case["noise"] * e
    grad = torch.randn(fits, top + 1, generator=g, device=DEV, dtype=torch.float64)
    return x, y, offsets, degrees, grad


def _range_args(case):
    """center and scale for a caller who knows the interval its x lie in."""
    if not case["given"]:
        return {}
    return {"center": 0.5 * (case["lo"] + case["hi"]), "scale": 0.5 * (case["hi"] - case["lo"])}


def prepare(case, seed):
    s = {"case": case, "kw": _range_args(case)}
    if "n" in case:
        s["x"], s["y"] = _single_data(case, seed)
        if case["kind"] != "qr":
            s["kw"].update(solver=case["solver"], basis=case["basis"], precision=case["precision"])
        return s
    s["x"], s["y"], s["offsets"], s["degrees"], s["grad"] = _batch_data(case, seed)
    if case["kind"] == "grad":
        s["x"].requires_grad_(True)
        s["y"].requires_grad_(True)
        s["kw"].update(precision=case["precision"], basis=case["basis"])
    elif case["kind"] == "batch":
        s["kw"].update(solver=case["solver"], basis=case["basis"], precision=case["precision"])
        if case["plan"]:   # a program that repeats one shape keeps the plan and the result buffers
            top = case["degree"]
            s["kw"]["plan"] = lf.Plan(case["fits"], top, dtype=DT[case["dtype"]], precision=case["precision"])
            s["kw"]["out"] = (torch.zeros(case["fits"], top + 1, dtype=torch.float64, device=DEV),
                              torch.empty(case["fits"], dtype=torch.int32, device=DEV))
    return s


# ---------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------
def run(s):
    case, kind, m = s["case"], s["case"]["kind"], s["case"]["degree"]
    x, y, kw = s["x"], s["y"], s["kw"]
    if kind == "fit":
        r = lf.fit(x, y, m, **kw)
        other = r.coef_cheb if case["basis"] == "chebyshev" else r.coef_t
        return {"coef": r.coef, "basis": other, "status": r.status, "moments": r.moments}
    if kind == "resid":
        r = lf.fit(x, y, m, **kw)
        sse, e = lf.residuals(x, y, r, store=True)
        return {"coef": r.coef, "status": r.status, "sse": sse, "residuals": e}
    if kind == "qr":
        r = lf.fit_qr(x, y, m, **kw)
        return {"coef": r.coef, "basis": r.coef_t, "status": r.status, "info": r.info}
    off, deg = s["offsets"], s["degrees"]
    if kind == "batch":
        coef, status, _ = lf.fit_batched(x, y, off, deg, m, **kw)
        return {"coef": coef, "status": status}
    if kind == "qrb":
        coef, status, sse, _ = lf.fit_qr_batched(x, y, off, deg, m, **kw)
        return {"coef": coef, "status": status, "sse": sse}
    coef = lf.lsefit(x, y, off, deg, m, **kw)
    gx, gy = torch.autograd.grad(coef, (x, y), grad_outputs=s["grad"])
    return {"coef": coef, "grad_x": gx, "grad_y": gy}


def work(case):
    """Each point read once, each result written once (per point where results are per
    point); operations of the sums the method names: 2m power sums and m+1 products."""
    size = 4 if case["dtype"] == "f32" else 8
    n, m, kind = _points(case), case["degree"], case["kind"]
    fits = case.get("fits", 1)
    moved = n * 2 * size + fits * 8 * (m + 1) + (fits * 12 if fits > 1 else 0)
    ops = n * (7 * m + 2)
    if kind == "resid":
        moved += n * size
        ops += n * (2 * m + 3)
    if kind == "grad":
        moved += n * 2 * size + fits * 8 * (m + 1)
        ops += n * (8 * m + 6)
    if kind in ("qr", "qrb"):
        ops = n * (m + 1) * (m + 2) * 2
    return {"bytes": float(moved), "flops": float(ops)}


# ---------------------------------------------------------------------------
# the same outputs in plain float64 torch
# ---------------------------------------------------------------------------
def _basis(u, m):
    """Legendre polynomials P_0..P_m of u, a column each."""
    cols = [torch.ones_like(u), u]
    for k in range(1, m):
        cols.append(((2 * k + 1) * u * cols[k] - k * cols[k - 1]) / (k + 1))
    return torch.stack(cols[:m + 1], dim=-1)


def _to_powers(c, mid, half, m):
    """Coefficients of powers of x from Legendre coefficients of u = (x - mid)/half, in
    long double on the host (the change of basis cancels at higher degree)."""
    P = np.zeros((m + 1, m + 1), dtype=np.longdouble)
    P[0, 0] = 1
    if m:
        P[1, 1] = 1
    for k in range(1, m):
        P[k + 1, 1:] += np.longdouble(2 * k + 1) / (k + 1) * P[k, :-1]
        P[k + 1] -= np.longdouble(k) / (k + 1) * P[k - 1]
    b = c.astype(np.longdouble) @ P                        # powers of u
    mid, half = np.asarray(mid, np.longdouble), np.asarray(half, np.longdouble)
    a = np.zeros_like(b)
    for k in range(m + 1):
        for j in range(k, m + 1):
            a[..., k] += b[..., j] * math.comb(j, k) * (-mid) ** (j - k) / half ** j
    return a.astype(np.float64)


def _to_chebyshev(case, x, c, mid, half, m):
    """Chebyshev coefficients over the basis' own interval (the data's extent, or the given one)."""
    k = np.arange(m + 1)
    t = np.cos((k + 0.5) * np.pi / (m + 1))
    if case["given"]:
        c0, s0 = 0.5 * (case["lo"] + case["hi"]), 0.5 * (case["hi"] - case["lo"])
    else:
        lo, hi = float(x.min()), float(x.max())
        c0, s0 = 0.5 * hi + 0.5 * lo, 0.5 * hi - 0.5 * lo
    u = torch.from_numpy((c0 + s0 * t - mid) / half)
    f = (_basis(u, m) @ torch.from_numpy(c)).numpy()
    out = np.array([2.0 / (m + 1) * np.sum(f * np.cos(j * (k + 0.5) * np.pi / (m + 1))) for j in k])
    out[0] *= 0.5
    return out


def _exact_single(case, seed):
    x, y = _single_data(case, seed)
    n, m = case["n"], case["degree"]
    mid, half = 0.5 * (case["lo"] + case["hi"]), 0.5 * (case["hi"] - case["lo"])
    step = CHUNK // 4

    def parts():
        for a in range(0, n, step):
            V = _basis((x[a:a + step].double() - mid) / half, m)
            yield a, V, y[a:a + step].double()

    G = torch.zeros(m + 1, m + 1, dtype=torch.float64, device=DEV)
    r = torch.zeros(m + 1, dtype=torch.float64, device=DEV)
    for _, V, v in parts():
        Vt = V.t().contiguous()
        G += Vt @ V
        r += Vt @ v
    c = torch.linalg.solve(G, r)
    for _ in range(2):                                     # refinement with the data's own residuals
        r.zero_()
        for _, V, v in parts():
            r += V.t().contiguous() @ (v - V @ c)
        c = c + torch.linalg.solve(G, r)
    host = c.cpu().numpy()
    out = {"coef": _to_powers(host, mid, half, m), "status": None}
    if case["kind"] == "fit":
        out["moments"] = out["basis"] = None
        if case["basis"] == "chebyshev":
            out["basis"] = _to_chebyshev(case, x, host, mid, half, m)
    elif case["kind"] == "qr":
        out["basis"] = out["info"] = None
    else:
        e = torch.empty(n, dtype=torch.float64, device=DEV)
        for a, V, v in parts():
            e[a:a + step] = v - V @ c
        out["sse"] = (e * e).sum().reshape(1)
        out["residuals"] = e
    return out


def _exact_batch(case, seed):
    x, y, off, deg, grad = _batch_data(case, seed)
    if case["basis"] == "chebyshev" and not case["given"]:
        return None                                        # each fit has an interval of its own
    fits, m, total = case["fits"], case["degree"], x.numel()
    mid, half = 0.5 * (case["lo"] + case["hi"]), 0.5 * (case["hi"] - case["lo"])
    mask = (torch.arange(m + 1, device=DEV)[None, :] <= deg[:, None]).double()
    eye = torch.diag_embed(1.0 - mask)
    bounds = off.cpu().numpy()
    cuts = [0]                                             # whole fits, about CHUNK points at a time
    while cuts[-1] < fits:
        cuts.append(max(cuts[-1] + 1, int(np.searchsorted(bounds, bounds[cuts[-1]] + CHUNK, side="right")) - 1))
    coef = torch.zeros(fits, m + 1, dtype=torch.float64, device=DEV)
    sse = torch.zeros(fits, dtype=torch.float64, device=DEV)
    gx = torch.zeros(total, dtype=torch.float64, device=DEV) if case["kind"] == "grad" else None
    gy = torch.zeros_like(gx) if gx is not None else None
    x, y = x.detach(), y.detach()
    for f0, f1 in zip(cuts, cuts[1:]):
        a, b = int(bounds[f0]), int(bounds[f1])
        n = (off[f0 + 1:f1 + 1] - off[f0:f1])
        idx = torch.repeat_interleave(torch.arange(f1 - f0, device=DEV), n)
        u, v = (x[a:b].double() - mid) / half, y[a:b].double()
        V = _basis(u, m)

        def sums(z):
            return torch.segment_reduce(z.contiguous(), "sum", lengths=n, unsafe=True)

        mk = mask[f0:f1]
        G = torch.zeros(f1 - f0, m + 1, m + 1, dtype=torch.float64, device=DEV)
        for i in range(m + 1):
            for j in range(i, m + 1):
                G[:, i, j] = G[:, j, i] = sums(V[:, i] * V[:, j])
        G = G * mk[:, :, None] * mk[:, None, :] + eye[f0:f1]

        def solve(rhs):
            return torch.linalg.solve(G, (rhs * mk)[:, :, None])[:, :, 0]

        c = torch.zeros(f1 - f0, m + 1, dtype=torch.float64, device=DEV)
        for _ in range(3):                                 # a solve and two refinements
            e = v - (V * c[idx]).sum(1)
            c = c + solve(torch.stack([sums(V[:, k] * e) for k in range(m + 1)], 1))
        e = v - (V * c[idx]).sum(1)
        coef[f0:f1], sse[f0:f1] = c, sums(e * e)
        if gx is not None:
            # dL/dc in the Legendre basis: a = P c with P the change to powers of x
            P = torch.from_numpy(_to_powers(np.eye(m + 1), mid, half, m)).to(DEV)     # row k: powers of P_k
            lam = solve(grad[f0:f1] @ P.t())
            D = torch.zeros_like(V)                        # derivatives of the basis with respect to u
            for k in range(1, m + 1):
                D[:, k] = k * V[:, k - 1] + u * D[:, k - 1]
            q, dq = (V * lam[idx]).sum(1), (D * lam[idx]).sum(1)
            df = (D * c[idx]).sum(1)
            gy[a:b] = q
            gx[a:b] = (dq * e - q * df) / half
    host = coef.cpu().numpy()
    if case["basis"] == "chebyshev":                       # the given interval is the basis' own
        k = np.arange(m + 1)
        T = np.cos(np.outer(k + 0.5, k) * np.pi / (m + 1))                            # T_j at the nodes
        node = _basis(torch.from_numpy(np.cos((k + 0.5) * np.pi / (m + 1))), m).numpy()
        rows = np.linalg.solve(T, node @ host.T).T * mask.cpu().numpy()
        for f, d in enumerate(deg.tolist()):               # center and scale follow where the row has room
            if d + 3 <= m + 1:
                rows[f, d + 1:d + 3] = mid, half
        out = {"coef": rows, "status": None}
    else:
        out = {"coef": _to_powers(host, mid, half, m), "status": None}
    if case["kind"] == "qrb":
        out["sse"] = sse
    if gx is not None:
        out = {"coef": out["coef"], "grad_x": gx, "grad_y": gy}
    return out


def exact(case, seed):
    return _exact_single(case, seed) if "n" in case else _exact_batch(case, seed)
