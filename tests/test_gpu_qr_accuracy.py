"""fit_qr's errors are roundings of the problem, whatever route the fit takes: the coefficients in
powers of t against the least-squares solution of the same t (QR in float64, refined in long
double).  The gate is the perturbation bound with a constant of 64
roundings, 16 times below that of the other QR tests."""
import numpy as np
import pytest

from gpu_common import announce, normwise, to_dev, torch
from oracle import qr

pytestmark = pytest.mark.gpu

lf = pytest.importorskip("paper_1512_08017_amd")
EPS = np.finfo(np.float64).eps


def reference(x, y, m, c, s):
    """(b, kappa, kappa eta): the solution for t = (x - c)/s, its powers, residual and steps of
    refinement in long double, each step solved through the float64 factorisation."""
    t = (x.astype(np.longdouble) - c) / s
    V = np.vander(t, m + 1, increasing=True)
    q, u = np.linalg.qr(V.astype(np.float64))
    b = np.zeros(m + 1, np.longdouble)
    for _ in range(4):
        r = y.astype(np.longdouble) - V @ b
        b = b + np.linalg.solve(u, q.T @ r.astype(np.float64))
    sv = np.linalg.svd(V.astype(np.float64), compute_uv=False)
    eta = float(np.linalg.norm(r.astype(np.float64))) / (sv[0] * float(np.linalg.norm(b.astype(np.float64))))
    return b.astype(np.float64), sv[0] / sv[-1], sv[0] / sv[-1] * eta


def check(x, y, m, r):
    c, s = r.center, r.scale
    b, kappa, ke = reference(x, y, m, c, s)
    tol = 64 * EPS * kappa * (1.0 + ke)
    e = normwise(r.coef_t.cpu().numpy(), b)
    announce(f"  error {e:.1e} (gate {tol:.1e}, cond(V) {kappa:.1e})")
    assert int(r.status.cpu()[0]) == 0
    assert e <= tol


@pytest.mark.parametrize("m,lo,width", [(3, 1.6e9, 3600.0), (5, 1.6e9, 3600.0), (4, -1e6, 1.0), (3, 1000.0, 1.0), (8, 3.0, 1e-3)])
def test_far_from_zero(m, lo, width):
    """Time stamps, frequencies: x in a window narrow against its distance from zero."""
    announce(f"qr, x in [{lo}, {lo} + {width}], m={m}")
    rng = np.random.default_rng(m)
    n = 60_001
    x = lo + width * rng.uniform(0.0, 1.0, n)
    y = np.cos(3.0 * (x - lo) / width) + 0.01 * rng.normal(size=n)
    r = lf.fit_qr(to_dev(x), to_dev(y), m)
    torch.cuda.synchronize()
    check(x, y, m, r)


def clustered(form, rng, n, gap):
    """x in [-1, 1] whose neighbours nearly repeat: the rows that one lane takes first are nearly equal."""
    u = rng.uniform(-1.0, 1.0, n)
    if form == "pairs":
        u[1::2] = u[0::2][: n // 2] + gap
    elif form == "grid":
        u = np.round(5 * u) / 5 + gap * rng.uniform(-1, 1, n)
    elif form == "sorted grid":
        u = np.sort(np.round(5 * u) / 5 + gap * rng.uniform(-1, 1, n))
    elif form == "half":
        u[: n // 2] = 0.3 + gap * u[: n // 2]
    return u


def values(x, m, rng):
    return np.polynomial.polynomial.polyval(x, rng.standard_normal(m + 1)) + 0.1 * rng.standard_normal(x.size)


FORMS = ["pairs", "grid", "sorted grid", "half"]
GAPS = [1e-4, 1e-6, 1e-8, 1e-10, 1e-11]


@pytest.mark.parametrize("m", [1, 2, 3, 4, 6])
@pytest.mark.parametrize("form", FORMS)
def test_nearly_equal_x_in_batches(form, m):
    """Rotations whose first rows hold next to nothing of the higher columns, then meet others."""
    announce(f"qr batch, nearly equal x: {form}, m={m}")
    rng = np.random.default_rng(m)
    xs = [clustered(form, rng, n, gap) for n in (60, 100, 384, 2000, 20_000) for gap in GAPS]
    ys = [values(x, m, rng) for x in xs]
    off = np.concatenate([[0], np.cumsum([x.size for x in xs])]).astype(np.int64)
    deg = np.full(len(xs), m, np.int32)
    coef, status, _, _ = lf.fit_qr_batched(to_dev(np.concatenate(xs)), to_dev(np.concatenate(ys)), to_dev(off),
                                           to_dev(deg), m, center=0.0, scale=1.0)
    torch.cuda.synchronize()
    assert (status.cpu().numpy() == 0).all()
    coef, worst = coef.cpu().numpy(), 0.0
    for f, (x, y) in enumerate(zip(xs, ys)):
        b, kappa, ke = reference(x, y, m, 0.0, 1.0)
        tol = 64 * EPS * kappa * (1.0 + ke)
        e = normwise(coef[f, : m + 1], b)
        worst = max(worst, e)
        assert e <= tol, (x.size, GAPS[f % len(GAPS)], e, tol)
    announce(f"  largest error {worst:.1e}")


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("m", [1, 2, 3, 4, 6])
def test_equal_x_in_batches(m, dtype):
    """x that repeat exactly, with the same gate: roundings times cond(V)."""
    announce(f"qr batch, equal x, m={m} {np.dtype(dtype).name}")
    rng = np.random.default_rng(m)
    xs = [clustered(form, rng, n, 0.0).astype(dtype) for n in (60, 100, 129, 384, 2000, 20_000) for form in FORMS]
    ys = [values(x.astype(np.float64), m, rng).astype(dtype) for x in xs]
    off = np.concatenate([[0], np.cumsum([x.size for x in xs])]).astype(np.int64)
    deg = np.full(len(xs), m, np.int32)
    coef, status, _, _ = lf.fit_qr_batched(to_dev(np.concatenate(xs)), to_dev(np.concatenate(ys)), to_dev(off),
                                           to_dev(deg), m, center=0.0, scale=1.0)
    torch.cuda.synchronize()
    assert (status.cpu().numpy() == 0).all()
    coef, worst = coef.cpu().numpy(), 0.0
    for f, (x, y) in enumerate(zip(xs, ys)):
        b, kappa, ke = reference(x, y, m, 0.0, 1.0)
        e = normwise(coef[f, : m + 1], b)
        worst = max(worst, e / (EPS * kappa * (1.0 + ke)))
        assert e <= 64 * EPS * kappa * (1.0 + ke), (x.size, FORMS[f % len(FORMS)], e)
    announce(f"  largest error {worst:.2g} roundings")


@pytest.mark.parametrize("m,n", [(1, 5001), (2, 70_001), (3, 999), (6, 1001)])
def test_nearly_equal_x_in_one_fit(m, n):
    announce(f"qr, nearly equal x, {n} points, m={m}")
    rng = np.random.default_rng(m)
    for form in FORMS:
        for gap in GAPS:
            x = clustered(form, rng, n, gap)
            y = values(x, m, rng)
            r = lf.fit_qr(to_dev(x), to_dev(y), m, center=0.0, scale=1.0)
            torch.cuda.synchronize()
            check(x, y, m, r)


def left(r):
    """What the sampled polynomials left of the fit (first word of its workspace): 0 nothing, 1 the
    rotations, 2 a second pass in the polynomials of all the points."""
    return int(r.ws[:8].view(torch.int64).item())


SPREADS = {
    "uniform": lambda rng, n: rng.uniform(-1, 1, n),
    "normal": lambda rng, n: rng.normal(size=n),
    "sorted normal": lambda rng, n: np.sort(rng.normal(size=n)),
    "Laplace": lambda rng, n: rng.laplace(size=n),
    "logistic": lambda rng, n: rng.logistic(size=n),
    "exponential": lambda rng, n: rng.exponential(size=n),
    "lognormal": lambda rng, n: rng.lognormal(sigma=0.5, size=n),
    "wide lognormal": lambda rng, n: rng.lognormal(sigma=2.0, size=n),
    "Student 3": lambda rng, n: rng.standard_t(3, size=n),
    "sweeps": lambda rng, n: (np.arange(n) % (n // 255)) / (n // 255),
}


@pytest.mark.parametrize("m", [3, 4, 5, 6, 7, 8])
@pytest.mark.parametrize("kind", list(SPREADS))
def test_spreads_of_x(kind, m):
    """Ten draws each: whatever route a fit takes, the largest error is that of the rotations (a
    batch of one fit in the same range), within a factor of 4 between two largest of ten and
    16 roundings of the reference, and the fit's term by term that of a backward stable solver."""
    announce(f"qr, x {kind}, m={m}")
    routes, qr_err, rot_err, worst = [], 0.0, 0.0, 0.0
    for seed in range(10):
        rng = np.random.default_rng([seed, m])
        n = 20_001 + 17 * seed
        x = SPREADS[kind](rng, n)
        lo, hi = x.min(), x.max()
        y = np.cos(2.0 * (2 * x - lo - hi) / (hi - lo) + rng.normal()) + rng.choice([0.05, 0.5, 3.0]) * rng.normal(size=n)
        X, Y = to_dev(x), to_dev(y)
        r = lf.fit_qr(X, Y, m)
        c, s = r.center, r.scale
        sse, _ = lf.residuals(X, Y, r)
        # t itself as x: the batch's a_0..a_m are then powers of t
        t = (x - c) / s
        rot = lf.fit_qr_batched(to_dev(t), Y, to_dev(np.array([0, n])), to_dev(np.array([m], np.int32)), m, center=0.0,
                                scale=1.0)
        torch.cuda.synchronize()
        b, _, _ = reference(x, y, m, c, s)
        got = r.coef_t.cpu().numpy()
        qr_err = max(qr_err, normwise(got, b))
        rot_err = max(rot_err, normwise(rot[0][0].cpu().numpy(), b))
        V = qr.vandermonde(x, m, c, s)
        norms = np.linalg.norm(V, axis=0)
        kappa = np.linalg.cond(V / norms)
        size = np.linalg.norm(y) + kappa * np.linalg.norm(y - V @ b)
        e = np.max(np.abs(got - b) * norms) / (EPS * kappa * size)
        worst = max(worst, e)
        assert int(r.status.cpu()[0]) == 0 and int(rot[1].cpu()[0]) == 0
        assert e <= 8, (seed, left(r), e)
        assert abs(r.sse - float(sse.cpu()[0])) <= 1e-9 * r.sse
        routes.append(left(r))
    announce(f"  left: {routes}, largest error {qr_err:.1e} (rotations {rot_err:.1e}); by terms {worst:.2g} roundings")
    assert qr_err <= 4 * rot_err + 16 * EPS
    if kind == "uniform":
        assert set(routes) == {0}
    elif kind in ("exponential", "Laplace", "lognormal") and m in (5, 6):
        assert set(routes) == {2}
    elif kind == "wide lognormal" and m == 8:
        assert set(routes) == {1}


@pytest.mark.parametrize("m,n", [(1, (1 << 23) + 5), (2, (1 << 21) + 5)])
def test_low_degrees_with_tails(m, n):
    """The sizes from which degrees 1 and 2 take the sampled polynomials."""
    announce(f"qr, tails, m={m}, n={n}")
    for seed, kind in enumerate(("normal", "exponential", "lognormal", "Student 3", "wide lognormal")):
        rng = np.random.default_rng(seed)
        x = SPREADS[kind](rng, n)
        y = np.cos(x / x.std()) + 0.1 * rng.normal(size=n)
        r = lf.fit_qr(to_dev(x), to_dev(y), m)
        torch.cuda.synchronize()
        t = ((x.astype(np.longdouble) - r.center) / r.scale)
        V = np.vander(t, m + 1, increasing=True)
        b = np.linalg.solve((V.T @ V).astype(np.float64), (V.T @ y.astype(np.longdouble)).astype(np.float64))
        for _ in range(3):
            g = (V.T @ (y.astype(np.longdouble) - V @ b)).astype(np.float64)
            b = b + np.linalg.solve((V.T @ V).astype(np.float64), g)
        norms = np.sqrt(np.sum(V.astype(np.float64) ** 2, axis=0))
        e = np.max(np.abs(r.coef_t.cpu().numpy() - b) * norms) / np.linalg.norm(y)
        announce(f"  {kind}: left {left(r)}, {e / EPS:.2g} roundings")
        assert int(r.status.cpu()[0]) == 0 and e <= 8 * EPS


@pytest.mark.parametrize("dtype,shift", [(np.float64, 0), (np.float64, 1), (np.float32, 1), (np.float32, 2)])
@pytest.mark.parametrize("waves,wpb", [(2048, 4), (512, 1), (6, 2), (1, 1)])
def test_second_pass_on_other_grids(waves, wpb, dtype, shift):
    """The second pass and the rotations are finished by their launch's last block: blocks of
    one, two and four waves, many blocks and one, x and y misaligned alike and differently."""
    announce(f"qr, second pass and rotations, {waves} waves, {wpb} per block, {np.dtype(dtype).name} shift {shift}")
    rng = np.random.default_rng(waves + shift)
    m, n = 5, 30_011
    pad = np.zeros(2, dtype)
    try:
        lf.set_default_schedule({"waves": waves, "waves_per_block": wpb, "tile": 2048, "unroll": 2})
        for x, want in ((rng.exponential(size=n), 2), (rng.lognormal(sigma=3.0, size=n), 1)):
            x = x.astype(dtype)
            y = (np.sin(x) + 0.1 * rng.normal(size=n)).astype(dtype)
            X = to_dev(np.concatenate([pad[:shift], x]))[shift:]
            Y = to_dev(np.concatenate([pad[:1 if shift else 0], y]))[1 if shift else 0:]
            r, again = lf.fit_qr(X, Y, m), lf.fit_qr(X, Y, m)
            torch.cuda.synchronize()
            assert left(r) == want
            assert torch.equal(r.coef, again.coef) and torch.equal(r.info, again.info)
            b, _, _ = reference(x, y, m, r.center, r.scale)
            norms = np.linalg.norm(qr.vandermonde(x, m, r.center, r.scale), axis=0)
            kappa = np.linalg.cond(qr.vandermonde(x, m, r.center, r.scale) / norms)
            e = np.max(np.abs(r.coef_t.cpu().numpy() - b) * norms)
            assert e <= 8 * EPS * kappa * kappa * np.linalg.norm(y)
    finally:
        lf.set_default_schedule(None)


@pytest.mark.parametrize("kind", ["exponential", "rotations"])
def test_replayed_with_other_data(kind):
    """One captured call, its inputs replaced between replays by data of another route."""
    draw = dict(SPREADS, rotations=lambda rng, n: rng.lognormal(sigma=3.0, size=n))
    rng = np.random.default_rng(3)
    n, m = 20_000, 5
    X, Y = torch.empty(n, dtype=torch.float64, device="cuda"), torch.empty(n, dtype=torch.float64, device="cuda")
    ws = torch.empty(lf.workspace_bytes(1, m), dtype=torch.uint8, device="cuda")

    def fill(k):
        x = draw[k](rng, n)
        X.copy_(to_dev(x))
        Y.copy_(to_dev(np.sin(x) + 0.1 * rng.normal(size=n)))

    fill("uniform")
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        lf.fit_qr(X, Y, m, ws=ws)
    torch.cuda.current_stream().wait_stream(side)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        r = lf.fit_qr(X, Y, m, ws=ws)
    seen = []
    for k in ("uniform", kind, "uniform", kind, kind):
        fill(k)
        r.coef.zero_()
        g.replay()
        torch.cuda.synchronize()
        seen.append(left(r))
        assert torch.equal(r.coef, lf.fit_qr(X, Y, m).coef) and int(r.status.cpu()[0]) == 0
    assert seen == [0, 2, 0, 2, 2] if kind == "exponential" else seen == [0, 1, 0, 1, 1]
