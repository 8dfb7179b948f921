"""fit_qr's errors are roundings of the problem, whatever route the fit takes: the coefficients in
powers of t against the least-squares solution of the same t (Householder QR in float64, with one
step of refinement in long double).  The gate is the perturbation bound with a constant of 64
roundings, 16 times below that of the other QR tests."""
import numpy as np
import pytest

from gpu_common import announce, normwise, to_dev, torch
from oracle import qr

pytestmark = pytest.mark.gpu

lf = pytest.importorskip("paper_1512_08017_amd")
EPS = np.finfo(np.float64).eps


def reference(x, y, m, c, s):
    """(b, kappa, kappa eta): the solution with one step of refinement, residual and step in long double."""
    V = qr.vandermonde(x, m, c, s)
    b = qr.lstsq_qr(x, y, m, c, s)
    r = y.astype(np.longdouble) - V.astype(np.longdouble) @ b.astype(np.longdouble)
    db = qr.lstsq_qr(x, r.astype(np.float64), m, c, s)
    sv = np.linalg.svd(V, compute_uv=False)
    eta = float(np.linalg.norm(r.astype(np.float64))) / (sv[0] * np.linalg.norm(b))
    return b + db, sv[0] / sv[-1], sv[0] / sv[-1] * eta


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
