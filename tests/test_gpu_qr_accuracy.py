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
