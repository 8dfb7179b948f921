"""Rotations on data whose x repeat: a lane may hold equal t only, and then columns 1.. of
its factor are the rounding of zero until a row with another t arrives."""
import numpy as np
import pytest

from gpu_common import announce, normwise, to_dev, torch
from oracle import qr

pytestmark = pytest.mark.gpu

lf = pytest.importorskip("paper_1512_08017_amd")
EPS = np.finfo(np.float64).eps

FORMS = {
    "values": lambda rng, n: rng.integers(-5, 6, n) / 5.0,
    "sorted": lambda rng, n: np.sort(rng.integers(-5, 6, n) / 5.0),
    "twice": lambda rng, n: np.repeat(rng.uniform(-1, 1, n // 2 + 1), 2)[:n],
    "period 8": lambda rng, n: (np.arange(n) % 8) / 4.0 - 1.0,
    "period 64": lambda rng, n: (np.arange(n) % 64) / 32.0 - 1.0,
    "offset": lambda rng, n: 3.0 + rng.integers(-12, 13, n) / 25.0,
}


def check(x, y, m, b, what):
    """Both sides factor the same rows: roundings times cond(V), and its square with the residual."""
    V = qr.vandermonde(x.astype(np.float64), m)
    tol = 1e3 * EPS * np.linalg.cond(V) ** 2
    ref = qr.lstsq_qr(x, y, m, 0.0, 1.0)
    assert normwise(b, ref) <= tol, (what, normwise(b, ref), tol)


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("m", [1, 2, 3, 4, 6])
@pytest.mark.parametrize("form", list(FORMS))
def test_repeated_x(form, m, dtype):
    announce(f"repeated x {form} degree {m} {np.dtype(dtype).name}")
    rng = np.random.default_rng(m)
    lens = [15, 40, 64, 100, 128, 129, 500, 2000, 20_000] * 3
    xs = [FORMS[form](rng, n).astype(dtype) for n in lens]
    ys = [(np.polynomial.polynomial.polyval(x.astype(np.float64), rng.standard_normal(m + 1))
           + 0.1 * rng.standard_normal(x.size)).astype(dtype) for x in xs]
    off = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    deg = np.full(len(lens), m, np.int32)
    coef, status, _, _ = lf.fit_qr_batched(to_dev(np.concatenate(xs)), to_dev(np.concatenate(ys)), to_dev(off),
                                           to_dev(deg), m, center=0.0, scale=1.0)
    torch.cuda.synchronize()
    assert (status.cpu().numpy() == 0).all()
    coef = coef.cpu().numpy()
    for f, (x, y) in enumerate(zip(xs, ys)):
        check(x, y, m, coef[f, : m + 1], (form, m, lens[f]))


@pytest.mark.parametrize("m,n", [(1, 999), (2, 5000), (3, 999), (5, 700)])
def test_repeated_x_single(m, n):
    """One fit below the sizes of the sampled polynomials: rotations."""
    announce(f"repeated x, one fit of {n} points, degree {m}")
    rng = np.random.default_rng(n)
    for form, gen in FORMS.items():
        x = gen(rng, n)
        y = np.polynomial.polynomial.polyval(x, rng.standard_normal(m + 1)) + 0.1 * rng.standard_normal(n)
        r = lf.fit_qr(to_dev(x), to_dev(y), m, center=0.0, scale=1.0)
        torch.cuda.synchronize()
        check(x, y, m, r.coef.cpu().numpy(), (form, m, n))
