"""Batches of short fits: a wave takes up to 8 neighbouring fits together, 8 lanes
each, when they are short enough for their number (at most 512 bytes of x per fit
taken together; float32: 128 points alone, 1,024 when 8 are).  The sizes below sit
at the edges of that rule, of the 16-byte vectors and of the rounds of 4 vectors per
lane, in batches whose last group of fits is full, one short of full and one over."""
import numpy as np
import pytest

from gpu_common import announce, normwise, to_dev, torch
from oracle import adjoint, cheb, fp64, qr
from paper_1512_08017_amd import workloads as W

pytestmark = pytest.mark.gpu

lf = pytest.importorskip("paper_1512_08017_amd")
EPS = np.finfo(np.float64).eps

EDGES = [3, 4, 5, 7, 8, 9, 15, 16, 17, 31, 33, 63, 64, 65, 127, 128, 129, 130, 131, 255, 256, 257, 383, 511, 512, 513,
         640, 1023, 1024, 1025, 1500, 2047, 2048, 2049, 5000]


def lengths(count, seed):
    """Runs of one size (whole groups of it) and sizes at random, empty fits among them."""
    rng = np.random.default_rng(seed)
    runs = np.concatenate([np.full(k, n) for n in (16, 128, 129, 256, 512, 513, 1024, 1025) for k in (1, 2, 9)])
    some = rng.choice(EDGES + [0, 1, 2], 120)
    return np.concatenate([runs, some, rng.choice([20, 100, 1000], count)])


def gate(x, m, c, s):
    """Both sides solve the same normal system, each with its own rounding of the sums."""
    V = np.vander((x.astype(np.float64) - c) / s, m + 1, increasing=True)
    return max(1e-12, 1e3 * EPS * np.linalg.cond(V.T @ V))


@pytest.mark.parametrize("dtype,maxdeg,count,shift", [(np.float32, 3, 8, 0), (np.float32, 5, 7, 1), (np.float64, 2, 1, 0),
                                                      (np.float64, 4, 9, 1), (np.float32, 1, 15, 2)])
def test_short_fits_against_oracle(dtype, maxdeg, count, shift):
    """shift 1: x starts one element in (every fit misaligned alike); 2: x and y differently."""
    announce(f"short fits {np.dtype(dtype).name} degree <= {maxdeg} count {count} shift {shift}")
    n = lengths(count, 40 + maxdeg)
    deg = np.random.default_rng(count).integers(1, maxdeg + 1, n.size).astype(np.int32)
    bf = W.random_batch(n, deg, seed=50 + maxdeg, dtype=dtype)
    pad = np.zeros(2, dtype)
    x = to_dev(np.concatenate([pad[:shift], bf.x]))[shift:]
    y = to_dev(np.concatenate([pad[:1 if shift else 0], bf.y]))[1 if shift else 0:]
    coef, status, _ = lf.fit_batched(x, y, to_dev(bf.offsets), to_dev(bf.degrees), maxdeg, center=0.0, scale=1.0)
    torch.cuda.synchronize()
    coef, status = coef.cpu().numpy(), status.cpu().numpy()
    for f in range(bf.batch):
        m, lo, hi = int(deg[f]), bf.offsets[f], bf.offsets[f + 1]
        if hi - lo < m + 1:
            assert status[f] == 2 and np.isnan(coef[f, : m + 1]).all(), (f, hi - lo, status[f])
            continue
        tol = gate(bf.x[lo:hi], m, 0.0, 1.0)
        if tol > 1e-3:        # a handful of points nearly on top of each other
            continue
        ref = fp64.fit(bf.x[lo:hi], bf.y[lo:hi], m)
        assert status[f] == 0, (f, hi - lo, m, status[f])
        e = normwise(coef[f, : m + 1], np.asarray(ref["a"], float))
        assert e <= tol, (f, hi - lo, m, e, tol)
        assert (coef[f, m + 1:] == 0).all()


def test_short_fits_compensated():
    """float32 sums of degree <= 2 with the refinement pass: an error of 2^-23 cond(A) before the
    refinement leaves about its square after it, below 1e-6 for cond(A) <= 1e3."""
    announce("short fits, compensated float32")
    n = lengths(9, 60)
    deg = np.random.default_rng(61).integers(1, 3, n.size).astype(np.int32)
    bf = W.random_batch(n, deg, seed=62)
    coef, status, _ = lf.fit_batched(to_dev(bf.x), to_dev(bf.y), to_dev(bf.offsets), to_dev(bf.degrees), 2,
                                     precision="f32c", center=0.0, scale=1.0)
    torch.cuda.synchronize()
    coef, status = coef.cpu().numpy(), status.cpu().numpy()
    done = 0
    for f in range(bf.batch):
        m, lo, hi = int(deg[f]), bf.offsets[f], bf.offsets[f + 1]
        if hi - lo < m + 1 or gate(bf.x[lo:hi], m, 0.0, 1.0) > 1e3 * EPS * 1e3:
            continue
        ref = fp64.fit(bf.x[lo:hi], bf.y[lo:hi], m)
        assert status[f] == 0
        e = normwise(coef[f, : m + 1], np.asarray(ref["a"], float))
        assert e <= 1e-6, (f, hi - lo, m, e)
        done += 1
    assert done > 100


@pytest.mark.parametrize("dtype,maxdeg,count,shift,solver", [(np.float32, 2, 8, 0, "gepp"), (np.float64, 3, 7, 1, "gepp"),
                                                             (np.float32, 3, 1, 2, "cholesky"),
                                                             (np.float64, 5, 9, 0, "gepp"), (np.float32, 1, 15, 1, "gepp")])
def test_short_fits_backward(dtype, maxdeg, count, shift, solver):
    """dL/dx and dL/dy of the same batches (solve in the walk up to degree 3, in its own
    launch above) against the closed form, each fit normwise.  Both sides solve with the
    same matrix; lambda and b carry cond(A) roundings, then the type's own."""
    announce(f"short fits backward {np.dtype(dtype).name} degree <= {maxdeg} count {count} shift {shift} {solver}")
    n = lengths(count, 70 + maxdeg)
    rng = np.random.default_rng(count + 100)
    deg = rng.integers(1, maxdeg + 1, n.size).astype(np.int32)
    bf = W.random_batch(n, deg, seed=71 + maxdeg, dtype=dtype)
    pad = np.zeros(2, dtype)
    x = to_dev(np.concatenate([pad[:shift], bf.x]))[shift:]
    y = to_dev(np.concatenate([pad[:1 if shift else 0], bf.y]))[1 if shift else 0:]
    off, dg = to_dev(bf.offsets), to_dev(bf.degrees)
    gbar = rng.standard_normal((n.size, maxdeg + 1))
    kw = dict(center=0.0, scale=1.0, solver=solver)
    _, status, ws = lf.fit_batched(x, y, off, dg, maxdeg, **kw)
    gx, gy = lf.fit_backward(x, y, off, dg, maxdeg, to_dev(gbar), ws=ws, **kw)
    torch.cuda.synchronize()
    gx, gy, status = gx.cpu().numpy(), gy.cpu().numpy(), status.cpu().numpy()
    assert gx.shape == bf.x.shape
    for f in range(bf.batch):
        m, lo, hi = int(deg[f]), bf.offsets[f], bf.offsets[f + 1]
        if hi - lo < m + 1:
            assert status[f] == 2 and np.isnan(gx[lo:hi]).all() and np.isnan(gy[lo:hi]).all()
            continue
        tol = gate(bf.x[lo:hi], m, 0.0, 1.0) + 2.0 * float(np.finfo(dtype).eps)
        if tol > 1e-3:
            continue
        ref = adjoint.gradients(bf.x[lo:hi], bf.y[lo:hi], m, gbar[f, : m + 1])
        # dL/dx = q' r - q f': gated against the size of its two terms
        t = bf.x[lo:hi].astype(np.float64)
        poly, r = np.polynomial.polynomial, bf.y[lo:hi] - np.polynomial.polynomial.polyval(t, ref["b"])
        size = np.max(np.abs(poly.polyval(t, poly.polyder(ref["lam"])) * r)) + np.max(
            np.abs(ref["dy"] * poly.polyval(t, poly.polyder(ref["b"]))))
        assert np.max(np.abs(gx[lo:hi] - ref["dx"])) <= tol * size, (f, hi - lo, m)
        assert np.max(np.abs(gy[lo:hi] - ref["dy"])) <= tol * np.max(np.abs(ref["dy"])), (f, hi - lo, m)


def cheb_check(bf, coef, status, maxdeg, fits):
    for f in fits:
        m, lo, hi = int(bf.degrees[f]), bf.offsets[f], bf.offsets[f + 1]
        if hi - lo < m + 1:
            assert status[f] == 2 and np.isnan(coef[f, : m + 1]).all()
            continue
        V = np.polynomial.chebyshev.chebvander(bf.x[lo:hi].astype(np.float64), m)
        tol = max(1e-12, 1e3 * EPS * np.linalg.cond(V.T @ V))
        if tol > 1e-3:
            continue
        ref = cheb.fit_cheb(bf.x[lo:hi], bf.y[lo:hi], m, 0.0, 1.0)
        assert status[f] == 0, (f, hi - lo, m, status[f])
        assert normwise(coef[f, : m + 1], np.asarray(ref["c"], float)) <= tol, (f, hi - lo, m)


@pytest.mark.parametrize("dtype,maxdeg,count,shift,given", [(np.float32, 3, 8, 0, True), (np.float64, 4, 7, 1, True),
                                                            (np.float32, 4, 1, 2, True), (np.float32, 6, 9, 0, True),
                                                            (np.float32, 3, 9, 1, False)])
def test_short_fits_chebyshev(dtype, maxdeg, count, shift, given):
    """The same batches in the Chebyshev basis (grouped up to degree 4, the range pass at
    every degree; mixed degrees in a group)."""
    announce(f"short fits Chebyshev {np.dtype(dtype).name} degree <= {maxdeg} count {count} shift {shift} given {given}")
    n = lengths(count, 80 + maxdeg)
    deg = np.random.default_rng(count + 5).integers(1, maxdeg + 1, n.size).astype(np.int32)
    bf = W.random_batch(n, deg, seed=81 + maxdeg, dtype=dtype)
    pad = np.zeros(2, dtype)
    x = to_dev(np.concatenate([pad[:shift], bf.x]))[shift:]
    y = to_dev(np.concatenate([pad[:1 if shift else 0], bf.y]))[1 if shift else 0:]
    kw = dict(center=0.0, scale=1.0) if given else {}
    coef, status, _ = lf.fit_batched(x, y, to_dev(bf.offsets), to_dev(bf.degrees), maxdeg, basis="chebyshev",
                                     coef_stride=maxdeg + 3, **kw)
    torch.cuda.synchronize()
    coef, status = coef.cpu().numpy(), status.cpu().numpy()
    if given:
        cheb_check(bf, coef, status, maxdeg, range(bf.batch))
        return
    for f in range(bf.batch):   # the exact extent of each fit
        m, lo, hi = int(deg[f]), bf.offsets[f], bf.offsets[f + 1]
        if hi - lo < m + 1 or status[f] != 0:
            continue
        a, b = float(bf.x[lo:hi].min()), float(bf.x[lo:hi].max())
        assert tuple(coef[f, m + 1: m + 3]) == (0.5 * b + 0.5 * a, 0.5 * b - 0.5 * a), f
    assert (status[n >= 64] == 0).all()


@pytest.mark.parametrize("batch,maxdeg", [(4095, 6), (4096, 5), (4097, 6), (8191, 8), (8192, 8), (8193, 7)])
def test_chebyshev_finish_forms(batch, maxdeg):
    """The batch sizes where the finish turns from a wave per fit to a thread per fit."""
    announce(f"Chebyshev finish of {batch} fits of degree <= {maxdeg}")
    rng = np.random.default_rng(batch)
    deg = rng.integers(1, maxdeg + 1, batch).astype(np.int32)
    bf = W.random_batch(rng.integers(40, 120, batch), deg, seed=batch)
    for solver in ("gepp", "cholesky"):
        coef, status, _ = lf.fit_batched(to_dev(bf.x), to_dev(bf.y), to_dev(bf.offsets), to_dev(bf.degrees), maxdeg,
                                         basis="chebyshev", center=0.0, scale=1.0, coef_stride=maxdeg + 1, solver=solver)
        torch.cuda.synchronize()
        coef, status = coef.cpu().numpy(), status.cpu().numpy()
        assert (status == 0).all()
        cheb_check(bf, coef, status, maxdeg, list(range(0, batch, 97)) + [batch - 2, batch - 1])


@pytest.mark.parametrize("dtype,maxdeg,count,shift", [(np.float32, 1, 8, 0), (np.float64, 3, 7, 1), (np.float32, 4, 1, 2),
                                                      (np.float64, 2, 9, 0), (np.float32, 6, 9, 1)])
def test_short_fits_qr(dtype, maxdeg, count, shift):
    """The same batches by rotations (grouped up to degree 4).  Both sides are QR factorisations of
    the same rows: their coefficients differ by roundings times cond(V), and by its square where the
    residual is of the size of the values."""
    announce(f"short fits QR {np.dtype(dtype).name} degree <= {maxdeg} count {count} shift {shift}")
    n = lengths(count, 90 + maxdeg)
    deg = np.random.default_rng(count + 9).integers(1, maxdeg + 1, n.size).astype(np.int32)
    bf = W.random_batch(n, deg, seed=91 + maxdeg, dtype=dtype)
    pad = np.zeros(2, dtype)
    x = to_dev(np.concatenate([pad[:shift], bf.x]))[shift:]
    y = to_dev(np.concatenate([pad[:1 if shift else 0], bf.y]))[1 if shift else 0:]
    coef, status, sse, _ = lf.fit_qr_batched(x, y, to_dev(bf.offsets), to_dev(bf.degrees), maxdeg, center=0.0, scale=1.0)
    torch.cuda.synchronize()
    coef, status, sse = coef.cpu().numpy(), status.cpu().numpy(), sse.cpu().numpy()
    for f in range(bf.batch):
        m, lo, hi = int(deg[f]), bf.offsets[f], bf.offsets[f + 1]
        if hi - lo < m + 1:
            assert status[f] == 2, (f, hi - lo, status[f])
            continue
        tol = gate(bf.x[lo:hi], m, 0.0, 1.0)     # holds cond(V)^2
        if tol > 1e-3:
            continue
        assert status[f] == 0, (f, hi - lo, m, status[f])
        b_ref = qr.lstsq_qr(bf.x[lo:hi], bf.y[lo:hi], m, 0.0, 1.0)
        assert normwise(coef[f, : m + 1], b_ref) <= tol, (f, hi - lo, m)
        r = bf.y[lo:hi].astype(np.float64) - np.polynomial.polynomial.polyval(bf.x[lo:hi].astype(np.float64), b_ref)
        yy = float(np.sum(bf.y[lo:hi].astype(np.float64) ** 2))
        assert abs(sse[f] - float(r @ r)) <= tol * yy, (f, hi - lo, m)
