"""Single fits of up to 16,384 points, which one launch of one block takes: sizes around
the range sample (256), the waves, the rounds of a lane and the last size, against the
float64 oracle and against the two-launch form of the same call (a schedule set by the
caller keeps that form)."""
import numpy as np
import pytest

from gpu_common import announce, normwise, to_dev, torch
from oracle import fp64
from paper_1512_08017_amd import workloads as W

pytestmark = pytest.mark.gpu

lf = pytest.importorskip("paper_1512_08017_amd")
EPS = np.finfo(np.float64).eps


def two_launches(call):
    old = lf.default_schedule().as_dict()
    try:
        lf.set_default_schedule(old)
        return call()
    finally:
        lf.set_default_schedule(None)


@pytest.mark.parametrize("dtype,precision", [(np.float32, "f64"), (np.float64, "f64"), (np.float32, "f32c")])
@pytest.mark.parametrize("n,m,shift", [(2, 1, 0), (9, 8, 0), (63, 4, 1), (64, 5, 0), (255, 3, 0), (256, 3, 1), (257, 3, 2),
                                       (511, 2, 0), (2049, 6, 1), (4097, 3, 0), (8191, 8, 0), (16_383, 5, 2), (16_384, 4, 1),
                                       (16_385, 4, 0)])
def test_sizes(n, m, shift, dtype, precision):
    """shift 1: x and y start one element in; 2: they are misaligned differently."""
    if precision == "f32c":
        m = min(m, 3)
    announce(f"small fit n={n} m={m} {np.dtype(dtype).name} {precision} shift {shift}")
    wl = W.random_small(n, m, seed=n + m, dtype=dtype, lo=-0.7, hi=1.3)
    pad = np.zeros(2, dtype)
    x = to_dev(np.concatenate([pad[:shift], wl.x]))[shift:]
    y = to_dev(np.concatenate([pad[:1 if shift else 0], wl.y]))[1 if shift else 0:]
    one = lf.fit(x, y, m, precision=precision)
    two = two_launches(lambda: lf.fit(x, y, m, precision=precision))
    split = lf.fit_split(x, y, m, precision=precision)
    sse, _ = lf.residuals(x, y, one)
    torch.cuda.synchronize()
    c, s = one.center, one.scale
    assert (c, s) == (two.center, two.scale)
    t = (wl.x.astype(np.float64) - c) / s
    V = np.vander(t, m + 1, increasing=True)
    cond = np.linalg.cond(V.T @ V)
    ref = fp64.fit(wl.x, wl.y, m, c, s)
    assert int(one.status.cpu()[0]) == 0
    # sums in float64: cond(A) roundings; compensated float32 sums: 2^-23 cond(A), squared by the refinement
    tol = max(1e-12, 1e3 * EPS * cond) if precision == "f64" else max(1e-6, (2.0 ** -20 * cond) ** 2)
    if tol < 1e-3:
        e = normwise(one.coef_t.cpu().numpy(), np.asarray(ref["b"], float))
        announce(f"  t-basis error {e:.1e} (gate {tol:.1e})")
        assert e <= tol
        want = fp64.sse(wl.x, wl.y, one.coef.cpu().numpy())
        size = float(np.square(wl.y, dtype=np.float64).sum())
        assert abs(float(sse.cpu()[0]) - want) <= 1e-9 * want + 1e3 * EPS * size
    assert torch.equal(one.coef, split.coef) and torch.equal(one.moments, split.moments)
    if precision == "f64":   # the two forms add the same terms in another order
        a, b = one.moments.cpu().numpy(), two.moments.cpu().numpy()
        assert np.all(np.abs(a - b) <= 64 * EPS * np.abs(V).sum() * max(1.0, np.abs(wl.y).max()))


@pytest.mark.parametrize("m", [2, 6])
def test_degenerate(m):
    n = 1000
    wl = W.random_small(n, m, seed=4, dtype=np.float64)
    flat, bad = np.full(n, 0.25), wl.y.copy()
    bad[777] = np.inf
    for X, Y, want in ((flat, wl.y, 2), (wl.x, bad, 3)):
        r = lf.fit(to_dev(X), to_dev(Y), m)
        sse, e = lf.residuals(to_dev(X), to_dev(Y), r, store=True)
        torch.cuda.synchronize()
        assert int(r.status.cpu()[0]) == want and np.isnan(r.coef.cpu().numpy()).all()
        assert np.isnan(sse.cpu().numpy()).all() and np.isnan(e.cpu().numpy()).all()
    nan_x = wl.x.copy()
    nan_x[:] = np.nan
    r = lf.fit(to_dev(nan_x), to_dev(wl.y), m)
    torch.cuda.synchronize()
    assert int(r.status.cpu()[0]) == 3 and (r.center, r.scale) == (0.0, 1.0)
