"""fit_qr's route through the sample's orthogonal polynomials, and what it leaves to the
rotations, against the oracle's Householder QR.  The gate is the perturbation bound of
the problem (as in test_gpu_qr.py), with cond(V) and the residual from the data."""
import numpy as np
import pytest

from gpu_common import announce, normwise, to_dev, torch
from oracle import qr
from paper_1512_08017_amd import workloads as W

pytestmark = pytest.mark.gpu

lf = pytest.importorskip("paper_1512_08017_amd")
EPS = np.finfo(np.float64).eps


def check(x, y, m, X=None, Y=None, **kw):
    r = lf.fit_qr(to_dev(x) if X is None else X, to_dev(y) if Y is None else Y, m, **kw)
    torch.cuda.synchronize()
    c, s = r.center, r.scale
    V = qr.vandermonde(x, m, c, s)
    b_ref = qr.lstsq_qr(x, y, m, c, s)
    sv = np.linalg.svd(V, compute_uv=False)
    kappa = sv[0] / sv[-1]
    res = np.asarray(y, np.float64) - V @ b_ref
    eta = np.linalg.norm(res) / (sv[0] * np.linalg.norm(b_ref))
    tol = 1e3 * EPS * (kappa + kappa * kappa * eta)
    e = normwise(r.coef_t.cpu().numpy(), b_ref)
    sse = float(res @ res)
    announce(f"  error {e:.1e} (gate {tol:.1e}), sse {r.sse:.6e}")
    assert int(r.status.cpu()[0]) == 0
    assert e <= tol
    # sum of squares: its own rounding, and that of values of y's size evaluated twice
    assert abs(r.sse - sse) <= 1e-9 * sse + 1e3 * EPS * EPS * kappa * kappa * float(np.square(y, dtype=np.float64).sum())
    return r


# the first size of the route (and one less: the rotations), around a multiple of the
# sample's spacing, and several rounds per lane; x and y misaligned alike and differently
@pytest.mark.parametrize("n,m,dtype,shift", [(1023, 3, np.float64, 0), (1024, 3, np.float64, 0), (1024, 8, np.float64, 0),
                                             (1025, 4, np.float32, 1), (1276, 5, np.float32, 0), (4097, 6, np.float64, 1),
                                             (70_001, 7, np.float32, 2), (300_007, 8, np.float32, 1),
                                             (2_100_003, 5, np.float32, 0), ((1 << 21) + 1, 2, np.float32, 0),
                                             ((1 << 21) - 1, 2, np.float64, 0)])
def test_sizes(n, m, dtype, shift):
    announce(f"qr n={n} m={m} {np.dtype(dtype).name} shift {shift}")
    wl = W.random_small(n, m, seed=n + m, dtype=dtype)
    pad = np.zeros(2, dtype)
    X = to_dev(np.concatenate([pad[:shift], wl.x]))[shift:]
    Y = to_dev(np.concatenate([pad[:1 if shift else 0], wl.y]))[1 if shift else 0:]
    check(wl.x, wl.y, m, X, Y)


def test_degree_one_at_its_first_size():
    n = (1 << 23) + 1
    wl = W.random_small(n, 1, seed=5, dtype=np.float32)
    announce(f"qr n={n} m=1")
    r = lf.fit_qr(to_dev(wl.x), to_dev(wl.y), 1)
    torch.cuda.synchronize()
    x, y = wl.x.astype(np.float64), wl.y.astype(np.float64)
    d = x - x.mean()
    a1 = (d @ y) / (d @ d)
    assert int(r.status.cpu()[0]) == 0
    assert normwise(r.coef.cpu().numpy(), [y.mean() - a1 * x.mean(), a1]) <= 1e3 * EPS * 4


def spread(kind, n, rng):
    u = rng.uniform(-1.0, 1.0, n)
    return {
        "sorted": np.sort(u),
        "given far off": u,
        "eleven values": rng.integers(0, 11, n) * 0.1,
        "normal": rng.normal(size=n),
        "heavy tail": rng.lognormal(sigma=2.0, size=n),             # left to the rotations
        "rare outliers": np.where(rng.random(n) < 1e-4, u, 1e-3 * u),  # left to the rotations
        "two clusters": np.where(u < 0, -1.0, 1.0) + 1e-3 * rng.normal(size=n),
    }[kind]


@pytest.mark.parametrize("kind,m", [("sorted", 5), ("given far off", 4), ("eleven values", 5), ("normal", 4), ("normal", 8),
                                    ("heavy tail", 3), ("heavy tail", 5), ("rare outliers", 3), ("two clusters", 3)])
def test_spread_of_x(kind, m):
    announce(f"qr, x {kind}, m={m}")
    rng = np.random.default_rng(77)
    n = 60_001
    x = spread(kind, n, rng)
    y = np.cos(2.0 * x / np.abs(x).max()) + 0.1 * rng.normal(size=n)
    kw = {"center": 3.0, "scale": 4.0} if kind == "given far off" else {}
    r = check(x, y, m, **kw)
    again = lf.fit_qr(to_dev(x), to_dev(y), m, **kw)
    sse, _ = lf.residuals(to_dev(x), to_dev(y), r)
    torch.cuda.synchronize()
    assert np.array_equal(r.coef.cpu().numpy(), again.coef.cpu().numpy()) and r.sse == again.sse
    assert abs(float(sse.cpu()[0]) - r.sse) <= 1e-9 * r.sse


@pytest.mark.parametrize("n", [5_000, 300_001])
def test_degenerate(n):
    rng = np.random.default_rng(n)
    x, y = rng.uniform(-1, 1, n), rng.normal(size=n)
    flat = np.full(n, 0.25)
    bad = y.copy()
    bad[n // 3 + 1] = np.nan
    inf = x.copy()
    inf[n // 7] = np.inf
    for X, Y, want in ((flat, y, 2), (x, bad, 3), (inf, y, 3)):
        r = lf.fit_qr(to_dev(X), to_dev(Y), 3)
        torch.cuda.synchronize()
        assert int(r.status.cpu()[0]) == want and np.isnan(r.coef.cpu().numpy()).all() and np.isnan(r.sse)
    zero = lf.fit_qr(to_dev(x), to_dev(np.zeros(n)), 4)
    torch.cuda.synchronize()
    assert int(zero.status.cpu()[0]) == 0 and (zero.coef.cpu().numpy() == 0).all() and zero.sse == 0


def test_replayed_graph_alternates_with_eager_calls():
    """Both routes captured (the second one left to the rotations, whose last block counts
    in the workspace): every replay equals the eager result."""
    rng = np.random.default_rng(9)
    n, m = 50_001, 3
    for x in (rng.uniform(-1, 1, n), rng.lognormal(sigma=2.0, size=n)):
        X, Y = to_dev(x), to_dev(np.sin(x) + 0.1 * rng.normal(size=n))
        want = lf.fit_qr(X, Y, m).coef.clone()
        ws = torch.empty(lf.workspace_bytes(1, m), dtype=torch.uint8, device=X.device)
        side = torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(side):
            lf.fit_qr(X, Y, m, ws=ws)
        torch.cuda.current_stream().wait_stream(side)
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            r = lf.fit_qr(X, Y, m, ws=ws)
        for _ in range(4):
            r.coef.zero_()
            g.replay()
            torch.cuda.synchronize()
            assert torch.equal(r.coef, want)
            assert torch.equal(lf.fit_qr(X, Y, m).coef, want)
