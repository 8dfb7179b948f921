"""The native marshalling of the Python surface against the Python form of the same calls
(the path it leaves everything unusual to): same results bit for bit, same errors."""
import numpy as np
import pytest

from gpu_common import to_dev, torch
from paper_1512_08017_amd import workloads as W

pytestmark = pytest.mark.gpu

lf = pytest.importorskip("paper_1512_08017_amd")
from paper_1512_08017_amd import _lib, api  # noqa: E402


class Declines:
    """A stand-in for the native module that takes no call."""
    def __getattr__(self, name):
        return lambda *a: None


def both(monkeypatch, call):
    native = call()
    with monkeypatch.context() as m:
        m.setattr(api, "_bind", Declines())
        plain = call()
    torch.cuda.synchronize()
    return native, plain


def same(a, b):
    if a is None or b is None:
        return a is b
    return a.dtype == b.dtype and a.shape == b.shape and a.stride() == b.stride() and torch.equal(
        a.nan_to_num(1e300), b.nan_to_num(1e300))


@pytest.mark.parametrize("kw", [{}, {"precision": "f32c"}, {"center": 0.25, "scale": 2}, {"solver": "cholesky", "center": 1},
                                {"basis": "chebyshev"}, {"precision": "f32c", "refine": 0}])
@pytest.mark.parametrize("n,m,dtype", [(1001, 3, np.float32), (5, 4, np.float64), (70_000, 8, np.float32)])
def test_single(monkeypatch, kw, n, m, dtype):
    if kw.get("precision") == "f32c" and dtype == np.float64:
        kw = {}
    wl = W.random_small(n, m, seed=n, dtype=dtype)
    x, y = to_dev(wl.x), to_dev(wl.y)
    a, b = both(monkeypatch, lambda: lf.fit(x, y, m, **kw))
    for f in ("coef", "coef_t", "coef_cheb", "status", "moments"):
        assert same(getattr(a, f), getattr(b, f)), f
    assert bytes(a.options) == bytes(b.options) and a.ws.numel() == b.ws.numel()
    for store in (False, True):
        ra, rb = both(monkeypatch, lambda: lf.residuals(x, y, a, store=store))
        assert same(ra[0], rb[0]) and same(ra[1], rb[1])
    ws = torch.empty(a.ws.numel() + 100, dtype=torch.uint8, device=x.device)
    assert lf.fit(x, y, m, ws=ws, **kw).ws.data_ptr() == ws.data_ptr()
    if not kw or "scale" in kw:
        qa, qb = both(monkeypatch, lambda: lf.fit_qr(x, y, m, **kw))
        for f in ("coef", "coef_t", "status", "info"):
            assert same(getattr(qa, f), getattr(qb, f)), f


@pytest.mark.parametrize("kw", [{}, {"output_basis": "x_and_t"}, {"coef_stride": 7}, {"basis": "chebyshev", "center": 0.0,
                                                                                   "scale": 1.0}])
def test_batched(monkeypatch, kw):
    bf = W.random_batch([50, 0, 2, 700, 3000, 90], [1, 2, 3, 2, 3, 1], seed=3)
    x, y, off, dg = (to_dev(v) for v in (bf.x, bf.y, bf.offsets, bf.degrees))
    a, b = both(monkeypatch, lambda: lf.fit_batched(x, y, off, dg, 3, **kw))
    assert same(a[0], b[0]) and same(a[1], b[1]) and a[2].numel() == b[2].numel()
    g = torch.randn_like(a[0])
    bk = {k: v for k, v in kw.items() if k in ("basis", "center", "scale")}
    for grad in (g, g.float(), g.t().contiguous().t()):
        ga, gb = both(monkeypatch, lambda: lf.fit_backward(x, y, off, dg, 3, grad, ws=a[2], **bk))
        assert same(ga[0], gb[0]) and same(ga[1], gb[1])
    plan = lf.Plan(6, 3)
    pa, pb = both(monkeypatch, lambda: lf.fit_batched(x, y, off, dg, 3, plan=plan, **kw))
    assert same(pa[0], a[0]) and same(pb[0], a[0]) and pa[2] is None and pb[2] is None


def test_what_is_refused_stays_refused(monkeypatch):
    wl = W.random_small(100, 2, seed=1, dtype=np.float64)
    x, y = to_dev(wl.x), to_dev(wl.y)
    off, dg = to_dev(np.array([0, 100])), to_dev(np.array([2], np.int32))
    calls = [lambda: lf.fit(x, y[:50], 2), lambda: lf.fit(x.float(), y, 2), lambda: lf.fit(x.cpu(), y.cpu(), 2),
             lambda: lf.fit(x[::2], y[::2], 2), lambda: lf.fit(x, y, 0), lambda: lf.fit(x, y, 17), lambda: lf.fit(x, y, 9),
             lambda: lf.fit(x, y, 2, precision="f16"), lambda: lf.fit(x, y, 2, solver="lu"), lambda: lf.fit(x[:2], y[:2], 2),
             lambda: lf.fit(x, y, 2, precision="f32c"), lambda: lf.fit(x, y, 2, center=0.0, scale=0.0),
             lambda: lf.fit(x.long(), y.long(), 2), lambda: lf.fit([1.0], [2.0], 1), lambda: lf.fit_qr(x, y, 9),
             lambda: lf.fit_batched(x, y, off.int(), dg, 2), lambda: lf.fit_batched(x, y, off, dg.long(), 2),
             lambda: lf.fit_batched(x, y, off, dg, 2, coef_stride=2), lambda: lf.fit_batched(x, y, off[:1], dg, 2),
             lambda: lf.fit_batched(x, y, off, dg, 2, output_basis="t"),
             lambda: lf.fit_backward(x, y, off, dg, 2, torch.zeros(1, 3, dtype=torch.float64, device=x.device),
                                     ws=torch.empty(8, dtype=torch.uint8, device=x.device))]
    for k, call in enumerate(calls):
        seen = []
        for native in (True, False):
            with monkeypatch.context() as m:
                if not native:
                    m.setattr(api, "_bind", Declines())
                with pytest.raises((TypeError, ValueError, RuntimeError, _lib.LsefitError)) as e:
                    call()
                seen.append((type(e.value), str(e.value)))
        assert seen[0] == seen[1], (k, seen)
    # a subclass of Tensor and a NumPy integer degree are taken by the Python form
    want = lf.fit(x, y, 2).coef
    assert torch.equal(lf.fit(torch.nn.Parameter(x, requires_grad=False), y, 2).coef, want)
    assert torch.equal(lf.fit(x, y, np.int32(2)).coef, want)
    assert lf.fit_batched(x[:0], y[:0], off[:1] * 0, dg[:0], 2)[0].shape == (0, 3)


@pytest.mark.parametrize("kw", [{}, {"coef_stride": 7}, {"center": 0.25, "scale": 2}])
def test_qr_batched(monkeypatch, kw):
    bf = W.random_batch([50, 0, 2, 700, 3000, 90], [1, 2, 3, 2, 3, 1], seed=4)
    x, y, off, dg = (to_dev(v) for v in (bf.x, bf.y, bf.offsets, bf.degrees))
    a, b = both(monkeypatch, lambda: lf.fit_qr_batched(x, y, off, dg, 3, **kw))
    assert all(same(u, v) for u, v in zip(a[:3], b[:3])) and a[3].numel() == b[3].numel()
    out = tuple(torch.full_like(v, 3) for v in a[:3])
    c = lf.fit_qr_batched(x, y, off, dg, 3, ws=a[3], out=out, **kw)
    torch.cuda.synchronize()
    assert all(u.data_ptr() == v.data_ptr() for u, v in zip(c[:3], out)) and c[3].data_ptr() == a[3].data_ptr()
    assert same(c[0][:, :2], a[0][:, :2]) and same(c[1], a[1]) and same(c[2], a[2])
    calls = [lambda: lf.fit_qr_batched(x, y, off.int(), dg, 3), lambda: lf.fit_qr_batched(x, y, off, dg, 9),
             lambda: lf.fit_qr_batched(x, y, off, dg, 3, coef_stride=2), lambda: lf.fit_qr_batched(x[::2], y, off, dg, 3),
             lambda: lf.fit_qr_batched(x, y, off, dg, 3, center=0.0, scale=0.0)]
    for k, call in enumerate(calls):
        seen = []
        for native in (True, False):
            with monkeypatch.context() as m:
                if not native:
                    m.setattr(api, "_bind", Declines())
                with pytest.raises((TypeError, ValueError, RuntimeError, _lib.LsefitError)) as e:
                    call()
                seen.append((type(e.value), str(e.value)))
        assert seen[0] == seen[1], (k, seen)
