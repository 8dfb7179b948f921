"""Calls that the C ABI refuses stay refused, with the same error, whichever form marshals them;
and the calls that the native module is there for are taken by it, not left to the other form."""
import numpy as np
import pytest

from gpu_common import to_dev, torch
from paper_1512_08017_amd import workloads as W

pytestmark = pytest.mark.gpu

lf = pytest.importorskip("paper_1512_08017_amd")
from paper_1512_08017_amd import _lib, api  # noqa: E402


class Recorder:
    """The native module, noting which of its functions took a call."""
    def __init__(self):
        self.native, self.took = api._native(), []

    def __getattr__(self, name):
        f = getattr(self.native, name)

        def call(*a):
            r = f(*a)
            self.took.append((name, r is not None))
            return r
        return call


class Declines:
    def __getattr__(self, name):
        return lambda *a: None


def refused(monkeypatch, call, code):
    for native in (True, False):
        with monkeypatch.context() as m:
            if not native:
                m.setattr(api, "_bind", Declines())
            with pytest.raises(_lib.LsefitError) as e:
                call()
        assert e.value.code == code, native


@pytest.fixture
def batch():
    bf = W.random_batch([50, 700], [1, 2], seed=5)
    return tuple(to_dev(v) for v in (bf.x, bf.y, bf.offsets, bf.degrees))


def test_closed_plan(monkeypatch, batch):
    plan = lf.Plan(2, 2)
    coef, _, _ = lf.fit_batched(*batch, 2, plan=plan)
    plan.close()
    refused(monkeypatch, lambda: lf.fit_batched(*batch, 2, plan=plan), _lib.WORKSPACE)
    refused(monkeypatch, lambda: lf.fit_backward(*batch, 2, torch.ones_like(coef), plan=plan), _lib.WORKSPACE)


def test_results_left_out(monkeypatch, batch):
    """out without its tensors is refused, not taken for no out; the QR batch may leave its sse out."""
    coef, status, _ = lf.fit_batched(*batch, 2)
    for out in ((None, None), (coef, None), (None, status)):
        refused(monkeypatch, lambda: lf.fit_batched(*batch, 2, out=out), _lib.INVALID_ARG)
    for out in ((None, None, None), (coef, None, None), (None, status, None)):
        refused(monkeypatch, lambda: lf.fit_qr_batched(*batch, 2, out=out), _lib.INVALID_ARG)
    qr, _, sse, _ = lf.fit_qr_batched(*batch, 2)
    got = lf.fit_qr_batched(*batch, 2, out=(coef, status, None))
    torch.cuda.synchronize()
    assert got[2] is None and torch.equal(got[0], qr) and (status == 0).all() and torch.isfinite(sse).all()


def test_plain_calls_are_taken_natively(monkeypatch, batch):
    """The native module takes every plain call, and no odd one."""
    x, y, off, deg = batch
    ws1 = torch.empty(lf.workspace_bytes(1, 3), dtype=torch.uint8, device=x.device)
    done, plan = lf.fit(x, y, 2), lf.Plan(2, 2)
    coef, _, ws = lf.fit_batched(x, y, off, deg, 2)
    out = (torch.empty_like(coef), torch.empty(2, dtype=torch.int32, device=x.device))
    g = torch.ones_like(coef)
    xr = x.clone().requires_grad_()
    plain = {
        "fit": [lambda: lf.fit(x, y, 3), lambda: lf.fit(x, y, 3, precision="f32c", refine=0, ws=ws1),
                lambda: lf.fit(x, y, 3, center=0, scale=2.5, solver="cholesky"), lambda: lf.fit(xr, y, 12, basis="chebyshev")],
        "fit_qr": [lambda: lf.fit_qr(x, y, 3), lambda: lf.fit_qr(x, y, 3, center=0.5, scale=2, ws=ws1)],
        "residuals": [lambda: lf.residuals(x, y, done), lambda: lf.residuals(x, y, done, store=True)],
        "fit_batched": [lambda: lf.fit_batched(x, y, off, deg, 2), lambda: lf.fit_batched(x, y, off, deg, 2, plan=plan),
                        lambda: lf.fit_batched(x, y, off, deg, 2, out=out, ws=ws),
                        lambda: lf.fit_batched(x, y, off, deg, 2, output_basis="x_and_t", coef_stride=9),
                        lambda: lf.fit_batched(x, y, off, deg, 2, basis="chebyshev", precision="f64")],
        "fit_qr_batched": [lambda: lf.fit_qr_batched(x, y, off, deg, 2),
                           lambda: lf.fit_qr_batched(x, y, off, deg, 2, center=0.0, scale=1.0, coef_stride=5, ws=ws)],
        "fit_backward": [lambda: lf.fit_backward(x, y, off, deg, 2, g, ws=ws),
                         lambda: lf.fit_backward(x, y, off, deg, 2, g.float(), plan=plan)],
    }
    odd = [lambda: lf.fit(torch.nn.Parameter(x, requires_grad=False), y, np.int32(3)),
           lambda: lf.fit(x, y, np.int64(3)), lambda: lf.residuals(x, y, done, store=1)]
    lf.fit_batched(x, y, off, deg, 2, plan=plan)
    for name, calls in plain.items():
        for k, call in enumerate(calls):
            rec = Recorder()
            with monkeypatch.context() as m:
                m.setattr(api, "_bind", rec)
                call()
            assert rec.took == [(name, True)], (name, k, rec.took)
    for k, call in enumerate(odd):
        rec = Recorder()
        with monkeypatch.context() as m:
            m.setattr(api, "_bind", rec)
            call()
        assert len(rec.took) == 1 and not rec.took[0][1], (k, rec.took)
    torch.cuda.synchronize()
