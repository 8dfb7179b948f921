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
        self.took = []

    def __getattr__(self, name):
        f = getattr(api._native(), name)

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
