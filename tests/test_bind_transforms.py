"""The native marshalling and tensors without memory of their own: functorch's wrappers (vmap,
grad, jvp) have the exact type torch.Tensor, report the device of what they wrap and hold no
pointer.  The native module leaves them to the Python form of the call, which raises; nothing
throws while the interpreter is released."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
from torch._subclasses.fake_tensor import FakeTensorMode  # noqa: E402

lf = pytest.importorskip("paper_1512_08017_amd")
from paper_1512_08017_amd import api  # noqa: E402

TRANSFORMS = {
    "vmap": lambda f, x: torch.func.vmap(f)(torch.stack([x, x])),
    "grad": lambda f, x: torch.func.grad(lambda v: f(v).sum())(x),
    "jvp": lambda f, x: torch.func.jvp(f, (x,), (torch.ones_like(x),)),
}


@pytest.mark.parametrize("transform", list(TRANSFORMS))
def test_wrapped_tensors_are_declined(transform):
    """On tensors that only claim to be on a GPU: declined before anything asks for their memory."""
    from paper_1512_08017_amd import _bind
    seen = []

    class Seen(Exception):
        pass

    def f(x):
        seen.append(_bind.fit(x, x, 2, "f64", 1, None, None, None, "gepp", "monomial"))
        seen.append(_bind.fit_qr(x, x, 2, None, None, None, "f64", 0, "gepp", "monomial"))
        raise Seen   # there is no device for a backward pass

    with FakeTensorMode(), pytest.raises(Seen):
        TRANSFORMS[transform](f, torch.empty(16, dtype=torch.float64, device="cuda"))
    assert seen == [None, None]


class Declines:
    def __getattr__(self, name):
        return lambda *a: None


def same_error(monkeypatch, call):
    seen = []
    for native in (True, False):
        with monkeypatch.context() as m:
            if not native:
                m.setattr(api, "_bind", Declines())
            with pytest.raises(RuntimeError) as e:
                call()
            seen.append((type(e.value), str(e.value)))
    assert seen[0] == seen[1]
    return seen[0][1]


@pytest.mark.gpu
@pytest.mark.parametrize("transform", list(TRANSFORMS))
def test_errors_under_transforms(monkeypatch, transform):
    rng = np.random.default_rng(1)
    x, y = (torch.from_numpy(rng.standard_normal(200)).cuda() for _ in range(2))
    off = torch.tensor([0, 90, 200], device="cuda")
    deg = torch.tensor([1, 2], dtype=torch.int32, device="cuda")
    done = lf.fit(x, y, 2)
    _, _, ws = lf.fit_batched(x, y, off, deg, 2)
    g = torch.ones(2, 3, dtype=torch.float64, device="cuda")
    calls = {
        "fit": lambda v: lf.fit(v, y, 2).coef,
        "fit, y": lambda v: lf.fit(x, v, 2).coef,
        "fit_qr": lambda v: lf.fit_qr(v, y, 2).coef,
        "residuals": lambda v: lf.residuals(v, y, done, store=True)[1],
        "fit_batched": lambda v: lf.fit_batched(v, y, off, deg, 2)[0],
        "fit_qr_batched": lambda v: lf.fit_qr_batched(v, y, off, deg, 2)[0],
        "fit_backward": lambda v: lf.fit_backward(v, y, off, deg, 2, g, ws=ws)[0],
    }
    for name, f in calls.items():
        assert "data pointer" in same_error(monkeypatch, lambda: TRANSFORMS[transform](f, x)), name


@pytest.mark.gpu
def test_batched_gradients_of_the_adjoint(monkeypatch):
    """is_grads_batched hands the backward a wrapped gradient."""
    rng = np.random.default_rng(2)
    x, y = (torch.from_numpy(rng.standard_normal(200)).cuda().requires_grad_() for _ in range(2))
    off = torch.tensor([0, 90, 200], device="cuda")
    deg = torch.tensor([1, 2], dtype=torch.int32, device="cuda")
    grads = torch.ones(4, 2, 3, dtype=torch.float64, device="cuda")

    def call():
        torch.autograd.grad(lf.lsefit(x, y, off, deg, 2), (x, y), grad_outputs=grads, is_grads_batched=True)

    assert "data pointer" in same_error(monkeypatch, call)
