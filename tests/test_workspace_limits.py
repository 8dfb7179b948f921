"""Workspace sizes: one slot per wave and fit, and nothing for a pass that the fit does not run."""
import ctypes

import numpy as np
import pytest

from paper_1512_08017_amd import _lib


def sized(waves, wpb, degree, batch=1):
    s = _lib.Schedule(waves, wpb, 2048, 2)
    return _lib.load().lsefit_workspace_bytes(batch, degree, ctypes.byref(s))


@pytest.mark.parametrize("wpb", [1, 2, 4])
@pytest.mark.parametrize("degree", [1, 3, 8, 12, 16])
def test_bytes_per_wave(degree, wpb):
    """3m + 1 sums, or the 2 (m + 1) + m (m + 1)/2 + 1 entries of a QR factor where the degree has one."""
    sums = 3 * degree + 1
    slot = max(sums, 2 * (degree + 1) + degree * (degree + 1) // 2 + 1) if degree <= 8 else sums
    for batch in (1, 1000):
        assert sized(40_960, wpb, degree, batch) - sized(8_192, wpb, degree, batch) == 8 * slot * 32_768


@pytest.mark.parametrize("degree,waves", [(1, 87_000), (3, 34_800), (8, 9_480)])
def test_schedules_that_fit_the_static_array(degree, waves):
    assert 0 < sized(waves, 4, degree) <= _lib.NOALLOC_SCRATCH_BYTES


@pytest.mark.gpu
@pytest.mark.parametrize("degree,waves", [(1, 87_000), (3, 34_800)])
def test_noalloc_on_the_largest_schedules(degree, waves):
    from gpu_common import announce, normwise, to_dev, torch
    from oracle import c_oracle
    from paper_1512_08017_amd import api, workloads as W
    announce(f"noalloc, degree {degree}, {waves} waves")
    L, vp, m = _lib.load(), ctypes.c_void_p, degree
    wl = W.random_small(300_007, m, seed=m, dtype=np.float32)
    x, y = to_dev(wl.x), to_dev(wl.y)
    coef = torch.empty(2 * (m + 1), dtype=torch.float64, device=x.device)
    status = torch.empty(1, dtype=torch.int32, device=x.device)
    s, o = _lib.Schedule(waves, 4, 2048, 2), api.options(m)
    _lib.check(L.lsefit_set_default_schedule(ctypes.byref(s)), "lsefit_set_default_schedule")
    try:
        rc = L.fit_single_noalloc(vp(x.data_ptr()), vp(y.data_ptr()), x.numel(), _lib.F32, ctypes.byref(o),
                                  vp(coef.data_ptr()), vp(status.data_ptr()), None,
                                  vp(torch.cuda.current_stream().cuda_stream))
    finally:
        _lib.check(L.lsefit_set_default_schedule(None), "lsefit_set_default_schedule")
    torch.cuda.synchronize()
    assert rc == _lib.OK and int(status.cpu()[0]) == 0
    assert normwise(coef.cpu().numpy()[: m + 1], c_oracle.fit(wl.x, wl.y, m)["a"]) <= 1e-9


@pytest.mark.gpu
@pytest.mark.parametrize("degree", [1, 2, 8, 9, 16])
@pytest.mark.parametrize("waves,wpb", [(2048, 4), (2048, 1), (2047, 1), (1, 1), (63, 2)])
def test_range_pairs_stay_inside(degree, waves, wpb):
    """A Chebyshev fit with its range from the data, on exactly the bytes that it asks for: the
    extent found is that of the data, and nothing past the workspace changes."""
    from gpu_common import announce, normwise, to_dev, torch
    from oracle import cheb
    from paper_1512_08017_amd import api, workloads as W
    import paper_1512_08017_amd as lf
    announce(f"Chebyshev range pairs, degree {degree}, {waves} waves, {wpb} per block")
    wl = W.random_small(200_003, 3, seed=degree, dtype=np.float64)
    x, y = to_dev(wl.x), to_dev(wl.y)
    try:
        lf.set_default_schedule({"waves": waves, "waves_per_block": wpb, "tile": 2048, "unroll": 2})
        need = api.workspace_bytes(1, degree)
        space = torch.full((need + 65_536,), 0x5A, dtype=torch.uint8, device=x.device)
        r = lf.fit(x, y, degree, basis="chebyshev", ws=space[:need])
    finally:
        lf.set_default_schedule(None)
    torch.cuda.synchronize()
    assert bool((space[need:] == 0x5A).all())
    lo, hi = wl.x.min(), wl.x.max()
    assert (r.center, r.scale) == (0.5 * hi + 0.5 * lo, 0.5 * hi - 0.5 * lo) and int(r.status.cpu()[0]) == 0
    V = np.polynomial.chebyshev.chebvander((wl.x - r.center) / r.scale, degree)
    tol = max(1e-12, 1e3 * np.finfo(float).eps * np.linalg.cond(V.T @ V))
    ref = cheb.fit_cheb(wl.x, wl.y, degree, r.center, r.scale)
    assert normwise(r.coef_cheb.cpu().numpy(), np.asarray(ref["c"], float)) <= tol
