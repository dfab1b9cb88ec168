"""The largest solves dicodile_csc_noalloc takes, without a GPU: the check of
the workspace precedes any device access, so a solve that fits fails only for
want of a device, and one that does not is refused with EINVAL."""
import ctypes
import os

import pytest


@pytest.fixture(scope="module")
def dl():
    import paper_1901_09235_amd as dl
    from paper_1901_09235_amd import build
    if not os.path.exists(dl.library_path()):
        build.build()
    dl.load()
    return dl


def _ask(dl, ndim, T, L, K, dtype):
    s = dl.Shape()
    s.ndim, s.P, s.K = ndim, 1, K
    for i in range(ndim):
        s.T[i], s.L[i] = T[i], L[i]
    o = dl.CscOpts()
    o.lambda_, o.tol, o.dtype, o.warm_start = 1.0, 1e-3, dtype, 1
    p = ctypes.c_void_p(16)
    lib = dl.load()
    rc = lib.dicodile_csc_noalloc(ctypes.byref(s), p, p, ctypes.byref(o), p, None, None)
    return rc, lib.dicodile_last_error().decode()


# the largest T that fits 64 MiB, found with the first version of the call
@pytest.mark.parametrize("T,L,K,dtype", [((575673,), (64,), 5, 1), ((179074,), (128,), 40, 0),
                                         ((500, 2821), (8, 8), 4, 0), ((100, 5012), (12, 12), 16, 0)], ids=str)
def test_the_largest_solve_fits(dl, T, L, K, dtype):
    torch = pytest.importorskip("torch")
    if torch.cuda.is_available():
        pytest.skip("the call would run")
    rc, msg = _ask(dl, len(T), T, L, K, dtype)
    assert "scratch" not in msg, msg
    rc, msg = _ask(dl, len(T), T[:-1] + (T[-1] + 1,), L, K, dtype)
    assert rc == -1 and "fixed scratch" in msg, (rc, msg)
