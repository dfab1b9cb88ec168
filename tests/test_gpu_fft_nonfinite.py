"""Recordings with samples that are not finite, through the FP64 contraction
by overlap-save FFT: an infinite or NaN sample concerns the positions whose
windows hold it, as in the direct sums, and not the rest of its FFT block.
lambda_max and the KKT violation are maxima that pass over NaN.

Tolerance: that of the finite recordings, 1e-12 of the largest value."""
import numpy as np
import pytest

import oracle
from paper_1901_09235_amd import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def lib():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1901_09235_amd as dl
    dl.load()
    return dl


def dev(a, dtype=torch.float64):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda", dtype)


@pytest.fixture(scope="module")
def recording():
    # large enough that the library picks the FFT by itself
    pb = synth.make_problem("s", 81, P=8, T=60011, K=20, L=100, rho=0.001, amp="exp", sigma=0.1)
    G = oracle.corr(pb.X, pb.D)
    return pb.X, pb.D, np.abs(G).max(axis=0)


def _bad(X, best, kind):
    """X with samples of `kind` beside the loudest position: its own window stays clean."""
    X = X.copy()
    at = int(best.argmax())
    if kind == "all but a stretch":
        X[:, :at] = np.nan
        X[:, at + 400:] = np.nan
    elif kind == "last":
        X[3, -1] = np.nan
    elif kind == "two":
        X[1, at + 105], X[6, at - 7] = np.inf, -np.inf
    else:
        X[3, at + 110] = float(kind)
    return X


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("kind", ["inf", "-inf", "nan", "last", "two", "all but a stretch"])
def test_maxima_of_a_recording(lib, recording, kind, dtype):
    X, D, best = recording
    X = _bad(X, best, kind)
    Xr, Dr = (dev(a, dtype).cpu().double().numpy() for a in (X, D))
    with np.errstate(invalid="ignore"):
        G = oracle.corr(Xr, Dr)
    ref = float(np.nanmax(np.abs(G)))
    got = lib.dicodile_lambda_max(dev(X, dtype), dev(D, dtype))
    assert got == pytest.approx(ref, rel=1e-12)
    refp = float(max(0.0, np.nanmax(G)))
    assert lib.dicodile_lambda_max(dev(X, dtype), dev(D, dtype), positive=True) == pytest.approx(refp, rel=1e-12)
    lam = 0.5
    z = torch.zeros((D.shape[0], X.shape[1] - D.shape[2] + 1), dtype=dtype, device="cuda")
    _, kkt = lib.dicodile_objective_kkt(dev(X, dtype), dev(D, dtype), z, lam)
    assert kkt == pytest.approx((ref - lam) / lam, rel=1e-11)


def test_a_solve_leaves_only_the_windows_of_a_nan_sample(lib, recording):
    """A warm start builds beta with the FP64 contraction: by FFT and on the
    matrix cores it solves the same positions."""
    X, D, best = recording
    X = X.copy()
    X[3, int(best.argmax()) + 110] = np.nan
    lam = 0.2 * float(best.max())
    out = []
    for method in ("fft", "mfma"):
        z0 = torch.zeros((D.shape[0], X.shape[1] - D.shape[2] + 1), dtype=torch.float64, device="cuda")
        z, info = lib.dicodile_csc(dev(X), dev(D), lam, 1e-8 * lam, z_out=z0, warm_start=True, fp64_method=method,
                                   max_rounds=400, timeout_s=20)
        assert (info["n_fft64"] > 0) == (method == "fft")
        out.append(z.cpu().numpy())
    near = np.abs(np.arange(out[0].shape[1]) - int(best.argmax())) < 1000
    assert np.count_nonzero(out[1][:, near]) > 0
    np.testing.assert_allclose(out[0], out[1], rtol=0, atol=1e-6 * float(np.abs(out[1]).max()))
