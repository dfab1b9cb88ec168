"""The FP64 contraction of signals by overlap-save FFT against the oracle's
direct loops: block edges, one and several blocks, the short and the long
transform, and the tables and checks of a solve that use it.

Tolerance: FP64 transforms of N <= 8192 points have relative errors of order
log2(N) 2^-53 of the largest magnitudes, so |difference| <= 1e-12 max |G|, as
for images."""
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


def dev(a, dtype):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda", dtype)


# (P, K, T, L): one block, T at and beside a block's end, several blocks, long atoms
SHAPES = [(1, 1, 70, 64), (3, 5, 1024, 1), (2, 9, 1025, 100), (5, 17, 4000, 128), (2, 4, 2987, 512), (1, 3, 9000, 513),
          (2, 2, 20000, 1000)]


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("shape", SHAPES)
def test_solve_checks_by_fft(lib, shape, dtype):
    """A capped solve with the contractions forced to the FFT: the objective
    and KKT it reports are those of its iterate."""
    P, K, T, L = shape
    pb = synth.make_problem("s", 70 + K, P=P, T=T, K=K, L=L, rho=0.002, amp="uniform", sigma=0.1)
    lam = 0.2 * oracle.lambda_max(pb.X, pb.D)
    z, info = lib.dicodile_csc(dev(pb.X, dtype), dev(pb.D, dtype), lam, 1e-5 * lam, max_rounds=7, fp64_method="fft")
    assert info["n_fft64"] >= 1
    Z, X, D = z.cpu().double().numpy(), dev(pb.X, dtype).cpu().double().numpy(), dev(pb.D, dtype).cpu().double().numpy()
    assert info["objective"] == pytest.approx(oracle.objective(X, D, Z, lam), rel=1e-12)
    gmax = oracle.lambda_max(X, D)
    assert abs(info["kkt"] - oracle.kkt(X, D, Z, lam)) <= 1e-12 * gmax / lam
    # and the same solve on the matrix cores ends on the same iterate to FP64 rounding of the tables
    z2, _ = lib.dicodile_csc(dev(pb.X, dtype), dev(pb.D, dtype), lam, 1e-5 * lam, max_rounds=7, fp64_method="mfma")
    rtol = 1e-11 if dtype == torch.float64 else 1e-5
    assert float((z - z2).abs().max()) <= rtol * max(1.0, float(z2.abs().max()))


@pytest.mark.parametrize("positive", [False, True])
def test_lambda_max_of_a_long_recording(lib, positive):
    # large enough that the library picks the FFT by itself
    pb = synth.make_problem("s", 81, P=8, T=60011, K=20, L=100, rho=0.001, amp="exp", sigma=0.1)
    ref = oracle.lambda_max(pb.X, pb.D, positive=positive)
    assert lib.dicodile_lambda_max(dev(pb.X, torch.float64), dev(pb.D, torch.float64), positive=positive) == \
        pytest.approx(ref, rel=1e-12)


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
def test_dtd_of_many_channel_atoms(lib, dtype):
    D = np.random.default_rng(5).standard_normal((40, 16, 128))
    D /= np.sqrt((D ** 2).sum(axis=(1, 2), keepdims=True))
    C = lib.dicodile_dtd(dev(D, dtype)).cpu().double().numpy()
    ref = oracle.dtd(dev(D, dtype).cpu().double().numpy())
    np.testing.assert_allclose(C, ref, rtol=0, atol=1e-12 if dtype == torch.float64 else 1e-6)


def test_warm_start_polishes_by_fft(lib):
    pb = synth.make_problem("s", 91, P=8, T=30000, K=12, L=64, rho=0.001, amp="exp", sigma=0.1)
    lam = 0.2 * oracle.lambda_max(pb.X, pb.D)
    X, D = dev(pb.X, torch.float32), dev(pb.D, torch.float32)
    z, a = lib.dicodile_csc(X, D, lam, 1e-5 * lam, fp64_method="fft")
    z2, b = lib.dicodile_csc(X, D, lam, 1e-5 * lam, z_out=z.clone(), warm_start=True, fp64_method="fft")
    assert a["status"] == b["status"] == "OK" and b["n_fft64"] >= 2
    assert b["n_updates"] <= a["n_updates"] // 4
    assert b["objective"] <= a["objective"] * (1 + 1e-9)
