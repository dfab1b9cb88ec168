"""DtD of many-channel signal atoms (computed by FFT) whose norms differ by
orders of magnitude: every entry DtD[k, k0] is compared at the scale of its own
two atoms.

Tolerance: the rounding of a transform of 1024 points and of the sum over the
channels, relative to ||D_k|| ||D_k0||: 1e-12 as for equal norms (FP32: the
rounding of the result, 2^-24, on top)."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def lib():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1901_09235_amd as dl
    dl.load()
    return dl


def atoms():
    D = np.random.default_rng(5).standard_normal((40, 16, 128))
    return D / np.sqrt((D ** 2).sum(axis=(1, 2), keepdims=True))


def dtd(lib, D, dtype):
    d = torch.from_numpy(np.ascontiguousarray(D)).to("cuda", dtype)
    return lib.dicodile_dtd(d).cpu().double().numpy(), d.cpu().double().numpy()


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
def test_atoms_of_unequal_norms(lib, dtype):
    D = atoms()
    scale = np.ones(40)
    scale[3], scale[4], scale[17], scale[18], scale[39] = 1e-8, 3e5, 1e-4, 1e9, 1e-12
    C, Dr = dtd(lib, D * scale[:, None, None], dtype)
    n = np.sqrt((Dr ** 2).sum(axis=(1, 2)))
    err = np.abs(C - oracle.dtd(Dr)) / (n[:, None, None] * n[None, :, None])
    assert err.max() <= (1e-12 if dtype == torch.float64 else 1e-12 + 2.0 ** -24)


def test_atoms_whose_squares_leave_the_fp64_range(lib):
    D = atoms()
    scale = np.ones(40)
    scale[5], scale[6] = 1e-170, 1e160
    C, Dr = dtd(lib, D * scale[:, None, None], torch.float64)
    ref = oracle.dtd(D)
    for k, j in ((5, 9), (9, 5), (6, 9), (9, 6), (5, 6), (9, 9), (7, 8)):
        np.testing.assert_allclose(C[k, j] / (scale[k] * scale[j]), ref[k, j], rtol=0, atol=1e-12)


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
def test_zero_atoms_give_zeros(lib, dtype):
    D = atoms()
    D[7] = 0.0
    D[39] = 0.0
    C, Dr = dtd(lib, D, dtype)
    assert not C[[7, 39]].any() and not C[:, [7, 39]].any()
    np.testing.assert_allclose(C, oracle.dtd(Dr), rtol=0, atol=1e-12 if dtype == torch.float64 else 1e-6)


def test_a_tap_that_is_not_finite_concerns_its_atom_only(lib):
    D = atoms()
    D[11, 2, 5] = np.inf
    D[12] = 0.0
    C, _ = dtd(lib, D, torch.float64)
    rest = [k for k in range(40) if k != 11]
    D[11] = 0.0
    np.testing.assert_allclose(C[np.ix_(rest, rest)], oracle.dtd(D)[np.ix_(rest, rest)], rtol=0, atol=1e-12)
    assert np.isinf(C[11, 11, 127])
    assert not np.isfinite(C[11, [0, 20]][:, 127]).any() and not np.isfinite(C[[0, 20], 11][:, 127]).any()
