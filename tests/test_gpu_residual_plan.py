"""Objective and KKT over the sizes at which the residual's plan changes: one to
many channels, few and many tiles, small and large atoms, sparse and dense
codes, against the oracle and in the order of the library's own repeat.

Tolerance: FP64 sums of n terms in any order, n 2^-53 of the sum of magnitudes;
the objective sums at most 4e5 squares and magnitudes of one sign, each a sum of
at most 3e4 terms: 1e-10 relative."""
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


# (P, T, K, L, density)
CASES = [(1, (700,), 3, (64,), 0.3), (1, (3000,), 2, (2500,), 0.2), (2, (5000,), 4, (16,), 0.05),
         (3, (60000,), 3, (8,), 0.01), (5, (4000,), 70, (12,), 0.02), (16, (8000,), 5, (20,), 0.02),
         (64, (2300,), 3, (9,), 0.05), (1, (64, 64), 25, (32, 32), 0.2), (1, (40, 57), 3, (5, 5), 0.1),
         (1, (9, 4000), 4, (8, 8), 0.1), (1, (300, 310), 5, (3, 3), 0.1), (2, (200, 150), 66, (7, 5), 0.01),
         (3, (256, 256), 3, (8, 8), 0.02), (1, (300, 300), 2, (60, 60), 0.02), (6, (150, 140), 4, (24, 20), 0.01),
         (1, (500, 500), 2, (20, 20), 0.005)]


@pytest.mark.parametrize("case", CASES, ids=str)
@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
def test_objective_over_the_plan(lib, case, dtype):
    P, T, K, L, rho = case
    rng = np.random.default_rng(7)
    H = tuple(t - l + 1 for t, l in zip(T, L))
    dev = [torch.from_numpy(a).to("cuda", dtype) for a in
           (rng.standard_normal((P,) + T), rng.standard_normal((K, P) + L),
            np.where(rng.random((K,) + H) < rho, rng.standard_normal((K,) + H), 0.0))]
    X, D, z = (a.cpu().double().numpy() for a in dev)
    obj, kkt = lib.dicodile_objective_kkt(*dev, 0.7)
    assert obj == pytest.approx(oracle.objective(X, D, z, 0.7), rel=1e-10)
    assert kkt == pytest.approx(oracle.kkt(X, D, z, 0.7), rel=1e-10)
