"""The gathered FP64 residual against the oracle's direct loops, through the
objective and KKT of a given z: edges of the output tiles (64 columns, 8 or 32
rows; 256 samples, 8 channels), z with many non-zeros per position (several
passes over the list of a tile), more than 256 atoms (one position per thread
and pass), an empty z, and positions of z at every edge.

Tolerance: with a = |X| + |Z|*|D| and m = K #Theta terms per output, an output
of the residual is off by at most e = m 2^-53 a in either implementation, so
the objective differs by at most 2 sum |r| e + N 2^-53 of itself, and the KKT
by at most 2 (m + P #Theta) 2^-53 max corr(a, |D|) / lambda (the contraction's
own bound added)."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

U = 2.0 ** -53

# (P, K, T, L, share of non-zeros)
SHAPES = [
    (1, 1, (1,), (1,), 1.0),
    (7, 3, (256,), (16,), 0.3),
    (9, 5, (257,), (64,), 0.05),
    (1, 40, (700,), (9,), 1.0),
    (17, 300, (90,), (12,), 0.5),
    (1, 1, (1, 5), (1, 3), 1.0),
    (3, 4, (8, 64), (4, 4), 0.2),
    (1, 25, (33, 65), (5, 7), 1.0),
    (2, 300, (20, 30), (3, 6), 0.4),
    (1, 6, (40, 130), (16, 33), 0.0),
    (2, 3, (600, 1100), (8, 8), 0.01),
    (2, 5, (545, 1090), (5, 3), 1.0),
]


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("shape", SHAPES)
def test_objective_and_kkt(shape, dtype):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1901_09235_amd as dl
    P, K, T, L, share = shape
    rng = np.random.default_rng(1000 * P + K)
    nd = np.float64 if dtype == torch.float64 else np.float32
    V = tuple(t - l + 1 for t, l in zip(T, L))
    X = rng.standard_normal((P,) + T).astype(nd)
    D = rng.standard_normal((K, P) + L).astype(nd)
    Z = (rng.standard_normal((K,) + V) * (rng.random((K,) + V) < share)).astype(nd)
    edge = (0,) + tuple(v - 1 for v in V)
    if share:
        Z[(0,) * len(edge)] = Z[edge] = 0.5
    X64, D64, Z64 = X.astype(np.float64), D.astype(np.float64), Z.astype(np.float64)
    lam = 0.3 * oracle.lambda_max(X64, D64)
    obj, kkt = dl.dicodile_objective_kkt(*(torch.from_numpy(v).cuda() for v in (X, D, Z)), lam)

    Tr = T if len(T) == 2 else T[0]
    m, n = K * int(np.prod(L)), P * int(np.prod(L))
    a = np.abs(X64) + oracle.reconstruct(np.abs(Z64), np.abs(D64), Tr)
    r = np.abs(X64 - oracle.reconstruct(Z64, D64, Tr))
    want = oracle.objective(X64, D64, Z64, lam)
    assert abs(obj - want) <= 2 * m * U * float((r * a).sum()) + (X.size + Z.size) * U * want
    bound = 2 * (m + n) * U * float(oracle.corr(a, np.abs(D64)).max()) / lam
    assert abs(kkt - oracle.kkt(X64, D64, Z64, lam)) <= bound
