"""The (split) BF16 correlation of one-channel images in its atom-major form
against the FP64 oracle, at the edges of its tiles: ragged rows and columns of
positions, atoms of 1 to 33 columns (one to five groups of eight taps), counts
of groups that do not fill the last step, and one to five atom tiles.

The oracle gets what the products get: operands rounded to BF16 (hi), and for
the split form also their rounded remainders (lo), as hi hi + hi lo + lo hi.
Those products are exact in FP32, so what remains is the rounding of the FP32
sums: at most N 2^-23 of the sum of magnitudes over the N terms."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _split(a):
    hi = torch.from_numpy(a).bfloat16().float().numpy()
    lo = torch.from_numpy(a - hi).bfloat16().float().numpy()
    return hi.astype(np.float64), lo.astype(np.float64)


@pytest.mark.parametrize("prec", ["bf16", "bf16x3"])
@pytest.mark.parametrize("K,T,L", [(1, (2, 3), (1, 1)), (5, (9, 70), (3, 5)), (16, (40, 64), (8, 8)), (17, (37, 133), (12, 9)),
                                   (25, (64, 200), (16, 16)), (40, (50, 66), (5, 17)), (70, (33, 90), (2, 33)),
                                   (3, (20, 21), (20, 20)), (25, (90, 85), (32, 32)), (4, (70, 64), (60, 7))])
def test_matches_oracle(prec, K, T, L):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1901_09235_amd as dl
    rng = np.random.default_rng(K)
    X = rng.standard_normal((1,) + T).astype(np.float32)
    D = rng.standard_normal((K, 1) + L).astype(np.float32)
    G = dl.dicodile_corr(torch.from_numpy(X).cuda(), torch.from_numpy(D).cuda(), prec).cpu().double().numpy()
    (Xh, Xl), (Dh, Dl) = _split(X), _split(D)
    ref, size, terms = oracle.corr(Xh, Dh), oracle.corr(np.abs(Xh), np.abs(Dh)), L[0] * L[1]
    if prec == "bf16x3":
        ref = ref + oracle.corr(Xl, Dh) + oracle.corr(Xh, Dl)
        size = size + oracle.corr(np.abs(Xl), np.abs(Dh)) + oracle.corr(np.abs(Xh), np.abs(Dl))
        terms *= 3
    assert (np.abs(G - ref) <= terms * 2.0 ** -23 * size).all()
