"""The round kernel's ways of putting workers and atoms on a workgroup, against
the FP64 oracle: every lane map (how the lanes of a wave share a position's
atoms, up to atom counts that one wave loops over), teams of several workers
with each selection rule and several visits per round, regions too large for
the LDS score copy, and one worker per small workgroup.

Solves are compared by relative objective gap <= 1e-6 and strict KKT <= 1e-4
lambda, the target of every solve."""
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


def _solve_and_grade(lib, pb, dtype, tol_rel=1e-5, positive=False, **opts):
    lam = 0.1 * oracle.lambda_max(pb.X, pb.D, positive=positive)
    X, D = (torch.from_numpy(np.ascontiguousarray(a)).to("cuda", dtype) for a in (pb.X, pb.D))
    z, info = lib.dicodile_csc(X, D, lam, tol_rel * lam, positive=positive, max_rounds=20_000_000, timeout_s=60, **opts)
    assert info["status"] == "OK", info
    Zg = z.cpu().double().numpy()
    Zo, _ = oracle.lgcd(pb.X, pb.D, lam, 1e-7 * lam, positive=positive)
    fo = oracle.objective(pb.X, pb.D, Zo, lam)
    gap = (oracle.objective(pb.X, pb.D, Zg, lam) - fo) / abs(fo)
    assert gap <= 1e-6, gap
    assert oracle.kkt(pb.X, pb.D, Zg, lam, positive=positive) <= 1e-4
    return info


# 16-byte groups per position: FP32 ceil(K / 4), FP64 ceil(K / 2)
@pytest.mark.parametrize("dtype,K", [(torch.float32, K) for K in (1, 6, 9, 14, 18, 27, 33, 41, 67, 130)] +
                         [(torch.float64, K) for K in (1, 3, 5, 7, 12, 21, 34)])
def test_lane_maps(lib, dtype, K):
    pb = synth.make_problem("lanes", 300 + K, P=1, T=(23, 26), K=K, L=(4, 3), rho=0.02 / K, amp="uniform", sigma=0.1)
    _solve_and_grade(lib, pb, dtype, positive=K % 2 == 0)


@pytest.mark.parametrize("dtype,K", [(torch.float32, 900), (torch.float64, 420)])
def test_atoms_beyond_one_wave(lib, dtype, K):
    pb = synth.make_problem("wide", 31, P=1, T=(14, 15), K=K, L=(3, 3), rho=1e-4, amp="uniform", sigma=0.1)
    _solve_and_grade(lib, pb, dtype)


@pytest.mark.parametrize("opts", [{}, {"inner": 2}, {"strategy": "random", "seed": 5}, {"strategy": "greedy"},
                                  {"strategy": "cyclic"}], ids=["lgcd", "inner2", "random", "greedy", "cyclic"])
@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
def test_teams_of_workers(lib, dtype, opts):
    # more workers than CUs, a prime count per axis: full and ragged teams
    pb = synth.make_problem("teams", 41, P=1, T=(121, 163), K=2, L=(4, 5), rho=0.01, amp="uniform", sigma=0.1)
    info = _solve_and_grade(lib, pb, dtype, grid=(17, 23), tile=(4, 4), **opts)
    assert info["grid"] == (17, 23)


@pytest.mark.parametrize("T,grid", [((150, 170), (1, 1)), ((300, 290), (2, 1))])
def test_regions_beyond_the_score_copy(lib, T, grid):
    # 25,500 and 87,000 positions: more than the LDS scores, then than the non-zero bitmask of a region
    pb = synth.make_problem("large", 51, P=1, T=T, K=2, L=(4, 4), rho=0.001, amp="uniform", sigma=0.1)
    _solve_and_grade(lib, pb, torch.float32, grid=grid, tile=(40, 40))


def test_signal_workers_share_workgroups(lib):
    # more workers than CUs on a signal whose patches fill a large workgroup
    pb = synth.make_problem("sig", 61, P=2, T=9000, K=20, L=14, rho=0.001, amp="uniform", sigma=0.1)
    info = _solve_and_grade(lib, pb, torch.float32)
    assert info["grid"][1] > 256
