"""`inner` visits per round of a worker with one sub-domain: it makes one visit
and publishes its candidate like any other, so the round log holds it and the
rounds are those of inner = 1."""
import numpy as np
import pytest

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


def _log(lib, pb, rounds, nW, **kw):
    X, D = (torch.from_numpy(np.ascontiguousarray(a)).to("cuda", torch.float64) for a in (pb.X, pb.D))
    lam = 0.1 * lib.dicodile_lambda_max(X, D)
    audit = torch.full((rounds, nW), -1, dtype=torch.int64, device="cuda")
    z, info = lib.dicodile_csc(X, D, lam, 1e-8 * lam, audit=audit, max_rounds=rounds, max_polish=1, **kw)
    torch.cuda.synchronize()
    return audit.cpu().numpy(), z.cpu().numpy(), info


def test_round_log_of_greedy_workers(lib):
    pb = synth.make_problem("one", 81, P=1, T=(90, 100), K=3, L=(7, 6), rho=0.01, amp="uniform", sigma=0.1)
    ref, z0, i0 = _log(lib, pb, 60, 4, grid=(2, 2), strategy="greedy")
    log, z1, i1 = _log(lib, pb, 60, 4, grid=(2, 2), strategy="greedy", inner=3)
    assert (ref != 0).any() and np.array_equal(log, ref)
    assert np.array_equal(z0, z1) and i0["n_updates"] == i1["n_updates"]


def test_round_log_beside_a_worker_of_two_subdomains(lib):
    # 27 rows on two workers: 13 rows are one sub-domain of about 9, 14 rows two; the loudest
    # activation lies in the first worker, away from the border
    pb = synth.make_problem("two", 82, P=1, T=(32, 25), K=2, L=(6, 6), rho=0.01, amp="uniform", sigma=0.01)
    pb.X[:, 1:7, 9:15] += 50.0 * pb.D[1]
    log, _, _ = _log(lib, pb, 20, 2, grid=(2, 1), tile=(9, 20), inner=2)
    first = int(log[0, 0])
    assert first & (1 << 63) and first & (1 << 62)  # published and accepted
    assert (first >> 32) & 0xffff == 1 and first & 0xffffffff == 1 * 20 + 9
