"""Servers whose ready requests ask for more workers than one launch holds, and
requests whose worker grids do not divide into teams: every request is solved
as dicodile_csc solves it on its own (FP64: the same minimiser to 1e-6 of its
largest value; objectives to 1e-9)."""
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


def dev(a, dtype):
    return torch.from_numpy(np.ascontiguousarray(a)).to(device="cuda", dtype=dtype)


def serve(lib, pbs, D, dtype, rel, **kw):
    """Every problem through one server at once; compared with its own solve."""
    Dd = dev(D, dtype)
    Xs = [dev(pb.X, dtype) for pb in pbs]
    lams = [0.2 * lib.dicodile_lambda_max(X, Dd) for X in Xs]
    torch.cuda.synchronize()
    with lib.Server(Dd, **kw) as srv:
        tickets = [srv.submit(X, lam, rel * lam, timeout_s=60) for X, lam in zip(Xs, lams)]
        res = [srv.wait(t, timeout_s=120) for t in tickets]
        st = srv.stats()
    for X, lam, (z, info) in zip(Xs, lams, res):
        assert info["status"] == "OK", info
        z1, one = lib.dicodile_csc(X, Dd, lam, rel * lam, timeout_s=60)
        assert info["objective"] == pytest.approx(one["objective"], rel=1e-9 if dtype == torch.float64 else 1e-6)
        if dtype == torch.float64:
            assert float((z - z1).abs().max()) <= 1e-6 * float(z1.abs().max())
    return st, [info["grid"] for _, info in res]


def test_fp64_requests_of_more_workers_than_a_launch_holds(lib):
    """admit_workers = -1 admits all eight requests of 128 workers, more than the
    library counts as running together in FP64 (three per CU)."""
    D = synth.gaussian_dictionary(np.random.Generator(np.random.PCG64(21)), 5, 1, 64)
    pbs = [synth.make_problem(f"r{i}", 2100 + i, P=1, T=20000 + 37 * i, K=5, L=64, rho=0.004, amp="uniform",
                              sigma=0.1, D=D) for i in range(8)]
    st, grids = serve(lib, pbs, D, torch.float64, 1e-9, admit_workers=-1, max_len=32768)
    assert all(g == (1, 128) for g in grids)
    assert st["peak_active"] == 8


def test_image_request_whose_workers_make_too_many_teams(lib):
    """31 x 33 workers: 264 teams of four, more than one per CU, in one request."""
    D = synth.gaussian_dictionary(np.random.Generator(np.random.PCG64(22)), 4, 1, (10, 10))
    pbs = [synth.make_problem(f"i{i}", 2200 + i, P=1, T=t, K=4, L=(10, 10), rho=0.002, amp="uniform", sigma=0.1, D=D)
           for i, t in enumerate([(324, 344), (60, 70), (324, 344)])]
    _, grids = serve(lib, pbs, D, torch.float32, 1e-5, max_workers=1024, tile=(10, 10), max_len=1 << 17)
    assert grids[0] == (31, 33) and grids[2] == (31, 33)


def test_many_requests_of_a_few_workers(lib):
    """150 requests of five workers each: 300 teams of four, 150 of five."""
    D = synth.gaussian_dictionary(np.random.Generator(np.random.PCG64(23)), 32, 1, 64)
    pbs = [synth.make_problem(f"r{i}", 2300 + i, P=1, T=1663 + i, K=32, L=64, rho=0.001, amp="uniform", sigma=0.1, D=D)
           for i in range(150)]
    _, grids = serve(lib, pbs, D, torch.float32, 1e-5, tile=320, slice_rounds=16)
    assert all(g == (1, 5) for g in grids)


def test_a_request_of_too_many_teams_is_not_passed_over(lib):
    """The oldest request makes 264 teams of four, the younger ones 256 each, which
    hold more workers: the oldest still goes first."""
    D = synth.gaussian_dictionary(np.random.Generator(np.random.PCG64(24)), 4, 1, (10, 10))
    pbs = [synth.make_problem(f"i{i}", 2400 + i, P=1, T=t, K=4, L=(10, 10), rho=0.004, amp="uniform", sigma=0.1, D=D)
           for i, t in enumerate([(324, 344)] + 5 * [(334, 334)])]
    Xs, Dd = [dev(pb.X, torch.float32) for pb in pbs], dev(D, torch.float32)
    lams = [0.05 * lib.dicodile_lambda_max(X, Dd) for X in Xs]
    torch.cuda.synchronize()
    with lib.Server(Dd, max_workers=1024, tile=(10, 10), max_len=1 << 17, admit_workers=-1, slice_rounds=16) as srv:
        tickets = [srv.submit(X, lam, 1e-5 * lam, timeout_s=60) for X, lam in zip(Xs, lams)]
        infos = [srv.wait(t, timeout_s=120)[1] for t in tickets]
    assert [i["grid"] for i in infos] == [(31, 33)] + 5 * [(32, 32)]
    assert all(i["status"] == "OK" for i in infos)
    assert infos[0]["t_total_s"] < min(i["t_total_s"] for i in infos[1:])
