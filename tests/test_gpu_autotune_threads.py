"""The autotuner's `threads`: 128 and 256 stand for the same workers per CU in
FP32, so the choice stays at 256 whatever the noise of the trials."""
import numpy as np
import pytest

import oracle
from paper_1901_09235_amd import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def test_fp32_choice_keeps_256_threads():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1901_09235_amd as lib
    lib.load()
    for seed, lo in ((31, 30), (32, 60), (33, 100)):  # sizes apart: the tuner answers like sizes from its cache
        D = synth.gaussian_dictionary(np.random.Generator(np.random.PCG64(seed)), 3, 1, (5, 5))
        pbs = [synth.make_problem(f"t{i}", 100 * seed + i, P=1, T=(lo + 3 * i, lo + 5 * i), K=3, L=(5, 5), rho=0.01,
                                  amp="uniform", sigma=0.1, D=D) for i in range(3)]
        Xs = [torch.from_numpy(pb.X).to("cuda", torch.float32) for pb in pbs]
        lams = [0.1 * oracle.lambda_max(pb.X, D) for pb in pbs]
        kw, info = lib.dicodile_csc_batch_autotune(Xs, torch.from_numpy(D).to("cuda", torch.float32), lams,
                                                   [1e-5 * l for l in lams])
        assert info["cached"] == 0 and kw["threads"] == 256
