"""A batch with instances on both sides of 16384 candidates, the most that one block screens:
both screens' launch tables hold instances, beside the start values that only two-plane
instances need.  Statistics and incumbents equal the oracle's."""
import numpy as np
import pytest

import oracle
from paper_1706_00037_amd.inputs import make_instance

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def test_batch_across_the_one_block_screen():
    from paper_1706_00037_amd import ubqp
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    cases = [(70, 300, 100), (75, 16385, 30000), (66, 16384, 100), (80, 20000, 100), (90, 1, 30000),
             (64, 40000, 30000), (70, 16384, 30000)]
    Qs = [make_instance(n, 0.5, -hi, hi, 640 + k) for k, (n, _, hi) in enumerate(cases)]
    kws = [dict(M=M, H=3, lam_num=1, lam_den=2, G=3, run_seed=k) for k, (_, M, _) in enumerate(cases)]
    ctx = ubqp.Context(0)
    for r, Q, kw in zip(ctx.multistart_batched([ctx.problem(Q) for Q in Qs], kws), Qs, kws):
        want = oracle.multistart(Q, threads=8, **kw)
        assert np.array_equal(r["stats"], want["stats"])
        assert r["have_best"] == want["have_best"]
        if want["have_best"]:
            assert r["best_f"] == want["best_f"] and np.array_equal(r["best_x"], want["best_x"])
