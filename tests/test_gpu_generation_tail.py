"""Screening, ascent order, ranking and seed placement of a generation at the sizes where
their work changes hands: one block per instance up to 16384 candidates (1, 4 or 16 per
thread), several launches beyond, and more passers than the order keeps in registers.
Every generation's statistics, the incumbent and the objectives of the next generation
(which carry every seed) equal the oracle's, exactly: all values are integers."""
import numpy as np
import pytest

import oracle
from paper_1706_00037_amd.inputs import make_instance

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ub():
    from paper_1706_00037_amd import ubqp
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return ubqp


@pytest.mark.parametrize("M", [1, 2, 63, 1023, 1024, 1025, 4096, 4097, 16383, 16384, 16385, 40000])
@pytest.mark.parametrize("lam,lo,hi", [((1, 2), -100, 100), ((0, 1), -2, 2), ((0, 1), -30000, 30000)])
def test_generation_tail_matches_oracle(ub, M, lam, lo, hi):
    n, G = 70, 3
    Q = make_instance(n, 0.5, lo, hi, 900 + M)
    kw = dict(M=M, H=3, lam_num=lam[0], lam_den=lam[1], G=G, run_seed=M)
    want = oracle.multistart(Q, dump=True, threads=8, **kw)
    ctx = ub.Context(0)
    dump = torch.empty((G, M), dtype=torch.int64, device="cuda")
    got = ctx.multistart(ctx.problem(Q), f_dump=dump, **kw)
    assert np.array_equal(got["stats"], want["stats"])
    assert got["have_best"] == want["have_best"] and got["best_f"] == want["best_f"]
    if want["have_best"]:  # one candidate never passes a threshold: no incumbent, no solution
        assert np.array_equal(got["best_x"], want["best_x"])
    assert np.array_equal(dump.cpu().numpy(), want["f_all"])
