"""Ranking where the comparison range falls into slices shorter than a tile of 256: passer
counts just above 256 and 512 in a large population (slices of a few entries, tiles before,
after and across the ranked passers), many equal objectives.  The objectives of the next
generation carry every seed, so they show the ranks; all equal the oracle's."""
import numpy as np
import pytest

import oracle
from paper_1706_00037_amd.inputs import make_instance

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,lam,hi", [(4096, (2, 5), 100), (4096, (1, 3), 1), (16384, (1, 2), 100),
                                      (16384, (1, 2), 1), (16500, (1, 2), 2), (9000, (2, 5), 30000)])
def test_ranks_of_few_passers(M, lam, hi):
    from paper_1706_00037_amd import ubqp
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    n, G = 60, 3
    Q = make_instance(n, 0.4, -hi, hi, 800 + M + hi)
    kw = dict(M=M, H=2, lam_num=lam[0], lam_den=lam[1], G=G, run_seed=M)
    want = oracle.multistart(Q, dump=True, threads=8, **kw)
    assert (want["stats"][:, 2] > 256).any()
    ctx = ubqp.Context(0)
    dump = torch.empty((G, M), dtype=torch.int64, device="cuda")
    got = ctx.multistart(ctx.problem(Q), f_dump=dump, **kw)
    assert np.array_equal(got["stats"], want["stats"])
    assert np.array_equal(got["best_x"], want["best_x"])
    assert np.array_equal(dump.cpu().numpy(), want["f_all"])
