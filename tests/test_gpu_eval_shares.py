"""How many workgroups share a tile's K range: eleven column tiles (only parts that fit the
chip) and twelve (one more), around 256 and 512 tiles in the launch, and batches whose
instances share one launch.  Objectives, statistics and incumbents are integers and equal
the oracle's."""
import numpy as np
import pytest

import oracle
from paper_1706_00037_amd.inputs import make_instance, random_candidates

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_1706_00037_amd import ubqp
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return ubqp.Context(0)


@pytest.mark.parametrize("n,M,lo,hi", [
    (1408, 300, -100, 100), (1409, 300, -100, 100),        # eleven and twelve column tiles, few rows
    (600, 13056, -100, 100), (600, 13057, -100, 100),      # 255 and 260 tiles: two parts, one
    (384, 21760, -128, 127), (1536, 10752, -100, 100),     # 255 and 504 tiles
    (1500, 2800, -32768, 32767), (700, 4300, -32768, 32767),
])
def test_eval(ctx, n, M, lo, hi):
    Q = make_instance(n, 0.6, lo, hi, 60 + n)
    X = random_candidates(M, n, 61 + n)
    f = torch.full((M,), -7, dtype=torch.int64, device="cuda")
    ctx.eval(ctx.problem(Q), torch.from_numpy(X.view(np.int64)).cuda(), f)
    torch.cuda.synchronize()
    assert np.array_equal(f.cpu().numpy(), oracle.eval_many(Q, X, threads=8))


@pytest.mark.parametrize("sizes", [
    [(500, 1000), (130, 40)],                              # both split
    [(1500, 600), (200, 3000), (90, 1)],
    [(300, 20000), (1000, 9000), (128, 50)],               # a small one beside more tiles than the chip holds
])
@pytest.mark.parametrize("hi", [100, 30000])
def test_batch(ctx, sizes, hi):
    Qs = [make_instance(n, 0.3, -hi, hi, 70 + n) for n, _ in sizes]
    kws = [dict(M=M, H=3, lam_num=4, lam_den=5, G=2, run_seed=n) for n, M in sizes]
    for r, Q, kw in zip(ctx.multistart_batched([ctx.problem(Q) for Q in Qs], kws), Qs, kws):
        want = oracle.multistart(Q, threads=8, **kw)
        assert np.array_equal(r["stats"], want["stats"])
        if want["have_best"]:
            assert r["best_f"] == want["best_f"] and np.array_equal(r["best_x"], want["best_x"])
