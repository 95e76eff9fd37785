"""ubqp_ascent where workgroups of four waves take the passers (two or three blocks of
columns per lane): passer counts at the edges of its waves and blocks, counts and list
lengths around one passer for each SIMD, a list longer than a chunk, the neighbouring lane
ranges, a flip cap and an index out of range.  Rows, objectives and flips equal the
oracle's."""
import numpy as np
import pytest

import oracle
from paper_1706_00037_amd.inputs import make_instance, random_candidates

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ub():
    from paper_1706_00037_amd import ubqp
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return ubqp


def ascend(ctx, Q, X, f, idx, P, mf=0):
    Xd, fd = torch.from_numpy(X.view(np.int64)).cuda(), torch.from_numpy(f).cuda()
    fl = torch.full((len(X),), -1, dtype=torch.int32, device="cuda")
    ctx.ascent(ctx.problem(Q), Xd, torch.from_numpy(idx).cuda(), torch.tensor([P], dtype=torch.int64, device="cuda"),
               fd, fl, max_flips=mf)
    return Xd, fd, fl


def same(out, Q, X, f, idx, mf=0):
    Xo, fo, flo = oracle.ascent_many(Q, X, idx, f, max_flips=mf, threads=8)
    Xd, fd, fl = (t.cpu().numpy() for t in out)
    assert np.array_equal(Xd.view(np.uint64), Xo) and np.array_equal(fd, fo)
    assert np.array_equal(fl[idx], flo[idx])
    assert (fl[np.setdiff1d(np.arange(len(X)), idx)] == -1).all()


@pytest.mark.parametrize("lo,hi", [(-3, 3), (-32768, 32767)])
@pytest.mark.parametrize("n,rows,P,mf", [
    (1025, 769, 769, 0), (1025, 768, 768, 0), (1030, 800, 1, 0), (1030, 800, 0, 0), (2048, 1100, 255, 3),
    (2048, 1100, 257, 3), (2049, 1100, 1023, 3), (2049, 1100, 1024, 3), (2049, 1100, 1025, 3), (3072, 900, 513, 3),
    (1100, 4200, 4150, 2), (1100, 4200, 700, 2), (1024, 1000, 1000, 0), (3073, 1000, 900, 3),
])
def test_counts(ub, n, rows, P, mf, lo, hi):
    Q = make_instance(n, 0.2, lo, hi, 500 + n)
    X = random_candidates(rows, n, 501 + rows)
    f = oracle.eval_many(Q, X, threads=8)
    idx = np.random.default_rng(P).permutation(rows).astype(np.int32)
    ctx = ub.Context(0)
    out = ascend(ctx, Q, X, f, idx, P, mf)
    ctx.sync()
    same(out, Q, X, f, idx[:P], mf)


def test_index_out_of_range(ub):
    n, rows = 1100, 800
    Q = make_instance(n, 0.2, -100, 100, 21)
    X = random_candidates(rows, n, 22)
    f = oracle.eval_many(Q, X, threads=8)
    idx = np.arange(rows, dtype=np.int32)
    idx[300] = rows
    ctx = ub.Context(0)
    out = ascend(ctx, Q, X, f, idx, rows)
    with pytest.raises(ub.UbqpError):
        ctx.sync()
    same(out, Q, X, f, np.delete(np.arange(rows, dtype=np.int32), 300))
