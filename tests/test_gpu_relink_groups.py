"""Relinking with one wave per path at the path counts where the walk's launch changes:
the last count of single-wave workgroups and the first of grouped ones (768, 769), last
groups of one to four paths, the first count beyond the teams (513), and a pair outside
the elite set inside a group.  Every path's steps, values and row equal the oracle's."""
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


def walk(ctx, Q, elite, pairs):
    prob, P = ctx.problem(Q), len(pairs)
    X = torch.empty((P, prob.W), dtype=torch.int64, device="cuda")
    fm, fo = (torch.empty(P, dtype=torch.int64, device="cuda") for _ in range(2))
    st = torch.empty(P, dtype=torch.int32, device="cuda")
    ctx.relink(prob, torch.from_numpy(elite.view(np.int64)).cuda(), torch.from_numpy(pairs).cuda(), X, fm, fo, st)
    return X, fm, fo, st


def same(out, o, sel):
    X, fm, fo, st = (t.cpu().numpy()[sel] for t in out)
    assert np.array_equal(st, o["steps"]) and np.array_equal(fm, o["f_mid"])
    assert np.array_equal(fo, o["f_out"]) and np.array_equal(X.view(np.uint64), o["X"])


def all_pairs(E, P):
    return np.array([(a, b) for a in range(E) for b in range(E) if a != b], np.int32)[:P]


@pytest.mark.parametrize("n,P,lo,hi", [
    (130, 1, -100, 100), (130, 767, -100, 100), (130, 768, -100, 100), (130, 769, -100, 100),
    (130, 770, -100, 100), (130, 771, -32768, 32767), (1100, 772, -100, 100), (3100, 515, -100, 100),
    (3100, 514, -32768, 32767), (130, 4099, -100, 100),
])
def test_path_counts(ub, n, P, lo, hi):
    Q = make_instance(n, 0.3, lo, hi, 410 + P)
    E = 66 if P > 4000 else 29
    elite, pairs = random_candidates(E, n, 411 + n), all_pairs(E, P)
    ctx = ub.Context(0)
    out = walk(ctx, Q, elite, pairs)
    ctx.sync()
    same(out, oracle.relink_many(Q, elite, pairs, threads=8), slice(None))


def test_bad_pair_inside_a_group(ub):
    n, P, bad = 130, 801, 398
    Q = make_instance(n, 0.3, -100, 100, 17)
    elite, pairs = random_candidates(29, n, 18), all_pairs(29, P)
    sel = np.arange(P) != bad
    want = oracle.relink_many(Q, elite, pairs[sel], threads=8)
    pairs[bad] = (3, 29)
    ctx = ub.Context(0)
    out = walk(ctx, Q, elite, pairs)
    with pytest.raises(ub.UbqpError):
        ctx.sync()
    same(out, want, sel)
    assert int(out[3][bad]) == 0 and int(out[2][bad]) == np.iinfo(np.int64).min
