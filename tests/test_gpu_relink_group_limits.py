"""Relinking where the walk's launch goes back from workgroups of four waves to single ones:
more paths than SIMDs (1024, 1025) with four column blocks, and walks of so many registers
that a SIMD holds one (six blocks of int16, eight of int8).  Steps, values and rows equal
the oracle's."""
import numpy as np
import pytest

import oracle
from paper_1706_00037_amd.inputs import make_instance, random_candidates

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,P,hi", [(3100, 1024, 100), (3100, 1025, 100), (3100, 768, 32767), (3100, 769, 32767),
                                    (3100, 1025, 32767), (5121, 770, 32767), (6200, 517, 100), (7169, 517, 100)])
def test_limits(n, P, hi):
    from paper_1706_00037_amd import ubqp
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    Q = make_instance(n, 0.2, -hi, hi, 900 + n)
    # elite rows that differ in a few dozen variables, so that the oracle's walks are short
    E = 34
    base = random_candidates(1, n, 901 + n)
    elite = np.repeat(base, E, axis=0)
    rng = np.random.default_rng(n + P)
    for e in range(E):
        for j in rng.choice(n, 12, replace=False):
            elite[e, j // 64] ^= np.uint64(1) << np.uint64(j % 64)
    pairs = np.array([(a, b) for a in range(E) for b in range(E) if a != b], np.int32)[:P]
    ctx = ubqp.Context(0)
    prob = ctx.problem(Q)
    X = torch.empty((P, prob.W), dtype=torch.int64, device="cuda")
    fm, fo = (torch.empty(P, dtype=torch.int64, device="cuda") for _ in range(2))
    st = torch.empty(P, dtype=torch.int32, device="cuda")
    ctx.relink(prob, torch.from_numpy(elite.view(np.int64)).cuda(), torch.from_numpy(pairs).cuda(), X, fm, fo, st,
               max_flips=3)
    ctx.sync()
    some = np.r_[0:8, P // 2:P // 2 + 8, P - 8:P]
    o = oracle.relink_many(Q, elite, pairs[some], max_flips=3, threads=8)
    assert np.array_equal(st.cpu().numpy()[some], o["steps"])
    assert np.array_equal(fm.cpu().numpy()[some], o["f_mid"]) and np.array_equal(fo.cpu().numpy()[some], o["f_out"])
    assert np.array_equal(X.cpu().numpy()[some].view(np.uint64), o["X"])
