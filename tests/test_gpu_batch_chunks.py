"""Batches whose lists of passers are longer than the Delta workspace: every group's chunks
stay in order beside the other groups'.  Two and three chunks, one and two coefficient
planes, groups that share a stream (five lane ranges), and an instance whose later chunks
are empty.  A capped ascent keeps it short.  Each instance's statistics and incumbent equal
those of its run alone (whose chunks the full-size tests compare with the oracle)."""
import numpy as np
import pytest

from paper_1706_00037_amd.inputs import make_instance

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def test_batch_with_several_chunks():
    from paper_1706_00037_amd import ubqp
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    ctx = ubqp.Context(0)
    cases = [(8000, 42000, 30000, 0), (4500, 70000, 30000, 0), (6500, 90000, 100, 0), (2500, 3000, 100, 0),
             (3500, 40000, 30000, 1), (900, 500, 30000, 0)]
    probs = [ctx.problem(make_instance(n, 0.1, -hi, hi, 31 + n)) for n, _, hi, _ in cases]
    kws = [dict(M=M, H=10, lam_num=lam, lam_den=2, G=2, max_flips=6, run_seed=n) for n, M, _, lam in cases]
    alone = [ctx.multistart(p, **kw) for p, kw in zip(probs, kws)]
    chunk = [(1 << 30) // (p.planes * p.n_pad * 4) // 256 * 256 for p in probs]
    passers = [int(r["stats"][0][2]) for r in alone]
    assert sum(P > c for P, c in zip(passers, chunk)) >= 3 and passers[4] < chunk[4] < kws[4]["M"]
    for k, r in enumerate(ctx.multistart_batched(probs, kws)):
        assert np.array_equal(r["stats"], alone[k]["stats"]), k
        assert r["best_f"] == alone[k]["best_f"] and np.array_equal(r["best_x"], alone[k]["best_x"]), k
