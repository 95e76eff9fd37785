"""One Delta-initialisation launch for a batch: its instances' tiles, one to some dozens each and
at offsets that are no multiple of the eight XCDs, are each taken once (vs the oracle; all values
are integers and equal)."""
import numpy as np
import pytest

import oracle
from paper_1706_00037_amd.inputs import make_instance

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hi", [100, 32767])
def test_batch_of_one_to_many_tiles(hi):
    from paper_1706_00037_amd import ubqp
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    shapes = [(60, 100), (900, 600), (130, 256), (400, 257), (1100, 1500), (128, 513), (640, 900)]
    ctx = ubqp.Context(0)
    Qs = [make_instance(n, 0.5, -hi, hi, 500 + n) for n, _ in shapes]
    probs = [ctx.problem(Q) for Q in Qs]
    params = [dict(M=M, H=4, lam_num=1, lam_den=2, G=2, run_seed=n) for n, M in shapes]
    for Q, kw, r in zip(Qs, params, ctx.multistart_batched(probs, params)):
        o = oracle.multistart(Q, threads=8, **kw)
        assert np.array_equal(r["stats"], o["stats"]) and r["best_f"] == o["best_f"]
        assert np.array_equal(r["best_x"], o["best_x"])
