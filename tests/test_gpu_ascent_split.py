"""Few passers of instances too small for teams: the Delta initialisation splits its K
range and the one-wave ascent sums the partial rows.  One to three blocks of columns per
lane, one and several row tiles, little room in the list (fewer partials fit), the largest
population whose launches may split and the first that does not, both coefficient widths;
a batch whose launches hold neighbouring lane ranges, some of them split.  Every
generation's statistics and the incumbent are integers and equal the oracle's."""
import numpy as np
import pytest

import oracle
from paper_1706_00037_amd.inputs import make_instance

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_1706_00037_amd import ubqp
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return ubqp.Context(0)


def same(got, Q, kw):
    want = oracle.multistart(Q, threads=8, **kw)
    assert np.array_equal(got["stats"], want["stats"])
    assert got["best_f"] == want["best_f"] and np.array_equal(got["best_x"], want["best_x"])


@pytest.mark.parametrize("lo,hi", [(-100, 100), (-32768, 32767)])
@pytest.mark.parametrize("n,M", [(129, 2048), (300, 40), (300, 2049), (1000, 600), (1025, 300), (2049, 64), (2500, 700),
                                 (3072, 200), (400, 2048)])
def test_run_with_split_rows(ctx, n, M, lo, hi):
    Q = make_instance(n, 0.3, lo, hi, 7200 + n + M)
    kw = dict(M=M, H=5, lam_num=1, lam_den=2, G=2, run_seed=n)
    same(ctx.multistart(ctx.problem(Q), **kw), Q, kw)


@pytest.mark.parametrize("lo,hi", [(-100, 100), (-32768, 32767)])
def test_batch_of_neighbouring_lane_ranges(ctx, lo, hi):
    sizes = [(700, 300), (1500, 2049), (2500, 300), (3300, 200), (900, 2048)]
    Qs = [make_instance(n, 0.3, lo, hi, 7500 + n) for n, _ in sizes]
    kws = [dict(M=M, H=5, lam_num=1, lam_den=2, G=2, run_seed=n) for n, M in sizes]
    for r, Q, kw in zip(ctx.multistart_batched([ctx.problem(Q) for Q in Qs], kws), Qs, kws):
        same(r, Q, kw)
