"""The row dot with its K range shared by several workgroups, where the number of parts
changes: one tile, parts that are empty for short column tiles, the last tile count that
is split and the first that is not, both coefficient widths.  Objectives are integers
and equal the oracle's exactly."""
import numpy as np
import pytest

import oracle
from paper_1706_00037_amd.inputs import make_instance, random_candidates

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lo,hi", [(-128, 127), (-32768, 32767)])
@pytest.mark.parametrize("n,M", [(1, 1), (128, 1), (129, 256), (255, 257), (1000, 255), (1024, 513), (2000, 4),
                                 (1024, 8192), (1024, 16128), (1024, 16384)])
def test_split_row_dot_matches_oracle(n, M, lo, hi):
    from paper_1706_00037_amd import ubqp
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    Q = make_instance(n, 0.6, lo, hi, 40 + n)
    X = random_candidates(M, n, 50 + n + M)
    ctx = ubqp.Context(0)
    f = torch.full((M,), -7, dtype=torch.int64, device="cuda")
    ctx.eval(ctx.problem(Q), torch.from_numpy(X.view(np.int64)).cuda(), f)
    torch.cuda.synchronize()
    assert np.array_equal(f.cpu().numpy(), oracle.eval_many(Q, X, threads=8))
