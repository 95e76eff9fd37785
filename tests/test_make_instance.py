"""make_instance against the recipe written out entry by entry: for every i <= j in row-major
order a uniform draw decides whether the entry is nonzero, then the nonzero values are
drawn in the same order and mirrored."""
import numpy as np
import pytest

from paper_1706_00037_amd.inputs import make_instance


@pytest.mark.parametrize("n", [1, 2, 63, 65, 200])
@pytest.mark.parametrize("density", [0.0, 0.1, 1.0])
@pytest.mark.parametrize("lo,hi", [(-100, 100), (-32768, 32767), (0, 5), (-3, 0)])
def test_recipe(n, density, lo, hi):
    rng = np.random.Generator(np.random.PCG64(n + 9))
    keep = rng.random(n * (n + 1) // 2) < density
    v = iter(rng.integers(lo, hi, size=int(keep.sum()), dtype=np.int64).tolist())
    want, k = np.zeros((n, n), np.int32), 0
    for i in range(n):
        for j in range(i, n):
            if keep[k]:
                x = next(v)
                want[i, j] = want[j, i] = x + (x >= 0)
            k += 1
    Q = make_instance(n, density, lo, hi, n + 9)
    assert Q.dtype == np.int32 and Q.flags.c_contiguous and np.array_equal(Q, want)
