"""Weights that are not finite are refused by nm_prune wherever they are: the selection kernel sees them."""
import numpy as np
import pytest

from paper_2507_17301_amd import binding as nm
from gpu_util import say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape,n,m,tile", [((5, 1, 1, 8), 2, 4, 16), ((40, 3, 3, 12), 1, 4, 16), ((33, 3, 3, 64), 2, 8, 32),
                                            ((24, 1, 1, 600), 300, 600, 8), ((4, 3, 3, 3), 1, 1, 1),
                                            ((410, 3, 3, 36), 1, 4, 16), ((110, 1, 1, 1200), 300, 600, 8), ((980, 3, 3, 15), 1, 1, 1)])
@pytest.mark.parametrize("value", [np.nan, -np.nan, np.inf, -np.inf])
def test_refused_wherever_it_is(shape, n, m, tile, value):
    w = np.random.default_rng(1).standard_normal(shape, dtype=np.float32)
    w.flat[0] = np.finfo(np.float32).max     # (a sum of these is finite in the kernel's fp64)
    w[1:, 0, 0, 0] = np.finfo(np.float32).max
    for at in (0, w.size // 2, w.size - 1):
        bad = w.copy()
        bad.flat[at] = value
        bad.flat[w.size - 1] = value         # the first of them is named
        say(f"{shape} {n}:{m} T={tile} {value} at {at}")
        with pytest.raises(nm.NMError, match=f"weight {at} is not finite") as e:
            nm.nm_prune(bad, n, m, tile)
        assert e.value.code == nm.NM_ERR_ARG
    assert nm.nm_packed_indices(nm.nm_prune(w, n, m, tile)).shape[-1] == n
