"""The sum of a row of more than 2048 in-edges rounds no more often than its
folds in pairs do, in the resident loop and in a launch per iteration."""
import sys

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dfpr():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2401_03256_amd import dfpr as mod
    mod.lib()
    return mod


@pytest.mark.parametrize("first", [0, 7, 15])
@pytest.mark.parametrize("leaves", [2048, 5000])
def test_folds_of_a_long_row(dfpr, leaves, first):
    """A star: one wave's fold of the hub's row is 1, the other 15 are half a
    unit in the last place of it, which added to it one by one are all lost."""
    sys.stdout.write(f"\n[case] {leaves} leaves, large fold {first}\n")
    sys.stdout.flush()
    n = leaves + 1
    leaf = np.arange(1, n, dtype=np.int32)
    g = dfpr.Graph(n, leaf, np.zeros(leaves, np.int32))
    # entry k of the hub's row is vertex k; a leaf has two out-edges, the hub one
    want = np.zeros(n)
    want[64 * np.arange(16) + 1] = 2.0 ** -53
    want[64 * first + 1] = 1.0
    prev = 2.0 * want
    base = 0.5 / n
    # |r - exact|: the folds 0.5 + 0.5 * s in units of 2^-53, s after four
    # roundings of half a unit, then one of the sum with the base rank
    exact = np.longdouble(base) + np.longdouble(0.5) * (np.longdouble(1.0) + 15 * np.longdouble(2.0) ** -53)
    assert np.finfo(np.longdouble).nmant >= 60
    for loop in (dfpr.LOOP_LAUNCHES, dfpr.LOOP_ITERATION):
        R, _ = g.naive_dynamic(prev, dfpr.params(alpha=0.5, max_iters=1, loop=loop))
        err = abs(float(np.longdouble(R[0]) - exact)) * 2.0 ** 53
        assert err <= 2.5, (loop, err)
