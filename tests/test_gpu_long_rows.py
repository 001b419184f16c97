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


def test_long_rows_above_the_resident_line(dfpr):
    """A graph of more than 40M in-edges, whose calls iterate in the resident
    loop while on the class lists and in launches after: the long row of a
    vertex that both process has the same parts in them."""
    from paper_2401_03256_amd import synth
    sys.stdout.write("\n[case] 41M edges and a hub of 9000\n")
    sys.stdout.flush()
    n, hub = 2_500_000, 9000
    rng = np.random.default_rng(1)
    src = np.concatenate([rng.integers(0, n, 41_000_000, dtype=np.int32), np.arange(1, hub + 1, dtype=np.int32)])
    dst = np.concatenate([rng.integers(0, n, 41_000_000, dtype=np.int32), np.zeros(hub, np.int32)])
    g = dfpr.Graph(n, src, dst)
    assert g.m > 40_000_000
    R, st = g.static()
    want, _ = g.static(dfpr.params(loop=dfpr.LOOP_ITERATION))
    assert st.converged and np.array_equal(R, want)
    z = np.zeros(0, np.int32)
    b = synth.Batch(z, z, np.array([5, 77], np.int32), np.array([n - 1, 0], np.int32))
    g.apply_batch(b)
    a, sa = g.dynamic_frontier(b, R, dfpr.params(frontier_tol=1e-13))
    marks = g.affected()
    c, sc = g.dynamic_frontier(b, R, dfpr.params(frontier_tol=1e-13, loop=dfpr.LOOP_ITERATION))
    assert marks[0] and sa.iterations == sc.iterations and np.array_equal(a, c)
    assert np.array_equal(marks, g.affected())


def test_long_rows_of_a_graph_that_shrank(dfpr):
    """Loaded above the line and below it after a batch: the parts of its rows
    stay, and whole calls stay with launches."""
    from paper_2401_03256_amd import synth
    n, hub = 2_500_000, 9000
    rng = np.random.default_rng(2)
    src = np.concatenate([rng.integers(0, n, 37_900_000, dtype=np.int32), np.arange(1, hub + 1, dtype=np.int32)])
    dst = np.concatenate([rng.integers(0, n, 37_900_000, dtype=np.int32), np.zeros(hub, np.int32)])
    g = dfpr.Graph(n, src, dst)
    drop = g.m - 40_000_000 + 1000
    sys.stdout.write(f"\n[case] {g.m} edges, {drop} deleted\n")
    sys.stdout.flush()
    assert 1000 < drop < 2_000_000
    e = np.unique(src[:2 * drop].astype(np.int64) * n + dst[:2 * drop])
    e = e[e // n != e % n][:drop]
    z = np.zeros(0, np.int32)
    assert g.apply_batch(synth.Batch((e // n).astype(np.int32), (e % n).astype(np.int32), z, z)) == (drop, 0)
    assert g.m < 40_000_000
    R, st = g.static()
    want, _ = g.static(dfpr.params(loop=dfpr.LOOP_ITERATION))
    assert st.converged and np.array_equal(R, want)
    b = synth.Batch(z, z, np.array([5, 77], np.int32), np.array([n - 1, 0], np.int32))
    g.apply_batch(b)
    a, sa = g.dynamic_frontier(b, R, dfpr.params(frontier_tol=1e-13))
    c, sc = g.dynamic_frontier(b, R, dfpr.params(frontier_tol=1e-13, loop=dfpr.LOOP_ITERATION))
    assert sa.iterations == sc.iterations and np.array_equal(a, c)
