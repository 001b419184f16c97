"""Reachability searches with wide levels (no queues), narrow ones, and both:
the reachable set bit-exact and the ranks within 1e-9 of the oracle."""
import sys

import numpy as np
import pytest

import oracle
from paper_2401_03256_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dfpr():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2401_03256_amd import dfpr as mod
    mod.lib()
    return mod


def _chain(first, count):
    v = np.arange(first, first + count, dtype=np.int32)
    return v[:-1], v[1:]


def _core_and_tail(tail):
    """An R-MAT core whose vertex 0 starts a long path: wide levels, then one
    vertex a level; a second path that nothing reaches; a vertex with more
    out-edges than a workgroup's share, at the end of the first path."""
    n0, s, d = synth.rmat(12, 16, seed=2)
    a, b = _chain(n0, tail)
    c, e = _chain(n0 + tail, 50)
    n = n0 + tail + 50 + 5000
    fan = np.arange(n - 5000, n, dtype=np.int32)
    src = np.concatenate([s, [0], a, c, np.full(5000, n0 + tail - 1)]).astype(np.int32)
    dst = np.concatenate([d, [n0], b, e, fan]).astype(np.int32)
    return n, src, dst


GRAPHS = {
    "gnm40": lambda: (40, *synth.gnm(40, 300, seed=1)),
    "rmat13": lambda: synth.rmat(13, 16, seed=5),
    "tail3": lambda: _core_and_tail(3),
    "tail400": lambda: _core_and_tail(400),
    "grid64": lambda: synth.grid2d(64, seed=3),
}


@pytest.mark.parametrize("name", list(GRAPHS))
def test_search_matches_oracle(dfpr, name):
    sys.stdout.write(f"\n[case] traversal {name}\n")
    sys.stdout.flush()
    n, src, dst = GRAPHS[name]()
    g, o = dfpr.Graph(n, src, dst), oracle.OracleGraph(n, src, dst)
    R, _ = o.static()
    for k, (nd, ni) in enumerate([(0, 1), (1, 0), (3, 9)]):
        b = synth.random_batch(src, dst, n, nd, ni, seed=10 + k)
        if k == 0:
            b.ins_src[:] = src[0]       # from the core
        assert g.apply_batch(b) == tuple(o.apply_batch(b))
        want = o.mark_reachable(b)
        assert np.array_equal(g.mark_reachable(b), want)
        got, st = g.dynamic_traversal(b, R)
        assert st.affected_initial == st.affected_final == int(want.sum())
        assert np.abs(got - o.dynamic_traversal(b, R)[0]).max() <= 1e-9
        inv = synth.Batch(b.ins_src, b.ins_dst, b.del_src, b.del_dst)
        assert g.apply_batch(inv) == tuple(o.apply_batch(inv))


@pytest.mark.parametrize("n", [63, 65535, 65536, 65537])
def test_flags_of_small_and_larger_graphs(dfpr, n):
    """Flags come through pinned memory up to 65536 vertices, by a copy above."""
    sys.stdout.write(f"\n[case] flags {n}\n")
    sys.stdout.flush()
    src, dst = synth.gnm(n, 4 * n, seed=n)
    g, o = dfpr.Graph(n, src, dst), oracle.OracleGraph(n, src, dst)
    assert not g.affected().any()
    g.static()
    for seed in (1, 2):
        b = synth.random_batch(src, dst, n, 2, 3, seed=seed)
        o.apply_batch(b)
        g.apply_batch(b)
        assert np.array_equal(g.mark_affected(b), o.mark_initial(b))
        assert np.array_equal(g.mark_reachable(b), o.mark_reachable(b))
        g.dynamic_traversal(b)
        assert np.array_equal(g.affected(), o.mark_reachable(b))
        inv = synth.Batch(b.ins_src, b.ins_dst, b.del_src, b.del_dst)
        assert g.apply_batch(inv) == tuple(o.apply_batch(inv))
