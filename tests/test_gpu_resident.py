"""The resident loop (many iterations in one launch) against a launch per
iteration, bitwise, and against the oracle.  Profiled calls always take a
launch per iteration, so switching the profile on selects the comparison."""
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


def _star(leaves):
    v = np.arange(1, leaves + 1, dtype=np.int32)
    z = np.zeros(leaves, np.int32)
    return leaves + 1, np.concatenate([v, z]), np.concatenate([z, v])


GRAPHS = {
    "one": lambda: (1, np.zeros(0, np.int32), np.zeros(0, np.int32)),
    "gnm63": lambda: (63, *synth.gnm(63, 300, seed=1)),
    "gnm10000": lambda: (10_000, *synth.gnm(10_000, 80_000, seed=2)),
    # one workgroup-wide row among rows of one in-edge
    "star5000": lambda: _star(5000),
    # long rows in every class; n no multiple of a wave
    "rmat12": lambda: synth.rmat(12, 16, seed=3),
    "rmat17": lambda: synth.rmat(17, 16, seed=4),
    "grid301": lambda: synth.grid2d(301, seed=5),
}


def _same(tag, a, b):
    (Ra, sa), (Rb, sb) = a, b
    assert np.array_equal(Ra, Rb), f"{tag}: ranks differ by {np.abs(Ra - Rb).max()}"
    for f in ("iterations", "converged", "refine_sweeps", "final_linf", "affected_initial",
              "affected_final", "vertices_processed", "edges_processed"):
        assert getattr(sa, f) == getattr(sb, f), f"{tag}: {f}"


@pytest.mark.parametrize("name", list(GRAPHS))
def test_resident_loop_bitwise_equal_to_launches(dfpr, name):
    sys.stdout.write(f"\n[case] resident loop {name}\n")
    sys.stdout.flush()
    n, src, dst = GRAPHS[name]()
    g, h = dfpr.Graph(n, src, dst), dfpr.Graph(n, src, dst)
    h.profile_reset(True)                       # a launch per iteration
    o = oracle.OracleGraph(n, src, dst)
    a, b = g.static(), h.static()
    _same("static", a, b)
    R, _ = o.static()
    assert np.abs(a[0] - R).max() <= 1e-9
    for cap in (0, 1, 2, 7):
        p = dfpr.params(max_iters=cap)
        _same(f"cap {cap}", g.naive_dynamic(R, p), h.naive_dynamic(R, p))
    if n < 60:
        return
    for k, (nd, ni) in enumerate([(1, 4), (0, 1), (3, 0), (17, 40)]):
        nd = min(nd, src.size // 8)
        bt = synth.random_batch(src, dst, n, nd, ni, seed=30 + k)
        assert g.apply_batch(bt) == h.apply_batch(bt)
        for prec in (dfpr.FP64, dfpr.FP32_KAHAN):
            for ftol in (1e-13, -1.0):
                p = dfpr.params(frontier_tol=ftol, precision=prec)
                _same(f"df {k} {prec} {ftol}", g.dynamic_frontier(bt, R, p),
                      h.dynamic_frontier(bt, R, p))
                assert np.array_equal(g.affected(), h.affected())
        _same(f"traversal {k}", g.dynamic_traversal(bt, R), h.dynamic_traversal(bt, R))
        for cap in (1, 3):
            p = dfpr.params(max_iters=cap)
            _same(f"df {k} cap {cap}", g.dynamic_frontier(bt, R, p), h.dynamic_frontier(bt, R, p))
        inv = synth.Batch(bt.ins_src, bt.ins_dst, bt.del_src, bt.del_dst)
        assert g.apply_batch(inv) == h.apply_batch(inv)
    assert h.profile().launches > 0 and g.profile().launches == 0


@pytest.mark.parametrize("changes", [60, 600, 6000])
def test_first_frontiers_around_the_list_limits(dfpr, changes):
    """Out-edges of the first frontier below 1/64 of the vertices, between 1/64
    and 1/8 and above: appended, appended and marked in place."""
    n, src, dst = synth.grid2d(500, seed=9)
    g, h = dfpr.Graph(n, src, dst), dfpr.Graph(n, src, dst)
    h.profile_reset(True)
    R, _ = g.static()
    bt = synth.random_batch(src, dst, n, changes // 4, changes, seed=50)
    assert g.apply_batch(bt) == h.apply_batch(bt)
    for prec in (dfpr.FP64, dfpr.FP32_KAHAN):
        p = dfpr.params(frontier_tol=1e-9, precision=prec)
        _same(f"{changes} {prec}", g.dynamic_frontier(bt, R, p), h.dynamic_frontier(bt, R, p))
        assert np.array_equal(g.affected(), h.affected())
    o = oracle.OracleGraph(n, src, dst)
    o.apply_batch(bt)
    Ro, _ = o.static()
    Rd, _ = g.dynamic_frontier(bt, R)
    # both within tol 1e-10 of the fixed point, damping 0.85: 2 tol / (1 - 0.85)
    assert np.abs(Rd - Ro).max() <= 2e-9


@pytest.mark.parametrize("rows", [255, 1023, 1500])
def test_fp32_block_rows_over_the_workgroups(dfpr, rows):
    """More rows of many in-edges than workgroups, and than one round of them."""
    n = 20_000
    rng = np.random.default_rng(rows)
    deg = np.linspace(6000, 600, rows).astype(np.int64)
    dst = np.repeat(np.arange(rows, dtype=np.int32), deg)
    src = rng.integers(0, n, dst.size).astype(np.int32)
    back = np.arange(n, dtype=np.int32)
    src = np.concatenate([src, (back % rows).astype(np.int32)])
    dst = np.concatenate([dst, back])
    e = np.unique(src.astype(np.int64) * n + dst)
    e = e[e // n != e % n]
    src, dst = (e // n).astype(np.int32), (e % n).astype(np.int32)
    g, h = dfpr.Graph(n, src, dst), dfpr.Graph(n, src, dst)
    h.profile_reset(True)
    R = np.full(n, 1.0 / n)
    bt = synth.random_batch(src, dst, n, 10, 200, seed=60)
    assert g.apply_batch(bt) == h.apply_batch(bt)
    p = dfpr.params(precision=dfpr.FP32_KAHAN)
    _same(f"{rows}", g.dynamic_frontier(bt, R, p), h.dynamic_frontier(bt, R, p))


@pytest.mark.parametrize("name", ["rmat18", "grid739"])
def test_pairs_of_rows_bitwise_equal_to_launches(dfpr, name):
    """Full schedules of more than four wave units a wave: two rows a lane
    group, with odd rows left over and with self-loop rows."""
    n, src, dst = {"rmat18": lambda: synth.rmat(18, 16, seed=11),
                   "grid739": lambda: synth.grid2d(739, seed=12)}[name]()
    n = int(n)
    g, h = dfpr.Graph(n, src, dst), dfpr.Graph(n, src, dst)
    h.profile_reset(True)
    a, b = g.static(), h.static()
    _same("static", a, b)
    R = a[0]
    bt = synth.random_batch(src, dst, n, 500, n // 40, seed=70)
    assert g.apply_batch(bt) == h.apply_batch(bt)
    _same("df", g.dynamic_frontier(bt, R), h.dynamic_frontier(bt, R))
    assert np.array_equal(g.affected(), h.affected())
    _same("traversal", g.dynamic_traversal(bt, R), h.dynamic_traversal(bt, R))
    _same("naive", g.naive_dynamic(R), h.naive_dynamic(R))


def test_resident_loop_calls_from_two_threads(dfpr):
    """Two graphs updated at once: each call's workgroups may find the other's
    running; results stay those of calls one at a time."""
    import threading
    n, src, dst = synth.rmat(14, 16, seed=7)
    batches = [synth.random_batch(src, dst, n, 4, 16, seed=40 + k) for k in range(2)]
    want = []
    for b in batches:
        g = dfpr.Graph(n, src, dst)
        R0, _ = g.static()
        g.apply_batch(b)
        want.append((R0, g.dynamic_frontier(b, R0)[0]))
    graphs = [dfpr.Graph(n, src, dst) for _ in batches]
    bad = []

    def work(k):
        try:
            g, b = graphs[k], batches[k]
            g.apply_batch(b)
            for _ in range(20):
                if not np.array_equal(g.dynamic_frontier(b, want[k][0])[0], want[k][1]):
                    bad.append(k)
        except Exception as e:      # reported below, in the main thread
            bad.append(e)

    ts = [threading.Thread(target=work, args=(k,)) for k in range(2)]
    [t.start() for t in ts]
    [t.join() for t in ts]
    assert not bad
