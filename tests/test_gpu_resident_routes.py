"""Which route a call's iterations take: the resident loop by default, launches
when its workgroups do not all run (forced here by a launch that does not wait
for them), both over more than one resident launch and over a restart of the
barrier tags; results bitwise the same."""
import ctypes
import sys

import numpy as np
import pytest

from paper_2401_03256_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dfpr():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2401_03256_amd import dfpr as mod
    fn = mod.lib().dfpr_test_resident
    fn.argtypes = [ctypes.c_void_p, ctypes.c_int, ctypes.c_uint32, ctypes.c_void_p]
    return mod


def _resident(dfpr, g, refuse=0, tag=0):
    """Iterations in resident launches so far; sets the switch."""
    k = ctypes.c_int64()
    assert dfpr.lib().dfpr_test_resident(g.handle, refuse, tag, ctypes.byref(k)) == 0
    return k.value


def _say(msg):
    sys.stdout.write(f"\n[case] {msg}\n")
    sys.stdout.flush()


def _same(tag, a, b):
    assert np.array_equal(a[0], b[0]), f"{tag}: ranks differ by {np.abs(a[0] - b[0]).max()}"
    for f in ("iterations", "converged", "refine_sweeps", "final_linf", "affected_initial",
              "affected_final", "vertices_processed", "edges_processed"):
        assert getattr(a[1], f) == getattr(b[1], f), f"{tag}: {f}"


def _path(n):
    v = np.arange(n - 1, dtype=np.int32)
    return n, np.concatenate([v, v + 1]), np.concatenate([v + 1, v])


GRAPHS = {
    "one": lambda: (1, np.zeros(0, np.int32), np.zeros(0, np.int32)),
    "gnm10000": lambda: (10_000, *synth.gnm(10_000, 80_000, seed=2)),
    "rmat17": lambda: synth.rmat(17, 16, seed=4),
    "grid739": lambda: synth.grid2d(739, seed=12),
}


def _calls(dfpr, g, bt, R):
    """Every entry point that iterates, as (name, result)."""
    yield "static", g.static()
    yield "naive", g.naive_dynamic(R)
    for prec in (dfpr.FP64, dfpr.FP32_KAHAN):
        p = dfpr.params(frontier_tol=1e-13, precision=prec)
        yield f"df {prec}", g.dynamic_frontier(bt, R, p)
    yield "traversal", g.dynamic_traversal(bt, R)
    yield "cap", g.dynamic_frontier(bt, R, dfpr.params(max_iters=3))


@pytest.mark.parametrize("name", list(GRAPHS))
def test_routes_of_every_call(dfpr, name):
    _say(f"routes {name}")
    n, src, dst = GRAPHS[name]()
    n = int(n)
    if n > 1:
        bt = synth.random_batch(src, dst, n, 3, 9, seed=8)
    else:
        z = np.zeros(0, np.int32)
        bt = synth.Batch(z, z, z, z)
    kinds = {"default": (0, False), "refused": (1, False), "profiled": (0, True)}
    got = {}
    for kind, (refuse, profiled) in kinds.items():
        g = dfpr.Graph(n, src, dst)
        g.profile_reset(profiled)
        R, _ = g.static()
        g.apply_batch(bt)
        at = _resident(dfpr, g, refuse)
        got[kind] = []
        for what, (ranks, st) in _calls(dfpr, g, bt, R):
            now = _resident(dfpr, g, refuse)
            assert now - at == (st.iterations if kind == "default" else 0), (kind, what)
            at = now
            got[kind].append((what, (ranks, st), g.affected()))
    for kind in ("refused", "profiled"):
        for (what, a, fa), (_, b, fb) in zip(got["default"], got[kind]):
            _same(f"{kind} {what}", a, b)
            assert np.array_equal(fa, fb), (kind, what)


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("entries", [5, 1500])
def test_bad_id_when_the_resident_launch_does_not_start(dfpr, entries, precision):
    import torch
    _say(f"bad id, refused launch, {entries} entries, {precision}")
    n, src, dst = 9000, *synth.gnm(9000, 60_000, seed=3)
    b = synth.random_batch(src, dst, n, entries // 5, entries - entries // 5, seed=4)
    g = dfpr.Graph(n, src, dst)
    _resident(dfpr, g, refuse=1)
    p = dfpr.params(precision=dfpr.FP64 if precision == "fp64" else dfpr.FP32_KAHAN)
    before = g.ranks()
    b.ins_dst[-1] = n
    x = [torch.from_numpy(a.copy()).cuda() for a in (b.del_src, b.del_dst, b.ins_src, b.ins_dst)]
    for noalloc in (False, True):
        with pytest.raises(dfpr.DfprError) as e:
            g.dynamic_frontier_device(*x, p=p, noalloc=noalloc)
        assert e.value.code == dfpr.DFPR_E_RANGE
        assert np.array_equal(g.ranks(), before) and not g.affected().any()


@pytest.mark.parametrize("refuse", [(0, 0, 0), (1, 1, 1), (0, 1, 0)])
def test_serving_with_refused_launches(dfpr, refuse):
    _say(f"serving, refused {refuse}")
    graphs = [synth.rmat(12, 16, seed=5), (9000, *synth.gnm(9000, 60_000, seed=6)),
              synth.rmat(13, 16, seed=7)]
    srv = dfpr.Server(max_slots=3, hbm_budget_bytes=8 << 30)
    mine, alone, ids, reqs = [], [], [], []
    for i, (n, src, dst) in enumerate(graphs):
        p = dfpr.params(frontier_tol=1e-13, precision=dfpr.FP32_KAHAN if i == 2 else dfpr.FP64)
        g, h = dfpr.Graph(n, src, dst), dfpr.Graph(n, src, dst)
        R, _ = g.static()
        h.set_ranks(R)
        at = _resident(dfpr, g, refuse[i])
        mine.append((g, at))
        ids.append(srv.add_graph(g, p))
        bt = synth.random_batch(src, dst, n, 2, 9, seed=20 + i)
        for b in (bt, synth.Batch(bt.ins_src, bt.ins_dst, bt.del_src, bt.del_dst)):
            reqs.append((srv.submit(ids[i], 0.0, b), h, b, p))
        alone.append(h)
    srv.run()
    ran = [0, 0, 0]
    for rid, h, b, p in reqs:
        r = srv.result(rid)
        assert r["status"] == 0
        assert r["applied"] == h.apply_batch(b)
        _, st = h.dynamic_frontier(b, None, p)
        assert (r["iterations"], r["converged"], r["final_linf"], r["edges_processed"], r["affected"]) \
            == (st.iterations, st.converged, st.final_linf, st.edges_processed, st.affected_final)
        ran[r["graph_id"]] += st.iterations
    for i, ((g, at), h) in enumerate(zip(mine, alone)):
        assert np.array_equal(g.ranks(), h.ranks())
        here = _resident(dfpr, g) - at
        assert here == 0 if refuse[i] else here > 0
        if not any(refuse):
            assert here == ran[i]


@pytest.mark.parametrize("cap", [1023, 1024, 1025, 2100])
@pytest.mark.parametrize("graph", ["gnm", "path"])
def test_more_iterations_than_one_launch(dfpr, graph, cap):
    """1024 iterations are one resident launch; the path keeps its frontier on
    the class lists, the random graph on the full schedule."""
    _say(f"{graph}, cap {cap}")
    n, src, dst = _path(5000) if graph == "path" else (3000, *synth.gnm(3000, 20_000, seed=9))
    g, h = dfpr.Graph(n, src, dst), dfpr.Graph(n, src, dst)
    h.profile_reset(True)
    R, _ = g.static()
    bt = synth.random_batch(src, dst, n, 1, 2, seed=10)
    assert g.apply_batch(bt) == h.apply_batch(bt)
    at = _resident(dfpr, g)
    p = dict(tol=0.0, max_iters=cap)
    for what, call in (("static", lambda x: x.static(dfpr.params(**p))),
                       ("naive", lambda x: x.naive_dynamic(R, dfpr.params(**p))),
                       ("df", lambda x: x.dynamic_frontier(bt, R, dfpr.params(frontier_tol=1e-9, **p))),
                       ("df32", lambda x: x.dynamic_frontier(
                           bt, R, dfpr.params(frontier_tol=1e-9, precision=dfpr.FP32_KAHAN, **p)))):
        a, b = call(g), call(h)
        _same(f"{graph} {what} {cap}", a, b)
        now = _resident(dfpr, g)
        assert now - at == a[1].iterations
        at = now
        assert np.array_equal(g.affected(), h.affected())


def test_barrier_tags_start_over(dfpr):
    """A launch takes 1028 tags; the words are cleared before the tags that are
    left no longer hold two launches'."""
    _say("tags start over")
    n, src, dst = 10_000, *synth.gnm(10_000, 80_000, seed=2)
    g, h = dfpr.Graph(n, src, dst), dfpr.Graph(n, src, dst)
    want = h.static()
    for back in range(5):
        at = _resident(dfpr, g, tag=0xFFFFFFFF - 1028 * back - 7)
        for _ in range(3):
            got = g.static()
            _same(f"{back}", got, want)
        assert _resident(dfpr, g) - at == 3 * want[1].iterations


@pytest.mark.parametrize("name", ["gnm10000", "grid739"])
def test_a_launch_per_iteration_on_request(dfpr, name):
    _say(f"a launch per iteration, {name}")
    n, src, dst = GRAPHS[name]()
    bt = synth.random_batch(src, dst, n, 3, 9, seed=8)
    g, h = dfpr.Graph(n, src, dst), dfpr.Graph(n, src, dst)
    R, _ = g.static()
    assert g.apply_batch(bt) == h.apply_batch(bt)
    at = _resident(dfpr, g)
    for kw in (dict(), dict(precision=dfpr.FP32_KAHAN)):
        a = dfpr.params(frontier_tol=1e-13, loop=dfpr.LOOP_ITERATION, **kw)
        b = dfpr.params(frontier_tol=1e-13, **kw)
        for what, call in (("static", lambda x, p: x.static(p)),
                           ("naive", lambda x, p: x.naive_dynamic(R, p)),
                           ("df", lambda x, p: x.dynamic_frontier(bt, R, p)),
                           ("traversal", lambda x, p: x.dynamic_traversal(bt, R, p))):
            _same(what, call(g, a), call(h, b))
    assert _resident(dfpr, g) == at and _resident(dfpr, h) > 0
    srv = dfpr.Server(max_slots=2, hbm_budget_bytes=8 << 30)
    rid = srv.submit(srv.add_graph(g, a), 0.0, bt)
    srv.run()
    assert srv.result(rid)["status"] == 0 and _resident(dfpr, g) == at


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_profiled_small_frontiers(dfpr, precision):
    """DFPR_LOOP_DEVICE while profiled: small frontiers still iterate inside one
    launch, and the profile holds the other iterations."""
    _say(f"profiled small frontiers, {precision}")
    n, src, dst = synth.rmat(16, 16, seed=7)
    bt = synth.random_batch(src, dst, n, 0, 1, seed=8)
    p = dfpr.params(loop=dfpr.LOOP_DEVICE,
                    precision=dfpr.FP64 if precision == "fp64" else dfpr.FP32_KAHAN)
    g, h = dfpr.Graph(n, src, dst), dfpr.Graph(n, src, dst)
    R, _ = g.static()
    assert g.apply_batch(bt) == h.apply_batch(bt)
    h.profile_reset(True)
    a, b = g.dynamic_frontier(bt, R, p), h.dynamic_frontier(bt, R, p)
    _same("profiled", a, b)
    assert 0 < a[1].loop_iterations == b[1].loop_iterations < a[1].iterations
    pr = h.profile()
    assert pr.launches >= b[1].iterations - b[1].loop_iterations
    assert 0 < pr.rows < b[1].vertices_processed and 0 < pr.edges < b[1].edges_processed
