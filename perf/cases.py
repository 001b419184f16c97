"""Performance cases of the library: what a program has it do, over the range
of its sizes, methods, precisions and calling conventions.

A case is a dict of plain values.  ``kind`` is

- ``update``: a resident graph with previous ranks; one pass is a batch that
  arrives (applied to the graph, ranks updated by ``method``) and then expires
  (the inverse batch, ranks updated again), as in a sliding window over an
  edge stream.  The second update leaves the graph as it was, so every pass
  starts from the same graph; the first starts from the given ranks.
- ``cold``: a program's start.  Host edge arrays become a resident graph and
  its Static PageRank comes back.
- ``serve``: several resident graphs of uneven size behind a server; one pass
  serves a closed-loop set of update requests, half of them the inverses of
  the others.

Graphs are the synthetic families of this repository: uniform G(n, m), R-MAT
(0.57, 0.19, 0.19, 0.05) with edge factor 16, and bidirectional grids with 5%
diagonals.  The graph of an ``update`` or ``serve`` case is the long-lived
handle that a program keeps: it is the same for every seed and is built once,
while the seed draws the batches.  A ``cold`` graph is drawn from the seed.
"""
import math

import numpy as np
import torch

from paper_2401_03256_amd import dfpr, synth

DEV = "cuda" if torch.cuda.is_available() else "cpu"
ALPHA, TOL = 0.85, 1e-10


def listed():
    return [
        # the smallest call: one batch of 80 edges on a 10,000-vertex graph,
        # host arrays in and out, where launches and host looks are all there is
        dict(name="tiny_df_host", kind="update", graph="gnm", n=10_000, m=80_000, method="df",
             api="host", entries=80, ins=0.8, ftol=1e-13),
        # an interactive update of a small social graph: a dozen edges, device
        # arrays, previous ranks handed over
        dict(name="rmat16_df_dev", kind="update", graph="rmat", n=65_536, m=0, method="df",
             api="device", entries=11, ins=0.8, ftol=1e-13),
        # an odd-sized uniform graph and a deletion-only batch through the
        # entry point that allocates nothing, tau_f at its default
        dict(name="gnm_odd_df_noalloc", kind="update", graph="gnm", n=123_457, m=1_000_003,
             method="df", api="noalloc", entries=1001, ins=0.0, ftol=1e-15),
        # road-like graph, a localised batch: many iterations over a small
        # frontier
        dict(name="grid_local_df", kind="update", graph="grid", n=2048 * 2048, m=0, method="df",
             api="device", entries=213, ins=0.8, ftol=1e-13, local=True),
        # the same graph, a uniform batch with the adaptive frontier tolerance
        dict(name="grid_uniform_df", kind="update", graph="grid", n=2048 * 2048, m=0, method="df",
             api="device", entries=2137, ins=0.8, ftol=-1.0),
        # a bulk load of changes: 1e-3 of the edges of a mid-size graph, where
        # the batch applier and the marking count
        dict(name="rmat20_bulk_df", kind="update", graph="rmat", n=1 << 20, m=0, method="df",
             api="device", entries=16_786, ins=0.8, ftol=1e-13),
        # the headline workload: R-MAT scale 22, a batch of 1e-5 of the edges
        dict(name="rmat22_df", kind="update", graph="rmat", n=1 << 22, m=0, method="df",
             api="device", entries=694, ins=0.8, ftol=1e-13),
        # the precision form (FP32 contributions, Kahan row sums, FP64
        # refinement) on a graph whose size is no power of two
        dict(name="rmat_1m5_fp32", kind="update", graph="rmat", n=1_500_000, m=0, method="fp32",
             api="device", entries=2500, ins=0.8, ftol=1e-13),
        # full sweeps from the previous ranks, host ranks in and out
        dict(name="rmat18_naive_host", kind="update", graph="rmat", n=1 << 18, m=0,
             method="naive", api="host", entries=42, ins=0.8, ftol=1e-13),
        # the reachability comparator
        dict(name="rmat19_traversal", kind="update", graph="rmat", n=1 << 19, m=0,
             method="traversal", api="host", entries=86, ins=0.8, ftol=1e-13),
        # a program's start on a small graph: load, then Static
        dict(name="rmat16_cold", kind="cold", graph="rmat", n=65_536, m=0),
        # serving: six graphs of three sizes, one of each size in the FP32
        # form, 24 requests, eight slots
        dict(name="serve_6_graphs", kind="serve", n=1 << 18, graphs=6, pairs=2, frac=1e-5),
    ]


def draw(rng):
    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(["update"] * 8 + ["cold"] * 2 + ["serve"])
    if kind == "cold":
        graph = rng.choice(["rmat", "gnm"])
        n = log_int(3_000, 200_000)
        return dict(kind="cold", graph=graph, n=n, m=n * rng.randint(4, 16) if graph == "gnm" else 0)
    if kind == "serve":
        return dict(kind="serve", n=log_int(20_000, 1 << 18), graphs=rng.randint(2, 8),
                    pairs=rng.randint(1, 3), frac=10.0 ** rng.uniform(-7, -3))
    graph = rng.choice(["gnm", "rmat", "rmat", "grid"])
    method = rng.choice(["df"] * 5 + ["fp32", "naive", "traversal"])
    if graph == "grid":
        # the traversal of a grid is thousands of levels: R-MAT and G(n, m) only
        method = "df" if method == "traversal" else method
        side = log_int(60, 2048)
        n, m, edges = side * side, 0, 5 * side * side
    elif graph == "rmat":
        n, m = log_int(4_000, 1 << 21), 0
        edges = 16 * n
    else:
        n = log_int(4_000, 1 << 20)
        m = n * rng.randint(4, 16) + rng.randint(0, 999)
        edges = m + n
    entries = max(1, int(edges * 10.0 ** rng.uniform(-7, -3)))
    api = rng.choice(["device", "device", "noalloc", "host"])
    if method in ("naive", "traversal"):
        api = "host"
    c = dict(kind="update", graph=graph, n=n, m=m, method=method, api=api, entries=entries,
             ins=rng.choice([0.8, 0.8, 1.0, 0.0, 0.5]),
             ftol=rng.choice([1e-13, 1e-13, 1e-15, -1.0]))
    if graph == "grid":
        c["local"] = rng.random() < 0.5
    return c


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------


def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed) & 0x7FFFFFFFFFFF)
    return g


def _edges(graph, n, m, seed):
    """Sorted int64 keys u * n + v of a simple digraph (no self-loops)."""
    g = _gen(seed)
    if graph == "grid":
        side = math.isqrt(n)
        ids = torch.arange(n, device=DEV).view(side, side)
        pairs = [(ids[:, :-1], ids[:, 1:]), (ids[:-1, :], ids[1:, :])]
        pick = torch.randperm(n, generator=g, device=DEV)[: round(0.05 * n)]
        r, c = pick // side, pick % side
        dr = torch.randint(0, 2, (pick.numel(),), generator=g, device=DEV) * 2 - 1
        dc = torch.randint(0, 2, (pick.numel(),), generator=g, device=DEV) * 2 - 1
        dr = torch.where((r + dr < 0) | (r + dr >= side), -dr, dr)
        dc = torch.where((c + dc < 0) | (c + dc >= side), -dc, dc)
        pairs.append((pick, (r + dr) * side + (c + dc)))
        a = torch.cat([p[0].reshape(-1) for p in pairs])
        b = torch.cat([p[1].reshape(-1) for p in pairs])
        u, v = torch.cat([a, b]), torch.cat([b, a])
    elif graph == "rmat":
        draws = 16 * n
        u = torch.zeros(draws, dtype=torch.int64, device=DEV)
        v = torch.zeros(draws, dtype=torch.int64, device=DEV)
        for level in range(max(1, (n - 1).bit_length())):
            x = torch.rand(draws, generator=g, device=DEV)
            u += (x >= 0.76).to(torch.int64) << level
            v += (((x >= 0.57) & (x < 0.76)) | (x >= 0.95)).to(torch.int64) << level
        u, v = u % n, v % n
    else:
        u = torch.randint(0, n, (m,), generator=g, device=DEV)
        v = torch.randint(0, n, (m,), generator=g, device=DEV)
    keys = (u * n + v)[u != v]
    return torch.unique(keys)


def _member(keys, x):
    pos = torch.searchsorted(keys, x).clamp_(max=keys.numel() - 1)
    return keys[pos] == x


def _distinct(x):
    """`x` without repeats, in the order of the first ones."""
    x = x.cpu().numpy()
    _, first = np.unique(x, return_index=True)
    return x[np.sort(first)]


def _batch(case, n, keys, entries, ins, seed):
    """One batch of which every entry changes the graph: deletions of edges,
    insertions of pairs that are none, uniform or inside one window of a grid."""
    g = _gen(seed)
    n_ins = int(round(ins * entries))
    n_del = min(entries - n_ins, keys.numel() // 2)
    if case.get("local"):
        side = math.isqrt(n)
        w = min(side, max(4, math.isqrt(4 * entries) + 1))
        r0, c0 = (int(x) for x in torch.randint(0, side - w + 1, (2,), generator=g, device=DEV))

        def cells(count):
            rc = torch.randint(0, w, (2, count), generator=g, device=DEV)
            return rc[0], rc[1]

        def keyed(r, c, dr, dc):
            ok = (r + dr >= 0) & (r + dr < w) & (c + dc >= 0) & (c + dc < w) & ((dr != 0) | (dc != 0))
            k = ((r0 + r) * side + c0 + c) * n + (r0 + r + dr) * side + c0 + c + dc
            return k[ok]

        r, c = cells(8 * n_del + 64)
        way = torch.randint(0, 4, (r.numel(),), generator=g, device=DEV)
        dels = keyed(r, c, (way == 0).long() - (way == 1).long(), (way == 2).long() - (way == 3).long())
        r, c = cells(8 * n_ins + 64)
        hop = torch.randint(-2, 3, (2, r.numel()), generator=g, device=DEV)
        news = keyed(r, c, hop[0], hop[1])
        dels = dels[_member(keys, dels)]
    else:
        dels = keys[torch.randint(0, keys.numel(), (2 * n_del + 16,), generator=g, device=DEV)]
        uv = torch.randint(0, n, (2, 2 * n_ins + 16), generator=g, device=DEV)
        news = (uv[0] * n + uv[1])[uv[0] != uv[1]]
    d = _distinct(dels)[:n_del]
    i = _distinct(news[~_member(keys, news)])[:n_ins]
    return synth.Batch((d // n).astype(np.int32), (d % n).astype(np.int32),
                       (i // n).astype(np.int32), (i % n).astype(np.int32))


def _inverse(b):
    return synth.Batch(b.ins_src, b.ins_dst, b.del_src, b.del_dst)


def _on_device(b):
    return [torch.from_numpy(x).to(DEV) for x in (b.del_src, b.del_dst, b.ins_src, b.ins_dst)]


# ---------------------------------------------------------------------------
# the method in plain torch, 64 bits
# ---------------------------------------------------------------------------


class _Plain:
    """A graph given by sorted edge keys, self-loops added: Eq. 1 as sums over
    the in-edges in two levels of segments, so that a run repeats bit by bit."""

    def __init__(self, n, keys):
        self.n = n
        loops = torch.arange(n, device=DEV)
        u, v = torch.cat([keys // n, loops]), torch.cat([keys % n, loops])
        order = torch.argsort(v * n + u)
        self.src, self.dst = u[order], v[order]
        cnt = torch.bincount(self.dst, minlength=n)
        self.out = torch.bincount(self.src, minlength=n).double()
        end = torch.cumsum(cnt, 0)
        parts = (cnt + 63) // 64
        pend = torch.cumsum(parts, 0)
        zero = torch.zeros(1, dtype=torch.int64, device=DEV)
        row = torch.repeat_interleave(loops, parts)
        nth = torch.arange(row.numel(), device=DEV) - (pend - parts)[row]
        self.fine = torch.cat([(end - cnt)[row] + 64 * nth, end[-1:]])
        self.coarse = torch.cat([zero, pend])

    def pull(self, c):
        x = torch.segment_reduce(c[self.src], "sum", offsets=self.fine, unsafe=True)
        return torch.segment_reduce(x, "sum", offsets=self.coarse, unsafe=True)

    def solve(self, r, marks=None, ftol=math.inf, tol=TOL):
        """Iterate from ranks `r`: every vertex, or those of `marks`, which
        grow by the out-neighbours of a vertex that moves by more than `ftol`."""
        marks = None if marks is None else marks.clone()
        seen = torch.zeros(self.n, dtype=torch.bool, device=DEV)
        for _ in range(500):
            new = (1.0 - ALPHA) / self.n + ALPHA * self.pull(r / self.out)
            if marks is not None:
                new = torch.where(marks, new, r)
            moved = (new - r).abs()
            r = new
            if marks is not None and ftol < math.inf:
                grow = (moved > ftol) & ~seen
                seen |= grow
                marks[self.dst[grow[self.src]]] = True
            if float(moved.max()) <= tol:
                break
        return r

    def first_marks(self, b):
        """(G before and after).out of every batch source."""
        s = torch.zeros(self.n, dtype=torch.bool, device=DEV)
        s[torch.from_numpy(np.concatenate([b.del_src, b.ins_src])).to(DEV).long()] = True
        m = torch.zeros_like(s)
        m[self.dst[s[self.src]]] = True
        m[torch.from_numpy(b.del_dst).to(DEV).long()] = True
        return m

    def reachable(self, b):
        m = torch.zeros(self.n, dtype=torch.bool, device=DEV)
        m[torch.from_numpy(np.concatenate([b.del_src, b.ins_src, b.del_dst])).to(DEV).long()] = True
        while True:
            grown = m.clone()
            grown[self.dst[m[self.src]]] = True
            if bool((grown == m).all()):
                return m
            m = grown

    def update(self, b, r, method, ftol):
        if method == "naive":
            return self.solve(r)
        if method == "traversal":
            return self.solve(r, self.reachable(b))
        m = self.first_marks(b)
        if ftol < 0.0:      # chosen from the mean out-degree of the first frontier
            marked, reach = int(m.sum()), int(self.out[m].sum())
            k = 5 if not marked else next((j for j in range(1, 5) if reach <= (4 << j) * marked), 5)
            ftol = TOL / 10.0 ** k
        return self.solve(r, m, ftol)


def _changed(keys, b, n):
    """Edge keys after the batch."""
    d = torch.from_numpy(b.del_src.astype(np.int64) * n + b.del_dst).to(DEV)
    i = torch.from_numpy(b.ins_src.astype(np.int64) * n + b.ins_dst).to(DEV)
    if d.numel():
        keys = keys[~_member(torch.sort(d)[0], keys)]
    return torch.sort(torch.cat([keys, i]))[0]


# ---------------------------------------------------------------------------
# resident graphs
# ---------------------------------------------------------------------------

_resident = {}      # the graphs of one case at a time


def _graph_specs(case):
    if case["kind"] == "serve":
        # sizes n, n/4 and n/16, uneven and odd
        return [("rmat", max(1000, (case["n"] >> (2 * (i % 3))) - 7 * i), 0)
                for i in range(case["graphs"])]
    return [(case["graph"], case["n"], case["m"])]


def _base(case, handles=True):
    """[(n, edge keys, previous ranks, resident graph)] of a case."""
    specs = _graph_specs(case)
    at = repr(specs)
    if at not in _resident:
        _resident.clear()
        _resident[at] = []
        for i, (graph, n, m) in enumerate(specs):
            n = math.isqrt(n) ** 2 if graph == "grid" else n
            keys = _edges(graph, n, m, 1 + i)
            plain = _Plain(n, keys)
            r0 = plain.solve(torch.full((n,), 1.0 / n, dtype=torch.float64, device=DEV))
            del plain
            _resident[at].append([n, keys, r0, None])
    if handles:
        for b in _resident[at]:
            if b[3] is None:
                n, keys = b[0], b[1]
                b[3] = dfpr.Graph(n, (keys // n).int().cpu().numpy(), (keys % n).int().cpu().numpy())
    return _resident[at]


def _serve_batches(case, base, seed):
    """Per graph: `pairs` batches, each followed by its inverse."""
    got = []
    for i, (n, keys, _, _) in enumerate(base):
        entries = max(1, round(case["frac"] * (keys.numel() + n)))
        for k in range(case["pairs"]):
            b = _batch(case, n, keys, entries, 0.8, seed * 1009 + 31 * i + k)
            got += [(i, b), (i, _inverse(b))]
    # requests of the graphs interleave, those of one graph stay in order
    return [x for k in range(2 * case["pairs"]) for x in got[k::2 * case["pairs"]]]


def _precision(case, i):
    return dfpr.FP32_KAHAN if i >= 3 else dfpr.FP64


# ---------------------------------------------------------------------------
# the measured path
# ---------------------------------------------------------------------------


def prepare(case, seed):
    if case["kind"] == "cold":
        keys = _edges(case["graph"], case["n"], case["m"], 7919 * seed + 3)
        n = case["n"]
        return dict(kind="cold", n=n, src=(keys // n).int().cpu().numpy(),
                    dst=(keys % n).int().cpu().numpy(), p=dfpr.params())
    base = _base(case)
    if case["kind"] == "serve":
        server = dfpr.Server(max_slots=8, hbm_budget_bytes=32 << 30)
        ids = [server.add_graph(b[3], dfpr.params(frontier_tol=1e-13, precision=_precision(case, i)))
               for i, b in enumerate(base)]
        return dict(kind="serve", server=server, ids=ids, graphs=[b[3] for b in base],
                    ranks=[b[2] for b in base], out=[torch.empty_like(b[2]) for b in base],
                    requests=_serve_batches(case, base, seed))
    n, keys, r0, g = base[0]
    b = _batch(case, n, keys, case["entries"], case["ins"], seed)
    precision = dfpr.FP32_KAHAN if case["method"] == "fp32" else dfpr.FP64
    s = dict(kind="update", api=case["api"], method=case["method"], g=g,
             p=dfpr.params(frontier_tol=case["ftol"], precision=precision))
    if case["api"] == "host":
        s.update(arrive=b, expire=_inverse(b), ranks=r0.cpu().numpy())
    else:
        s.update(arrive=_on_device(b), expire=_on_device(_inverse(b)), ranks=r0,
                 out=[torch.empty_like(r0), torch.empty_like(r0)])
    return s


def _run_update(s):
    g, p = s["g"], s["p"]
    applied, ranks = [], []
    for k, b in enumerate((s["arrive"], s["expire"])):
        prev = s["ranks"] if k == 0 else None       # then the resident ranks
        if s["api"] == "host":
            applied += g.apply_batch(b)
            call = {"naive": lambda: g.naive_dynamic(prev, p),
                    "traversal": lambda: g.dynamic_traversal(b, prev, p)}.get(
                        s["method"], lambda: g.dynamic_frontier(b, prev, p))
            ranks.append(call()[0])
        else:
            applied += g.apply_batch_device(*b)
            g.dynamic_frontier_device(*b, prev=prev, out=s["out"][k], p=p,
                                      noalloc=s["api"] == "noalloc")
            ranks.append(s["out"][k])
    return dict(applied=applied, ranks=ranks)


def _run_cold(s):
    g = dfpr.Graph(s["n"], s["src"], s["dst"])
    ranks, _ = g.static(s["p"])
    m = g.m
    g.close()
    return dict(edges=m, ranks=ranks)


def _run_serve(s):
    for g, r in zip(s["graphs"], s["ranks"]):
        rc = dfpr.lib().dfpr_set_ranks(g.handle, r.data_ptr(), 1)
        if rc:
            raise dfpr.DfprError(rc, "dfpr_set_ranks")
    reqs = [s["server"].submit(s["ids"][i], 0.0, b) for i, b in s["requests"]]
    s["server"].run()
    done = [s["server"].result(r) for r in reqs]
    for g, out in zip(s["graphs"], s["out"]):
        g.ranks_device(out)
    return dict(status=np.array([d["status"] for d in done]),
                applied=np.array([d["applied"] for d in done]), ranks=s["out"])


def run(state):
    return {"update": _run_update, "cold": _run_cold, "serve": _run_serve}[state["kind"]](state)


# ---------------------------------------------------------------------------
# what a pass cannot do without, and its exact results
# ---------------------------------------------------------------------------


def work(case):
    """Bytes and operations of one pass.  A full iteration reads every in-edge
    (4 B) and contribution (8 B; 4 B in FP32) once and per row its start,
    length, rank and out-degree and writes two values (44 B); an update takes
    about 30 of them on R-MAT and G(n, m).  On a grid the frontier holds about
    100 vertices per batch edge (20 localised) over about 12 iterations."""
    def sweep(n, m, fp32=False):
        return 4 * m + (40 if fp32 else 52) * n, 2 * m + 3 * n

    def edges(graph, n, m):
        return (5 if graph == "grid" else 16) * n if graph != "gnm" else m + n

    if case["kind"] == "cold":
        m = edges(case["graph"], case["n"], case["m"])
        b, f = sweep(case["n"], m)
        return dict(bytes=8 * m + 8 * case["n"] + 60 * b, flops=60 * f)
    if case["kind"] == "serve":
        parts = [sweep(n, edges(graph, n, m), _precision(case, i) == dfpr.FP32_KAHAN)
                 for i, (graph, n, m) in enumerate(_graph_specs(case))]
        k = 2 * case["pairs"] * 25
        return dict(bytes=k * sum(p[0] for p in parts), flops=k * sum(p[1] for p in parts))
    n, m = case["n"], edges(case["graph"], case["n"], case["m"])
    ends = 2 * (16 * case["entries"] + 16 * n)      # batches in, ranks in and out
    if case["graph"] == "grid" and case["method"] in ("df", "fp32"):
        rows = min(n, case["entries"] * (20 if case.get("local") else 100))
        return dict(bytes=ends + 2 * 12 * rows * (5 * 12 + 44), flops=2 * 12 * 13 * rows)
    b, f = sweep(n, m, case["method"] == "fp32")
    its = 2 * (12 if case["graph"] == "grid" else 30)
    return dict(bytes=ends + its * b, flops=its * f)


def exact(case, seed):
    """The same updates in plain torch, 64 bits.  The FP32 form's exact values
    are those of the FP64 method it ends in."""
    if case["kind"] == "cold":
        n = case["n"]
        keys = _edges(case["graph"], n, case["m"], 7919 * seed + 3)
        r = _Plain(n, keys).solve(torch.full((n,), 1.0 / n, dtype=torch.float64, device=DEV))
        return dict(edges=None, ranks=r)
    base = _base(case, handles=False)
    if case["kind"] == "serve":
        keys = [b[1] for b in base]
        ranks = [b[2] for b in base]
        for i, b in _serve_batches(case, base, seed):
            n = base[i][0]
            keys[i] = _changed(keys[i], b, n)
            ranks[i] = _Plain(n, keys[i]).update(b, ranks[i], "df", 1e-13)
        return dict(status=None, applied=None, ranks=ranks)
    n, keys, r, _ = base[0]
    b = _batch(case, n, keys, case["entries"], case["ins"], seed)
    ranks = []
    for x in (b, _inverse(b)):
        keys = _changed(keys, x, n)
        r = _Plain(n, keys).update(x, r, case["method"], case["ftol"])
        ranks.append(r)
    return dict(applied=None, ranks=ranks)
