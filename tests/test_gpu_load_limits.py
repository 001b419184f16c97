"""Loads at their limits: more input edges than a launch has threads, a device
with room for the graph but not for the load's scratch, and more vertices than
edge slots.  And a batch whose buffers the device has no room for."""
import ctypes
import os
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
    mod.lib()
    return mod


def _say(msg):
    sys.stdout.write(f"\n[case] {msg}\n")
    sys.stdout.flush()


def _same_graph(g, h):
    assert g.m == h.m
    for out in (True, False):
        for x, y in zip(g.csr(out), h.csr(out)):
            assert np.array_equal(x, y)
    (a, sa), (b, sb) = g.static(), h.static()
    assert sa.iterations == sb.iterations and np.array_equal(a, b)


class _Ballast:
    """Leaves about `mb` MB of the device free."""

    def __init__(self, mb):
        import torch
        torch.cuda.empty_cache()
        self.held = []
        for _ in range(200):
            free = torch.cuda.mem_get_info()[0] - (mb << 20)
            if free < 4 << 20:
                break
            self.held.append(torch.empty(min(free, 16 << 30), dtype=torch.uint8, device="cuda"))
        free = torch.cuda.mem_get_info()[0] >> 20
        _say(f"free now {free} MB")
        assert mb - 25 <= free <= mb + 7

    def drop(self):
        import torch
        self.held = []
        torch.cuda.empty_cache()


def test_load_beside_other_allocations(dfpr):
    _say("load with 225 MB of the device free")
    n, src, dst = synth.rmat(19, 16, seed=21)
    want = dfpr.Graph(n, src, dst)              # 145 MB, and 190 MB more while it loads
    ballast = _Ballast(225)
    try:
        got = dfpr.Graph(n, src, dst)
    finally:
        ballast.drop()
    _same_graph(got, want)


def test_batches_after_one_without_room(dfpr):
    """A batch that fails for want of memory leaves the graph able to take others."""
    _say("batch of 6,000,000 entries with 150 MB of the device free")
    n, src, dst = synth.rmat(14, 16, seed=22)
    g, h = dfpr.Graph(n, src, dst), dfpr.Graph(n, src, dst)
    seq = synth.batch_sequence(src, dst, n, [(40, 160), (300, 1200), (5, 20)], seed=23)
    assert g.apply_batch(seq[0]) == h.apply_batch(seq[0])
    z = np.zeros(0, np.int32)
    rng = np.random.default_rng(24)
    big = synth.Batch(z, z, *rng.integers(0, n, (2, 6_000_000), dtype=np.int32))
    ballast = _Ballast(150)
    try:
        with pytest.raises(dfpr.DfprError) as e:    # 32 bytes of keys an entry
            g.apply_batch(big)
        assert e.value.code == dfpr.DFPR_E_NOMEM
        for b in seq[1:]:
            assert g.apply_batch(b) == h.apply_batch(b)
    finally:
        ballast.drop()
    _same_graph(g, h)


def test_relayout_without_room(dfpr):
    """A batch whose rows need the index array laid out anew and find no memory for it
    leaves the rows' capacities with the old array; the same batch later completes it."""
    _say("450,000 insertions into 3000 rows with 100 MB of the device free")
    n, m = 40_000, 30_000_000                   # 135 MB of slots an orientation
    rng = np.random.default_rng(25)
    src, dst = rng.integers(0, n, (2, m), dtype=np.int32)
    g, h = dfpr.Graph(n, src, dst), dfpr.Graph(n, src, dst)
    z = np.zeros(0, np.int32)
    rows = np.repeat(np.arange(3000, dtype=np.int32), 150)
    add = synth.Batch(z, z, rng.integers(0, n, rows.size, dtype=np.int32), rows)
    loops = np.arange(rows.size, dtype=np.int32) % n
    assert g.apply_batch(synth.Batch(loops, loops, z, z)) == (0, 0)     # its buffers
    ballast = _Ballast(100)
    try:
        with pytest.raises(dfpr.DfprError) as e:
            g.apply_batch(add)
        assert e.value.code == dfpr.DFPR_E_NOMEM
        for k in range(0, rows.size, 150 * 300):        # one more of every 300th row
            g.apply_batch(synth.Batch(z, z, add.ins_src[k:k + 1], add.ins_dst[k:k + 1]))
    except dfpr.DfprError as e:
        assert e.code == dfpr.DFPR_E_NOMEM
    finally:
        ballast.drop()
    g.apply_batch(add)
    h.apply_batch(add)
    (a, _), (b, _) = g.static(), h.static()
    assert np.array_equal(a, b)


def test_more_vertices_than_slots(dfpr):
    _say("2^31 - 1 vertices")
    z = np.zeros(0, np.int32)
    with pytest.raises(dfpr.DfprError) as e:
        dfpr.Graph(2**31 - 1, z, z)
    assert e.value.code == dfpr.DFPR_E_LIMIT


class _Repeated:
    """`a` over and over as one array of host memory, whose pages are shared."""

    def __init__(self, a, times):
        libc = ctypes.CDLL(None, use_errno=True)
        libc.mmap.restype = ctypes.c_void_p
        libc.mmap.argtypes = [ctypes.c_void_p, ctypes.c_size_t, ctypes.c_int, ctypes.c_int, ctypes.c_int,
                              ctypes.c_long]
        libc.munmap.argtypes = [ctypes.c_void_p, ctypes.c_size_t]
        self.libc, self.bytes = libc, a.nbytes * times
        fd = os.memfd_create("edges")
        os.write(fd, a.tobytes())
        prot, shared, private, fixed, anon = 1, 1, 2, 16, 32
        self.at = libc.mmap(None, self.bytes, 0, private | anon, -1, 0)
        assert self.at not in (None, ctypes.c_void_p(-1).value)
        for k in range(times):
            p = libc.mmap(self.at + k * a.nbytes, a.nbytes, prot, shared | fixed, fd, 0)
            assert p == self.at + k * a.nbytes
        os.close(fd)

    def close(self):
        self.libc.munmap(self.at, self.bytes)


def test_more_input_edges_than_a_launch_has_threads(dfpr):
    """2^32 + 2^24 input edges, 2^24 distinct ones 257 times."""
    _say("2^32 + 2^24 input edges")
    n, part, times = 1 << 20, 1 << 24, 257
    rng = np.random.default_rng(3)
    src = rng.integers(0, n, part, dtype=np.int32)
    dst = rng.integers(0, n, part, dtype=np.int32)
    many = [_Repeated(x, times) for x in (src, dst)]
    h = ctypes.c_void_p()
    try:
        rc = dfpr.lib().dfpr_load_graph(n, part * times, many[0].at, many[1].at, ctypes.byref(h))
        assert rc == 0, dfpr.lib().dfpr_last_error().decode()
    finally:
        for x in many:
            x.close()
    got = dfpr.Graph.__new__(dfpr.Graph)
    got._h, got.n = h, n
    want = dfpr.Graph(n, src, dst)
    assert got.m == want.m
    for out in (True, False):
        for x, y in zip(got.csr(out), want.csr(out)):
            assert np.array_equal(x, y)
