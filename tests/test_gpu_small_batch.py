"""Batches around the sizes where the applier and the start of a call change
kernels (a wave, a workgroup of 1024 entries), with repeats, no-ops and rows of
every kind, against the oracle: CSRs and applied counts bit-exact, initial
marks equal, ranks within 1e-9."""
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


def _messy(n, src, dst, size, seed):
    """`size` entries: a third deletions of edges, some of them repeated or
    self-loops, and insertions of which some are present, repeated, or deleted
    by the same batch; vertex 0 is the source and the target of many."""
    rng = np.random.default_rng(seed)
    nd = size // 3
    pick = rng.integers(0, src.size, nd)
    ds, dd = src[pick].copy(), dst[pick].copy()
    ds[::7] = dd[::7]
    ni = size - nd
    is_, id_ = rng.integers(0, n, ni).astype(np.int32), rng.integers(0, n, ni).astype(np.int32)
    is_[::3] = 0
    id_[1::3] = 0
    k = min(nd, ni) // 4
    is_[:k], id_[:k] = ds[:k], dd[:k]
    if ni > 5:
        is_[-2:], id_[-2:] = is_[0], id_[0]
    return synth.Batch(ds, dd, is_, id_)


@pytest.mark.parametrize("size", [1, 2, 63, 64, 65, 127, 129, 1023, 1024, 1025, 2049])
def test_batch_sizes_match_oracle(dfpr, size):
    sys.stdout.write(f"\n[case] batch of {size}\n")
    sys.stdout.flush()
    n, src, dst = synth.rmat(13, 16, seed=9)
    g, o = dfpr.Graph(n, src, dst), oracle.OracleGraph(n, src, dst)
    R, _ = o.static()
    b = _messy(n, src, dst, size, seed=size)
    assert g.apply_batch(b) == tuple(o.apply_batch(b))
    for out in (True, False):
        for x, y in zip(g.csr(out), o.csr(out)):
            assert np.array_equal(x, y)
    assert np.array_equal(g.mark_affected(b), o.mark_initial(b))
    got, st = g.dynamic_frontier(b, R)
    want, _ = o.dynamic_frontier(b, R)
    assert st.converged and np.abs(got - want).max() <= 1e-9
    assert st.affected_initial == int(o.mark_initial(b).sum())


@pytest.mark.parametrize("size", [8, 1024, 1500])
def test_bad_id_in_device_batch_leaves_the_graph(dfpr, size):
    import torch
    n, (src, dst) = 2000, synth.gnm(2000, 12000, seed=3)
    g = dfpr.Graph(n, src, dst)
    before = g.csr(True)
    b = _messy(n, src, dst, size, seed=5)
    b.ins_dst[-1] = n
    t = [torch.from_numpy(x).cuda() for x in (b.del_src, b.del_dst, b.ins_src, b.ins_dst)]
    R0 = g.ranks()
    for call in (g.apply_batch_device, g.dynamic_frontier_device):
        with pytest.raises(dfpr.DfprError) as e:
            call(*t)
        assert e.value.code == dfpr.DFPR_E_RANGE
    assert all(np.array_equal(x, y) for x, y in zip(before, g.csr(True)))
    assert np.array_equal(R0, g.ranks())
    # the next good batch goes through
    good = synth.random_batch(src, dst, n, 3, 5, seed=6)
    assert g.apply_batch(good) == (3, 5)
