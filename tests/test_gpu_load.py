"""Graphs built on the device: sizes around the tiles of the sort, repeated
edges, self-loops and unsorted input, against the oracle's CSRs."""
import sys

import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dfpr():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2401_03256_amd import dfpr as mod
    mod.lib()
    return mod


# (vertices, edges): below, at and above one tile of 4096 keys (edges and
# self-loops), two tiles, one vertex, ids of one and of nine bits, more
# degrees than one digit holds
@pytest.mark.parametrize("n,m", [(1, 0), (1, 5), (2, 1), (2, 300), (96, 3999), (96, 4000), (96, 4001),
                                 (257, 7935), (4095, 0), (4096, 1), (300, 90000), (70000, 5)])
def test_load_matches_oracle_csr(dfpr, n, m):
    sys.stdout.write(f"\n[case] load {n} {m}\n")
    sys.stdout.flush()
    rng = np.random.default_rng(n + m)
    src = rng.integers(0, n, m).astype(np.int32)
    dst = (rng.integers(0, n, m) * rng.random(m) ** 3).astype(np.int32)   # skewed targets
    if m > 10:
        src[-5:], dst[-5:] = src[0], dst[0]         # repeats
        dst[1:4] = src[1:4]                         # self-loops
    g, o = dfpr.Graph(n, src, dst), oracle.OracleGraph(n, src, dst)
    assert g.m == o.m
    for out in (True, False):
        for x, y in zip(g.csr(out), o.csr(out)):
            assert np.array_equal(x, y)
    R, _ = o.static()
    assert np.abs(g.static()[0] - R).max() <= 1e-9


@pytest.mark.parametrize("where", [0, 4999])
def test_load_rejects_bad_ids(dfpr, where):
    src = np.zeros(5000, np.int32)
    dst = np.arange(5000, dtype=np.int32) % 40
    for bad in (-1, 40):
        d = dst.copy()
        d[where] = bad
        with pytest.raises(dfpr.DfprError) as e:
            dfpr.Graph(40, src, d)
        assert e.value.code == dfpr.DFPR_E_RANGE
