"""A device batch with an id outside [0, n) ends in DFPR_E_RANGE on every route
that the iterations of a call can take, on a fresh graph and after a call, and
leaves ranks and marks as they were."""
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


def _device(arrays):
    import torch
    return [torch.from_numpy(np.ascontiguousarray(x)).cuda() for x in arrays]


ROUTES = {
    "default": lambda d: (dict(), False),
    "async": lambda d: (dict(mode=d.ASYNC), False),
    "profiled": lambda d: (dict(), True),
    "profiled_fp32": lambda d: (dict(precision=d.FP32_KAHAN), True),
    "async_fp32": lambda d: (dict(mode=d.ASYNC, precision=d.FP32_KAHAN), False),
}


# 5 entries: staged by the kernel that begins a call; 1500: by kernels of their own
@pytest.mark.parametrize("entries", [5, 1500])
@pytest.mark.parametrize("noalloc", [False, True])
@pytest.mark.parametrize("route", list(ROUTES))
def test_bad_id_is_refused_on_every_route(dfpr, route, noalloc, entries):
    import torch
    sys.stdout.write(f"\n[case] bad id, {route}, noalloc {noalloc}, {entries} entries\n")
    sys.stdout.flush()
    kw, profiled = ROUTES[route](dfpr)
    p = dfpr.params(**kw)
    n, src, dst = 9000, *synth.gnm(9000, 60_000, seed=3)
    good = synth.random_batch(src, dst, n, entries // 5, entries - entries // 5, seed=4)
    arrays = [good.del_src, good.del_dst, good.ins_src, good.ins_dst]
    g = dfpr.Graph(n, src, dst)
    g.profile_reset(profiled)
    prev = torch.from_numpy(np.random.default_rng(5).dirichlet(np.ones(n))).cuda()
    for fresh in (True, False):
        before, marks = g.ranks(), g.affected()
        for which in range(4):
            for bad in (-1, n):
                x = [a.copy() for a in arrays]
                x[which][-1] = bad
                x = _device(x)
                with pytest.raises(dfpr.DfprError) as e:
                    g.dynamic_frontier_device(*x, p=p, noalloc=noalloc)
                assert e.value.code == dfpr.DFPR_E_RANGE, (fresh, which, bad)
                assert np.array_equal(g.ranks(), before)
                assert np.array_equal(g.affected(), marks)
        with pytest.raises(dfpr.DfprError) as e:
            g.dynamic_frontier_device(*x, prev=prev, p=p, noalloc=noalloc)
        assert e.value.code == dfpr.DFPR_E_RANGE
        assert np.array_equal(g.ranks(), prev.cpu().numpy())
        g.set_ranks(before)
        if fresh:
            assert g.apply_batch(good) == (entries // 5, entries - entries // 5)
            st = g.dynamic_frontier_device(*_device(arrays), p=p, noalloc=noalloc)
            assert st.converged and g.affected().any()
