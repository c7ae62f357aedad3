"""The direct kernel's workgroup shapes (as many counters as the widest key
window of a launch needs) at the sizes where they change, alone and in batches
that mix graphs, and the default budget of a direct item's parts.  All counts
are integers and must equal the oracle's."""

import numpy as np
import pytest

from oracle import vp_counts
from synth import chung_lu_graph

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dbbc():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.set_device(0)
    import paper_2609_21848_amd as mod
    mod.load()
    return mod


def _graph(n, m=120_000, gamma=2.05, seed=0):
    g = chung_lu_graph(n, max(n // 2, 60), min(m, n * max(n // 2, 60) // 3), gamma, gamma, 0.4, seed=seed)
    r = vp_counts(g.n_u, g.n_v, g.u, g.v, g.sign)
    return g, (r.balanced, r.unbalanced, r.total, r.wedges)


@pytest.mark.parametrize("n", [300, 4096, 8191, 8192, 8193, 16384, 16385, 32768, 32769, 50000])
def test_window_widths_alone(dbbc, n):
    g, want = _graph(n, seed=n)
    with dbbc.Graph(g.n_u, g.n_v, g.u, g.v, g.sign) as h:
        for opts in ({}, dict(small_work=16), dict(small_work=16, part_work=4096), dict(window_L=8192, part_work=4096),
                     dict(window_L=16384, small_work=16)):
            assert tuple(h.count(**opts)) == want, opts


@pytest.mark.parametrize("widest", [5000, 8192, 12000, 40000])
def test_batches_that_mix_graphs(dbbc, widest):
    import torch
    gs = [_graph(n, m, seed=n) for n, m in ((60, 500), (widest, 90_000), (700, 30_000), (3000, 60_000), (200, 5_000),
                                            (widest, 40_000), (64, 64))]
    hs = [dbbc.Graph(g.n_u, g.n_v, g.u, g.v, g.sign) for g, _ in gs]
    for capture in (False, True):
        with dbbc.Batch(hs, capture=capture, small_work=16) as b:
            for _ in range(3):
                assert [tuple(c) for c in b.count()] == [want for _, want in gs]
                torch.zeros(1 << 20, device="cuda").sum().item()
    for h in hs:
        h.close()


def test_default_parts_of_heavy_items(dbbc):
    # a few items of more than 2^18 wedges: split by default, refused nowhere
    g, want = _graph(60_000, 700_000, 1.9, seed=3)
    with dbbc.Graph(g.n_u, g.n_v, g.u, g.v, g.sign) as h:
        assert tuple(h.count(flags=dbbc.DBBC_OPT_TIME_KERNELS)) == want
        assert sum(k["items"] for k in h.kernel_times() if k["name"] == "reduce") > 0
        assert tuple(dbbc.dbbc_count_noalloc(h.handle)) == want
        assert tuple(h.count(flags=dbbc.DBBC_OPT_HOST_PLAN)) == want
