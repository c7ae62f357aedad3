"""Small-item groups on either side of the number up to which four wavefronts
share a group: counts, per-vertex and per-edge values must equal the oracle's."""

import numpy as np
import pytest

from oracle import vp_counts

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,n", [(300, 20), (30000, 9000), (170000, 50000), (260000, 50000), (400000, 50000)])
def test_groups_around_the_team_bound(m, n):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.set_device(0)
    import paper_2609_21848_amd as dbbc
    rng = np.random.default_rng(m)
    key = np.unique(rng.integers(0, n * n, m))
    key = key[rng.permutation(len(key))]
    u, v = (key // n).astype(np.int32), (key % n).astype(np.int32)
    s = rng.choice([-1, 1], len(key)).astype(np.int8)
    r = vp_counts(n, n, u, v, s, per_vertex=True, per_edge=True)
    with dbbc.Graph(n, n, u, v, s) as h:
        for opts in ({}, dict(small_work=40)):
            c = h.count(**opts)
            assert (c.balanced, c.unbalanced, c.total) == (r.balanced, r.unbalanced, r.total)
            c, bu, bv, uu, uv = h.count_per_vertex(**opts)
            for t, want in ((bu, r.bal_u), (bv, r.bal_v), (uu, r.unb_u), (uv, r.unb_v)):
                assert np.array_equal(t.cpu().numpy(), want)
            c, be, ue = h.count_per_edge(**opts)
            assert np.array_equal(be.cpu().numpy(), r.bal_e) and np.array_equal(ue.cpu().numpy(), r.unb_e)
