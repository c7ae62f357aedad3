"""Counts of pairs with more than 46,340 wedges of one sign (squares of 2^31 and
more), as keys of a hub pivot past the dense block and as plain window keys.
The expected counts follow from the graph's form: every V vertex is adjacent to
the same `common` U vertices with positive edges, so every V pair has `common`
balanced wedges."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("common", [46340, 46341, 60000])
@pytest.mark.parametrize("n_v,hub_T", [(3, 0), (131, 128)])
def test_pairs_of_many_wedges(common, n_v, hub_T):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.set_device(0)
    import paper_2609_21848_amd as dbbc
    u = np.tile(np.arange(common, dtype=np.int32), n_v)
    v = np.repeat(np.arange(n_v, dtype=np.int32), common)
    pairs = n_v * (n_v - 1) // 2
    want = pairs * (common * (common - 1) // 2)
    with dbbc.Graph(common, n_v, u, v, np.ones(len(u), np.int8)) as h:
        for opts in (dict(hub_T=hub_T), {}):
            c = h.count(**opts)
            assert (c.balanced, c.unbalanced, c.total) == (want, 0, want)
