"""The radix sort with 64-bit published words, the form for 2^30 elements and
more, on inputs of a few tiles: both tile shapes around their edges, keys of one
to four passes, all equal and all different; stable, against numpy."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lib():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.set_device(0)
    torch.zeros(1, device="cuda")
    from radix_wide import load
    return load()


@pytest.mark.parametrize("n", [1, 1023, 1024, 1025, 40_000, (1 << 20) - 1, 1 << 20, (1 << 20) + 1, 5 * 4096 * 256 + 4095])
@pytest.mark.parametrize("bits,kind", [(3, "random"), (8, "equal"), (17, "random"), (32, "random"), (32, "few")])
def test_wide_words_sort(lib, n, bits, kind):
    import torch
    rng = np.random.default_rng(n + bits)
    if kind == "equal":
        key = np.full(n, 77, np.uint32)
    elif kind == "few":
        key = rng.choice(np.array([0, 1, 255, 256, 1 << 31, (1 << 32) - 1], np.uint32), n)
    else:
        key = rng.integers(0, 1 << bits, n).astype(np.uint32)
    k = torch.from_numpy(key.view(np.int32)).cuda()
    out = torch.empty((2, n), dtype=torch.int32, device="cuda")
    torch.cuda.synchronize()
    assert lib.radix_wide_sort(k.data_ptr(), n, bits, out[0].data_ptr(), out[1].data_ptr()) == 0
    order = np.argsort(key, kind="stable")
    got = out.cpu().numpy().view(np.uint32)
    assert np.array_equal(got[1], order.astype(np.uint32))
    assert np.array_equal(got[0], key[order])
