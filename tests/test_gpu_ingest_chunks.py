"""Text ingestion where its chunks can go wrong: line starts at every place
around a chunk's end, lines longer than a chunk and its tail, texts that start
at any alignment, and lines that are no records in between.  The expected
records are read in plain Python; results are integers and must be equal."""

import numpy as np
import pytest

from oracle import vp_counts

pytestmark = pytest.mark.gpu

CHUNK = 8192


@pytest.fixture(scope="module")
def dbbc():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.set_device(0)
    import paper_2609_21848_amd as mod
    mod.load()
    return mod


def _check(dbbc, text: bytes, lead: int = 0):
    import torch
    recs = []
    for line in text.decode().split("\n"):
        f = line.replace(",", " ").split()
        if f and f[0][0] not in "#%":
            recs.append((int(f[0]), int(f[1]), 1 if int(f[2]) == 1 else -1))
    ru, u = np.unique([r[0] for r in recs], return_inverse=True)
    rv, v = np.unique([r[1] for r in recs], return_inverse=True)
    s = np.array([r[2] for r in recs], np.int8)
    key = u.astype(np.int64) * len(rv) + v
    last = np.sort(len(u) - 1 - np.unique(key[::-1], return_index=True)[1])
    r = vp_counts(len(ru), len(rv), u[last].astype(np.int32), v[last].astype(np.int32), s[last], per_edge=True)
    t = torch.frombuffer(bytearray(b"7" * lead + text), dtype=torch.uint8).to("cuda:0")[lead:]
    with dbbc.Graph.from_text(t) as h:
        c, be, _ = h.count_per_edge()
        assert h.info == {"lines": text.count(b"\n") + (not text.endswith(b"\n")), "records": len(recs),
                          "n_u": len(ru), "n_v": len(rv)}
        assert h.raw_ids(0).cpu().tolist() == list(ru) and h.raw_ids(1).cpu().tolist() == list(rv)
    assert (c.balanced, c.unbalanced) == (r.balanced, r.unbalanced)
    full = np.zeros(len(u), np.int64)
    full[last] = r.bal_e
    assert np.array_equal(be.cpu().numpy(), full)


def _lines(rng, n):
    return [b"%d %d %d" % (rng.integers(1, 10 ** rng.integers(1, 4)), rng.integers(1, 60), rng.integers(0, 2))
            for _ in range(n)]


@pytest.mark.parametrize("lead", [0, 1, 7, 15])
@pytest.mark.parametrize("shift", [-2, -1, 0, 1, 2])
def test_line_starts_around_a_chunk_end(dbbc, lead, shift):
    rng = np.random.default_rng(10 * lead + shift + 2)
    head = b"\n".join(_lines(rng, 700)) + b"\n"
    # a comment that ends `shift` bytes from the first chunk's end
    pad = CHUNK - lead + shift - len(head) - 1
    assert pad > 0
    tail = b"\n".join(_lines(rng, 900))
    _check(dbbc, head + b"#" + b"x" * (pad - 1) + b"\n" + tail + (b"\n" if shift % 2 else b""), lead)


@pytest.mark.parametrize("length", [100, 255, 256, 257, CHUNK - 1, CHUNK, 3 * CHUNK + 5])
def test_long_lines(dbbc, length):
    rng = np.random.default_rng(length)
    a, b = _lines(rng, 650), _lines(rng, 650)
    a[40] += b" " + b"9" * length          # fields after the third
    a[-1] = b" " * length + a[-1]          # leading spaces past the chunk's tail
    b[3] = b"%" + b"0" * length
    _check(dbbc, b"\n".join(a + b) + b"\n", length % 16)


def test_one_line_and_only_newlines_between(dbbc):
    _check(dbbc, b"9223372036854775807 3 1")
    _check(dbbc, b"\n" * (2 * CHUNK + 3) + b"5 3 1\n5,4,0" + b"\n" * CHUNK, 3)
