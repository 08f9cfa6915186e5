"""GPU parity of the word scanner at the edges of its pieces: lanes (64 bytes),
wavefront sub-blocks (4 KiB), a work-group's round of sub-blocks (32 KiB),
tokens of 16 and 17 bytes across each of them, queries that share their first
four bytes or their filter bit, and one token per two bytes everywhere."""
import os

import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gs():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1705_06965_amd as g
    ctx = g.Context(ring_slots=1 << 12, device_timeout_ns=20_000_000_000)
    yield g, ctx
    assert ctx.shutdown() == 0


QUERIES = [b"a", b"b", b"ab", b"abc", b"abcd", b"abcde", b"abcdX", b"abcdefghijklmnop",
           b"abcdefghijklmnoq", b"abcdefghijklmno", b"zzzz", b"zzz", b"\x00", b"\x00\x00",
           b"\xff\x80\x7f", b"aaaa", b"aaaaa"]


def texts():
    rng = np.random.default_rng(3)
    out = [b"", b"a", b" ", b"abcdefghijklmnop", b"abcdefghijklmnopq", b"a " * 40000, b"x" * 70000]
    words = QUERIES + [w + b"q" for w in QUERIES[:-2]] + [b"abcdefghijklmnop" * 3]
    for edge in (64, 4096, 32768, 65536):
        for w in (b"abcdefghijklmnop", b"abcdefghijklmnopq", b"abcd", b"a"):
            # the word placed so that it starts, ends and crosses at the edge
            for at in (edge - len(w) - 1, edge - len(w), edge - 1, edge, edge - len(w) // 2):
                t = bytearray(b" " * (edge + 100))
                t[at:at + len(w)] = w
                out.append(bytes(t[:at + len(w)] if at % 2 else t))
    for n in (1, 63, 4095, 4097, 40000, 140000):
        b = b""
        while len(b) < n:
            b += words[rng.integers(len(words))] + (b"\n" if rng.random() < 0.2 else b" ")
        out.append(b[:n])
    return out


@pytest.mark.parametrize("chunk", [64, 4096, 4160, 1 << 20])
@pytest.mark.parametrize("form", ["plain", "persistent", "graph"])
def test_edges_match_oracle(gs, tmpdata, chunk, form):
    g, ctx = gs
    from paper_1705_06965_amd.wordscan import WordScanRunner
    d = os.path.join(tmpdata, "edges")
    os.makedirs(d, exist_ok=True)
    paths = []
    for i, t in enumerate(texts()):
        if chunk == 64 and len(t) > 40000:
            continue
        p = os.path.join(d, "t%03d" % i)
        with open(p, "wb") as f:
            f.write(t)
        paths.append(p)
    want = oracle.wordcount(paths, QUERIES)
    print("edges", chunk, form, len(paths), flush=True)
    r = WordScanRunner(ctx, paths, QUERIES, chunk_max=chunk)
    got = r.run({"plain": g.PLAIN, "persistent": g.PERSISTENT, "graph": g.GRAPH}[form])
    r.close()
    r.staging_p.free()
    if r.staging_w is not None:
        r.staging_w.free()
    assert (got == want).all(), np.argwhere(got != want)[:10]


@pytest.mark.parametrize("chunk", [64, 4096, 65536])
def test_open_edges_match_oracle(gs, tmpdata, chunk):
    g, ctx = gs
    from paper_1705_06965_amd.wordscan import WordOpenRunner
    d = os.path.join(tmpdata, "open_edges_%d" % chunk)
    os.makedirs(d, exist_ok=True)
    names = []
    for i, t in enumerate(texts()):
        if chunk == 64 and len(t) > 5000:
            continue
        names.append("t%03d" % i)
        with open(os.path.join(d, names[-1]), "wb") as f:
            f.write(t)
    paths = [os.path.join(d, n) for n in names]
    want = oracle.wordcount(paths, QUERIES)
    print("open edges", chunk, len(names), flush=True)
    r = WordOpenRunner(ctx, d, names, QUERIES, chunk=chunk, groups=48)
    counts, ret = r.run(timeout_s=30.0)
    r.close()
    assert ret.tolist() == [os.path.getsize(p) for p in paths]
    assert (counts == want).all(), np.argwhere(counts != want)[:10]


@pytest.mark.parametrize("n", [2, 3, 4, 5, 6, 7, 97, 193])
def test_width_and_grid_rules(gs, tmpdata, n):
    """File counts on both sides of the lines between wide and narrow
    work-groups (two of them, and the 96 of the search by name) and past the
    grid; every progress record ends."""
    g, ctx = gs
    from paper_1705_06965_amd.wordscan import WordOpenRunner, WordScanRunner
    rng = np.random.default_rng(n)
    d = os.path.join(tmpdata, "rules%d" % n)
    os.makedirs(d, exist_ok=True)
    names = []
    for i in range(n):
        words = [QUERIES[k] for k in rng.integers(0, len(QUERIES), rng.integers(0, 3000))]
        names.append("f%d.txt" % i)
        with open(os.path.join(d, names[-1]), "wb") as f:
            f.write(b" ".join(words))
    paths = [os.path.join(d, x) for x in names]
    want = oracle.wordcount(paths, QUERIES)
    print("rules", n, flush=True)
    r = WordScanRunner(ctx, paths, QUERIES, persistent_buffers=4)
    assert (r.run(g.PERSISTENT) == want).all()
    assert (r.run(g.GRAPH) == want).all()
    r.close()
    for groups, chunk in ((2, 4096), (2, 65536), (2, 1 << 18), (256, 1 << 18)):
        r = WordOpenRunner(ctx, d, names, QUERIES, chunk=chunk, groups=groups)
        print("rules by name", n, groups, chunk, flush=True)
        got, ret = r.run()
        assert (got == want).all() and ret.tolist() == [os.path.getsize(p) for p in paths]
        assert all(p[1] == 5 for p in r.progress_records())
        r.close()
