"""Equal queries: the first of them gets the counts, the others none, in every
form of the word search."""
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


def first_only(queries):
    """Index of the first query equal to each one."""
    return np.array([queries.index(q) for q in queries])


@pytest.mark.parametrize("queries", [
    [b"one"] * 64, [b"one", b"two"] * 32, [b"two"] + [b"one"] * 5 + [b"two", b"abcdefghijklmnop"] * 3,
    [bytes([97 + i % 26]) for i in range(64)], [b"%d" % (i % 23) for i in range(60)]],
    ids=["all", "two", "mixed", "letters", "numbers"])
def test_the_first_of_equal_queries_counts(gs, tmpdata, queries):
    g, ctx = gs
    from paper_1705_06965_amd.wordscan import WordOpenRunner, WordScanRunner
    rng = np.random.default_rng(len(queries))
    d = os.path.join(tmpdata, "equal")
    os.makedirs(d, exist_ok=True)
    words = sorted(set(queries)) + [b"absent", b"onetwo"]
    names = ["e%d" % i for i in range(5)]
    for n in names:
        with open(os.path.join(d, n), "wb") as f:
            f.write(b" ".join(words[k] for k in rng.integers(0, len(words), 4000)))
    paths = [os.path.join(d, n) for n in names]
    want = oracle.wordcount(paths, queries)
    want[:, first_only(queries) != np.arange(len(queries))] = 0
    print("equal", len(queries), flush=True)
    r = WordScanRunner(ctx, paths, queries, chunk_max=8192)
    for form in (g.PLAIN, g.PERSISTENT, g.GRAPH):
        assert (r.run(form) == want).all()
    r.close()
    o = WordOpenRunner(ctx, d, names, queries, chunk=4096)
    got, _ = o.run()
    o.close()
    assert (got == want).all()
