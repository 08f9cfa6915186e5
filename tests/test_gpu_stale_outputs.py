"""Results of a runner's earlier run are never returned by a later one: every
cell and form of the drivers stores each of its results, and a launch that
stored nothing would show (the drivers keep their result tensors and do not
clear them; conftest.py poisons them before every run a GPU test makes)."""
import os

import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

FORMS = ["plain", "persistent", "graph"]


@pytest.fixture(scope="module")
def gs():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1705_06965_amd as g
    ctx = g.Context(ring_slots=1 << 12, device_timeout_ns=20_000_000_000)
    yield g, ctx
    assert ctx.shutdown() == 0


@pytest.fixture(scope="module")
def data(tmp_path_factory):
    d = tmp_path_factory.mktemp("stale")
    p = str(d / "in.bin")
    np.random.default_rng(11).integers(0, 256, 1 << 20, dtype=np.uint8).tofile(p)
    return p


def words(g, ctx, tmpdata, by_name):
    from paper_1705_06965_amd.wordscan import WordOpenRunner, WordScanRunner
    d = os.path.join(tmpdata, "stale_words")
    os.makedirs(d, exist_ok=True)
    names = ["a", "b", "c"]
    for i, n in enumerate(names):
        with open(os.path.join(d, n), "wb") as f:
            f.write(b"one two " * (i + 1))
    if by_name:
        return WordOpenRunner(ctx, d, names, [b"one", b"two"], chunk=4096)
    return WordScanRunner(ctx, [os.path.join(d, n) for n in names], [b"one", b"two"])


@pytest.mark.parametrize("which", ["fnv", "permute", "scan", "open"])
def test_a_run_that_stores_nothing_shows(gs, data, tmpdata, which):
    """With the launch left out, a second run gives the poison, not the first
    run's results."""
    g, ctx = gs
    from conftest import POISON
    if which == "fnv":
        from paper_1705_06965_amd.fnv import FnvRunner
        r = FnvRunner(ctx, data, np.arange(70, dtype=np.uint64) * 4096, 4096)
    elif which == "permute":
        from paper_1705_06965_amd.permute import PermuteRunner
        out = os.path.join(tmpdata, "stale_permute.bin")
        np.zeros(3 * 8192, dtype=np.uint8).tofile(out)
        r = PermuteRunner(ctx, out, np.arange(3 * 1024, dtype=np.uint64), np.arange(1024),
                          np.arange(64))
    else:
        r = words(g, ctx, tmpdata, which == "open")
    args = (1,) if which == "permute" else ()
    print("stale", which, flush=True)
    first = r.run(*args)
    r.launch = lambda *a, **k: 0
    second = r.run(*args)
    r.close()
    for a, b in zip(first if isinstance(first, tuple) else (first,),
                    second if isinstance(second, tuple) else (second,)):
        assert not (a == np.array(POISON).astype(b.dtype)).any()
        assert (b == np.array(POISON).astype(b.dtype)).all()


@pytest.mark.parametrize("item,wg,n", [(256, 64, 200), (4096, 256, 300), (4096, 1024, 1100),
                                       (8256, 128, 130), (65536, 64, 9)])
def test_every_cell_and_form_stores_every_item(gs, data, item, wg, n):
    """One runner, other offsets in each run: whole, short and empty reads."""
    import torch
    g, ctx = gs
    from paper_1705_06965_amd.fnv import FnvRunner
    rng = np.random.default_rng([item, wg, n])
    r = FnvRunner(ctx, data, np.zeros(n, dtype=np.uint64), item, wg_size=wg)
    for form in FORMS:
        for cell in (g.LEGAL_CELLS if form == "plain" else g.LEGAL_CELLS[:1]):
            offs = rng.integers(0, (1 << 20) + item, n).astype(np.uint64)
            r.offsets.copy_(torch.from_numpy(offs.view(np.int64)))
            want, want_ret = oracle.pread_fnv(data, offs, item)
            print("every item", item, wg, n, form, cell, flush=True)
            f, ret = r.run(*cell, form={"plain": g.PLAIN, "persistent": g.PERSISTENT,
                                        "graph": g.GRAPH}[form])
            assert (ret == want_ret).all() and (f == want).all(), (form, cell)
    r.close()


@pytest.mark.parametrize("n,cell,form,cleared", [
    (100, ("WI", "strong", "block"), "plain", False),
    (65536, ("WI", "strong", "block"), "plain", False),
    (70000, ("WI", "strong", "block"), "plain", True),
    (70000, ("WG", "strong", "block"), "plain", False),
    (70000, ("WI", "strong", "block"), "persistent", False),
    (70000, ("WI", "strong", "block"), "graph", False)])
def test_large_runs_clear_their_results_first(gs, data, n, cell, form, cleared):
    """Launches of more work-item calls than a ring has slots clear the results
    before it, on its stream; others would only be slower for it."""
    g, ctx = gs
    from conftest import POISON
    from paper_1705_06965_amd.fnv import FnvRunner
    import torch
    code = {"plain": g.PLAIN, "persistent": g.PERSISTENT, "graph": g.GRAPH}[form]
    r = FnvRunner(ctx, data, np.arange(n, dtype=np.uint64), 64, wg_size=64)
    want = oracle.pread_fnv(data, np.arange(n, dtype=np.uint64), 64)
    side = torch.cuda.Stream()
    for s in (None, side):  # on the stream of the launch, so never after it
        print("cleared", n, cell, form, s, flush=True)
        f, ret = r.run(*cell, form=code, stream=s)
        assert (f == want[0]).all() and (ret == want[1]).all()
    switched = []
    stream = torch.cuda.stream
    r.launch = lambda *a, **k: 0
    for s in (None, side):
        torch.cuda.stream = lambda x: switched.append(x) or stream(x)
        try:
            f, ret = r.run(*cell, form=code, stream=s)
        finally:
            torch.cuda.stream = stream
        left = -12345 if cleared else POISON
        assert (ret == left).all() and (f.view(np.int64) == left).all()
        # torch's own stream is not switched to: that takes longer than the rest
        assert len(switched) == (cleared and s is side)
    r.close()
