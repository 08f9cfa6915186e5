"""GPU parity of gsys_fnv4k_consume with the oracle where items are shorter than
their slots: lengths on which the kernel hashes all of a wavefront's items with
the chains, some groups of them, or none, one and two looks at the lengths per
wavefront, groups of 1 to 8 items, and the ends of items in every position of
the chains' 16-byte pieces."""
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
    ctx = g.Context(ring_slots=1 << 10, device_timeout_ns=20_000_000_000)
    yield g, ctx
    assert ctx.shutdown() == 0


def lengths(kind, rng, n, item):
    r = np.full(n, item, dtype=np.int64)
    if kind == "short":
        r = rng.integers(0, 513, n)
    elif kind == "tiny":
        r = rng.integers(-5, 101, n)
    elif kind == "none":
        r[:] = rng.integers(-9, 1, n)
    elif kind == "uniform":
        r = rng.integers(0, item + 1, n)
    elif kind == "equal":
        r[:] = 384
    elif kind == "runs":     # short and full ones in turn, in every wavefront
        r[np.arange(n) // 5 % 2 == 0] = 100
    elif kind == "half":
        r[rng.random(n) < 0.5] = 0
    elif kind == "few":
        at = rng.random(n) < 0.05
        r[at] = rng.integers(-1, item, int(at.sum()))
    elif kind == "edges":
        e = [0, 1, 15, 16, 17, 31, 127, 128, 129, 255, 256, 257, 511, 512, 513, item - 1, item]
        r = np.array(e)[rng.integers(0, len(e), n)]
    elif kind == "region":   # all short but the last
        r = rng.integers(0, 300, n)
        r[-3:] = item
    return r.astype(np.int64)


KINDS = ["short", "tiny", "none", "uniform", "equal", "runs", "half", "few", "edges", "region"]


# 16 wavefronts of the explicit grids: 70 items each of at most 1 KiB, 88 of 2
# and 4 KiB are more than one look
@pytest.mark.parametrize("item,n", [(576, 1121), (1024, 1100), (1088, 1400), (2048, 1390),
                                    (4096, 1409), (4160, 700), (8192, 333), (8256, 200),
                                    (65600, 40)])
@pytest.mark.parametrize("wg,grid", [(256, 0), (256, 4), (1024, 1)])
def test_lengths_match_oracle(gs, item, n, wg, grid):
    import torch
    g, ctx = gs
    from paper_1705_06965_amd.fnv import consume
    rng = np.random.default_rng([item, n])
    data = rng.integers(0, 256, (n, item), dtype=np.uint8)
    d = torch.from_numpy(data.reshape(-1)).to("cuda")
    for kind in KINDS:
        lens = lengths(kind, rng, n, item)
        want = [oracle.fnv1a64(data[i, :max(0, lens[i])]) for i in range(n)]
        out = torch.full((n,), -1, dtype=torch.int64, device="cuda")
        print("lengths", item, n, wg, grid, kind, flush=True)
        consume(ctx, d.data_ptr(), torch.from_numpy(lens).to("cuda"), item, out, wg, grid)
        got = out.cpu().numpy().view(np.uint64)
        assert got.tolist() == want, kind


def test_chains_at_every_tail(gs):
    """Items of up to 512 bytes (always the chains), all lengths."""
    import torch
    g, ctx = gs
    from paper_1705_06965_amd.fnv import consume
    rng = np.random.default_rng(5)
    n, item = 513 * 3, 512
    data = rng.integers(0, 256, (n, item), dtype=np.uint8)
    lens = rng.permutation(np.arange(n) % 513).astype(np.int64)
    want = [oracle.fnv1a64(data[i, :lens[i]]) for i in range(n)]
    d = torch.from_numpy(data.reshape(-1)).to("cuda")
    for wg in (64, 1024):
        out = torch.zeros(n, dtype=torch.int64, device="cuda")
        print("tails", wg, flush=True)
        consume(ctx, d.data_ptr(), torch.from_numpy(lens).to("cuda"), item, out, wg)
        assert out.cpu().numpy().view(np.uint64).tolist() == want
