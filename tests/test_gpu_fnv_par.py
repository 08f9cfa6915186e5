"""GPU parity of the many-lanes FNV-1a (items of more than 512 bytes) with the
oracle: item sizes around its column, step and lane-group edges, every kind of
short item, the rule between it and the one-lane-per-item chain, helper
wavefronts and the shorter lists of small persistent launches."""
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
    ctx = g.Context(ring_slots=1 << 14, device_timeout_ns=20_000_000_000)
    yield g, ctx
    assert ctx.shutdown() == 0


def lengths(rng, n, item):
    """Byte counts of n items: full, empty, negative (an errno), one byte, and
    around 16-byte, lane (128), column (512) and step (8192) edges."""
    edges = [item, 0, -9, 1, item - 1, 15, 16, 17, 127, 128, 129, 511, 512, 513, 8191, 8192, 8193]
    e = np.array([x for x in edges if x <= item], dtype=np.int64)
    r = rng.integers(0, item + 1, n)
    r[:min(n, len(e))] = e[:n]
    r[rng.random(n) < 0.4] = item
    return r.astype(np.int64)


@pytest.mark.parametrize("item,n", [(576, 33), (960, 40), (1024, 37), (1088, 50), (4096, 67),
                                    (4160, 34), (8192, 21), (8256, 35), (16384, 9), (65600, 20),
                                    (1 << 20, 3)])
@pytest.mark.parametrize("wg,grid", [(256, 0), (64, 2), (512, 1), (1024, 1)])
def test_consume_matches_oracle(gs, item, n, wg, grid):
    import torch
    g, ctx = gs
    from paper_1705_06965_amd.fnv import consume
    rng = np.random.default_rng([item, n])
    data = rng.integers(0, 256, (n, item), dtype=np.uint8)
    lens = lengths(rng, n, item)
    want = [oracle.fnv1a64(data[i, :max(0, lens[i])]) for i in range(n)]
    d = torch.from_numpy(data.reshape(-1)).to("cuda")
    rets = torch.from_numpy(lens).to("cuda")
    out = torch.full((n,), -1, dtype=torch.int64, device="cuda")
    print("consume", item, n, wg, grid, flush=True)
    consume(ctx, d.data_ptr(), rets, item, out, wg, grid)
    got = out.cpu().numpy().view(np.uint64)
    assert got.tolist() == want


@pytest.mark.parametrize("item", [640, 1024])
def test_consume_rule_both_sides(gs, item):
    """Enough sparse items for the chains to fill the chip take the chain,
    dense ones and fewer items many lanes; all give the same hashes."""
    import torch
    g, ctx = gs
    from paper_1705_06965_amd.fnv import consume
    rng = np.random.default_rng(item)
    one = rng.integers(0, 256, (1000, item), dtype=np.uint8)
    want = np.array([oracle.fnv1a64(r) for r in one], dtype=np.uint64)
    for reps in (1, 180):
        d = torch.from_numpy(one.reshape(-1)).to("cuda").repeat(reps)
        n = 1000 * reps
        out = torch.zeros(n, dtype=torch.int64, device="cuda")
        rets = torch.full((n,), item, dtype=torch.int64, device="cuda")
        print("rule", item, n, flush=True)
        consume(ctx, d.data_ptr(), rets, item, out)
        assert (out.cpu().numpy().view(np.uint64).reshape(reps, 1000) == want).all()


@pytest.mark.parametrize("n,item,wg", [(1, 4096, 64), (65, 4096, 64), (300, 832, 128),
                                       (70, 20480, 512), (40, 65536, 1024), (3000, 1024, 256),
                                       (9, 1 << 20, 256)])
@pytest.mark.parametrize("form,cell", [("plain", ("WI", "strong", "block")),
                                       ("plain", ("WG", "strong", "nonblock")),
                                       ("plain", ("K", "relaxed", "block")),
                                       ("persistent", ("WI", "strong", "block")),
                                       ("graph", ("WI", "strong", "block"))])
def test_helpers_and_short_lists(gs, tmpdata, n, item, wg, form, cell):
    g, ctx = gs
    import os
    from paper_1705_06965_amd.fnv import FnvRunner
    rng = np.random.default_rng([n, item, wg])
    size = 2 * item + 1234
    path = os.path.join(tmpdata, "par_%d.bin" % item)
    rng.integers(0, 256, size, dtype=np.uint8).tofile(path)
    offs = rng.integers(0, size + 100, n).astype(np.uint64)  # some end or start past the end
    want, want_ret = oracle.pread_fnv(path, offs, item)
    r = FnvRunner(ctx, path, offs, item, wg_size=wg)
    print("helpers", n, item, wg, form, cell, flush=True)
    f, ret = r.run(*cell, form={"plain": g.PLAIN, "persistent": g.PERSISTENT, "graph": g.GRAPH}[form])
    r.close()
    assert (ret == want_ret).all() and (f == want).all()


def test_drain_reads_the_counter_after_an_error_of_the_callers(gs, tmpdata):
    """A runtime error that the caller has not cleared (a device that does not
    exist) is not the drain's: the claimed count is the device's."""
    import ctypes
    import os
    from paper_1705_06965_amd.fnv import FnvRunner
    g, ctx = gs
    path = os.path.join(tmpdata, "drain.bin")
    np.zeros(4096, dtype=np.uint8).tofile(path)
    r = FnvRunner(ctx, path, np.zeros(3, dtype=np.uint64), 64, wg_size=64)
    r.run()
    r.close()
    with open("/proc/self/maps") as f:
        so = next(l.split()[-1] for l in f if "libamdhip64" in l)
    hip = ctypes.CDLL(so)
    before = ctx.stats()["claimed"]
    assert before >= 3
    try:
        assert hip.hipSetDevice(1 << 20) != 0
        assert ctx.stats()["claimed"] == before
    finally:
        hip.hipGetLastError()


@pytest.mark.parametrize("wg", [64, 1024])
@pytest.mark.parametrize("over", [0, 1])
def test_spread_work_groups_at_the_last_size(gs, tmpdata, wg, over):
    """The most items that work-groups of 16 spread over all compute units
    take, and one more."""
    import os
    import torch
    from paper_1705_06965_amd.fnv import FnvRunner
    g, ctx = gs
    n = 16 * torch.cuda.get_device_properties(0).multi_processor_count + over
    rng = np.random.default_rng(n)
    path = os.path.join(tmpdata, "spread.bin")
    rng.integers(0, 256, 100000, dtype=np.uint8).tofile(path)
    offs = rng.integers(0, 100100, n).astype(np.uint64)
    want, want_ret = oracle.pread_fnv(path, offs, 4096)
    r = FnvRunner(ctx, path, offs, 4096, wg_size=wg)
    print("spread", n, wg, flush=True)
    f, ret = r.run("WI", "strong", "block")
    r.close()
    assert (ret == want_ret).all() and (f == want).all()
