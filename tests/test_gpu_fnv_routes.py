"""GPU parity with the oracle of the plain-form launches whose route the rules
of fnv_rules.hpp choose: chains in wide work-groups of long items, work-item
calls with and without helper wavefronts, and more calls than ring slots."""
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
    ctx = g.Context(ring_slots=1 << 15, device_timeout_ns=20_000_000_000)
    yield g, ctx
    assert ctx.shutdown() == 0


@pytest.mark.parametrize("cell,n,item,wg", [
    (("WG", "strong", "block"), 1030, 16448, 1024), (("WG", "relaxed", "nonblock"), 515, 8256, 512),
    (("K", "relaxed", "block"), 259, 8256, 256), (("WG", "strong", "block"), 9000, 4160, 512),
    (("WG", "relaxed", "block"), 30, 1 << 20, 512),
    (("WI", "strong", "block"), 17001, 1088, 512),     # many lanes, no helpers
    (("WI", "strong", "nonblock"), 17001, 1024, 256),  # chains
    (("WI", "strong", "block"), 40001, 576, 1024),     # more calls than slots
    (("WI", "strong", "block"), 40001, 1088, 512)])
def test_routes_match_oracle(gs, tmpdata, cell, n, item, wg):
    g, ctx = gs
    from paper_1705_06965_amd.fnv import FnvRunner
    rng = np.random.default_rng([n, item, wg])
    size = 4 << 20
    path = os.path.join(tmpdata, "routes.bin")
    rng.integers(0, 256, size, dtype=np.uint8).tofile(path)
    offs = rng.integers(0, size + 100, n).astype(np.uint64)  # some end past the end
    want, want_ret = oracle.pread_fnv(path, offs, item, threads=8)
    r = FnvRunner(ctx, path, offs, item, wg_size=wg)
    print("routes", cell, n, item, wg, flush=True)
    f, ret = r.run(*cell)
    r.close()
    assert (ret == want_ret).all() and (f == want).all()
