"""Timed cases of the framework: GPU-issued system calls and the kernels that
consume what they return, through the Python drivers a program uses.

Kinds
  fnv       pread of n items and their FNV-1a-64 checksums (FnvRunner.run), at
            any granularity, ordering and blocking, or persistent / graph
  split     checksums of items that are already in HBM or in registered host
            memory (consume), the kernel-split form
  scan      word search over opened files (WordScanRunner.run)
  wordopen  word search that opens files by name (WordOpenRunner.run)
  files     write files, read them back and compare (FileRoundtrip)
  permute   permute 8 KiB blocks and pwrite them (PermuteRunner.run)
  serve     a queue of scan, pwrite and release jobs (ServeRun.run)
  kv        key-value GETs over loopback UDP (KVServer, loadgen)

One context serves every case, as one program would keep it: the default ring
and a service thread on all cores but four.  Files live in memory (tmpfs), as
in the benchmark, so no storage device enters.
"""
import mmap
import os
import resource
import shutil
import tempfile
import types

import numpy as np
import torch

import paper_1705_06965_amd as g
from paper_1705_06965_amd.fileio import FileRoundtrip
from paper_1705_06965_amd.fnv import FnvRunner, consume
from paper_1705_06965_amd.kv import KVServer, loadgen, make_requests
from paper_1705_06965_amd.permute import BLOCK, PermuteRunner
from paper_1705_06965_amd.serve import JOB_PWRITE, JOB_RELEASE, JOB_SCAN, ServeRun
from paper_1705_06965_amd.wordscan import WordOpenRunner, WordScanRunner

MIB = 1 << 20
ARENA_BLOCKS = 512
CELLS = ["%s/%s/%s" % c for c in g.LEGAL_CELLS]
FORMS = {"plain": g.PLAIN, "persistent": g.PERSISTENT, "graph": g.GRAPH}


def listed():
    return [
        # the smallest use of the library: 64 blocking work-item preads of
        # 4 KiB in one launch, where launch, call and checksum latency count
        dict(name="tiny", kind="fnv", n=64, item=4096, wg=64, form="plain",
             cell="WI/strong/block", ring=False, eof=False),
        # an ordinary request with a ragged item count
        dict(name="sweep_5k", kind="fnv", n=5003, item=4096, wg=256, form="persistent",
             cell="WI/strong/block", ring=False, eof=True),
        # the benchmark's headline sweep: 1 GiB in 4 KiB random preads
        dict(name="sweep_1g", kind="fnv", n=262144, item=4096, wg=256, form="graph",
             cell="WI/strong/block", ring=False, eof=False),
        # many short records, one work-item call each (the coalescing study's
        # small pieces)
        dict(name="records_256b", kind="fnv", n=16384, item=256, wg=64, form="plain",
             cell="WI/strong/block", ring=False, eof=False),
        # few long items, one work-group list call per 64 of them
        dict(name="items_64k", kind="fnv", n=1500, item=65536, wg=64, form="plain",
             cell="WG/strong/block", ring=False, eof=True),
        # checksums of data that is already on the GPU
        dict(name="split_hbm", kind="split", n=50000, item=4096, wg=256, where="hbm", eof=True),
        # the word-count corpus: 2,000 files, about 214 MiB, one pass
        dict(name="scan_2000", kind="scan", files=2000, median=65536, queries=64,
             form="persistent", passes=1),
        # a small directory searched by name: openat, read, close per file
        dict(name="wordopen_40", kind="wordopen", files=40, median=65536, queries=64,
             chunk=MIB),
        # stateful writes and reads: 64 files of 4 MiB in 1 MiB pieces
        dict(name="files_64x4m", kind="files", files=64, size=4 * MIB, piece=MIB,
             order="strong"),
        # compute, then write out: 16 MiB of blocks, 1,024 rounds, nobody waits
        dict(name="permute_16m", kind="permute", blocks=2048, iters=1024,
             cell="WG/relaxed/nonblock"),
        # a queue of 1,500 mixed jobs handed over at once
        dict(name="serve_1500", kind="serve", jobs=1500, pages_log2=12, form="persistent"),
        # 100,000 GETs from four client threads
        dict(name="kv_100k", kind="kv", keys=100000, gets=100000, clients=4, window=128,
             grid=32, batch=64, pipelined=False),
    ]


def _log(rng, lo, hi):
    return int(round(lo * (hi / lo) ** rng.random()))


def draw(rng):
    kind = rng.choice(["fnv"] * 6 + ["split"] * 2 + ["scan", "wordopen", "files", "permute",
                                                     "serve", "kv"])
    if kind == "fnv":
        form = rng.choice(["plain", "plain", "persistent", "graph"])
        cell = rng.choice(CELLS) if form == "plain" else CELLS[0]
        # 4 KiB pages are the usual item; records and long items around it
        item = 4096 if rng.random() < 0.4 else 64 * _log(rng, 1, 16384)
        most = 32 * MIB if cell.startswith("K/") else 256 * MIB
        n = _log(rng, 1, max(2, min(100000, most // item)))
        return dict(kind=kind, n=n, item=item, wg=rng.choice([64, 128, 256, 512, 1024]), form=form,
                    cell=cell, ring=form != "plain" and rng.random() < 0.3,
                    eof=rng.random() < 0.5)
    if kind == "split":
        item = 4096 if rng.random() < 0.4 else 64 * _log(rng, 1, 16384)
        where = rng.choice(["hbm", "hbm", "host"])
        n = _log(rng, 1, max(2, min(200000, 256 * MIB // item)))
        return dict(kind=kind, n=n, item=item, wg=rng.choice([64, 128, 256, 512, 1024]),
                    where=where, eof=rng.random() < 0.5)
    if kind == "scan":
        form = rng.choice(["plain", "persistent", "persistent", "graph"])
        return dict(kind=kind, files=_log(rng, 1, 300 if form == "plain" else 1500), median=rng.choice([4096, 65536]),
                    queries=rng.randint(1, 64), form=form,
                    passes=1 if form == "plain" else rng.choice([1, 1, 2, 3]))
    if kind == "wordopen":
        return dict(kind=kind, files=_log(rng, 1, 800), median=rng.choice([4096, 65536]),
                    queries=rng.randint(1, 64), chunk=64 * _log(rng, 256, 16384))
    if kind == "files":
        size = _log(rng, 1000, 4 * MIB)
        return dict(kind=kind, files=rng.randint(1, 64), size=size,
                    piece=_log(rng, max(64, size // 64), max(size, 65)),
                    order=rng.choice(["strong", "relaxed"]))
    if kind == "permute":
        return dict(kind=kind, blocks=_log(rng, 1, 4000), iters=_log(rng, 1, 1024),
                    cell=rng.choice([c for c in CELLS if c.startswith("WG")]))
    if kind == "serve":
        return dict(kind=kind, jobs=_log(rng, 20, 1500), pages_log2=rng.randint(4, 12),
                    form="persistent" if rng.random() < 0.8 else "plain")
    return dict(kind=kind, keys=_log(rng, 100, 200000), gets=_log(rng, 1000, 90000),
                clients=rng.choice([1, 2, 4]), window=rng.choice([32, 64, 128]),
                grid=rng.choice([8, 16, 32]), batch=rng.choice([64, 100, 128, 256]),
                pipelined=rng.random() < 0.5)


# ------------------------------------------------------------------- inputs

def _rng(case, seed, stream=0):
    return np.random.Generator(np.random.SFC64([seed, stream, 170506965]))


def _bytes(r, n):
    return r.integers(0, 1 << 64, (n + 7) // 8, dtype=np.uint64).view(np.uint8)[:n]


def _fnv_file(case, seed):
    """The file's bytes and the items' offsets: any byte offset, and with eof
    some items that end past the end of the file or start beyond it."""
    r = _rng(case, seed)
    n, item = case["n"], case["item"]
    size = min(max(n * item, MIB), 1 << 30)
    if case["eof"]:
        size += 777
    data = _bytes(r, size)
    if case["eof"]:
        offs = r.integers(0, size - min(item, size // 2), n, dtype=np.uint64)
        late = r.random(n) < 0.01
        offs[late] = size - item // 3 + r.integers(0, item // 2, int(late.sum()), dtype=np.uint64)
    else:
        offs = r.integers(0, size // item, n, dtype=np.uint64) * np.uint64(item)
    return data, offs


def _split_rets(case, seed):
    n, item = case["n"], case["item"]
    rets = np.full(n, item, dtype=np.int64)
    if case["eof"]:
        r = _rng(case, seed, 1)
        short = r.random(n) < 0.02
        rets[short] = r.integers(-9, item, int(short.sum()))
    return rets


def _text(case, seed):
    """(file contents, queries): Zipf words of 1..12 letters separated by
    spaces and newlines, log-normal file sizes, queries from and outside the
    vocabulary."""
    r = _rng(case, seed)
    nv = 20000
    lens = r.integers(1, 13, nv)
    letters = r.integers(97, 123, (nv, 12), dtype=np.uint8)
    vocab = [bytes(letters[i, :lens[i]]) for i in range(nv)]
    pool = 4 * MIB
    p = 1.0 / np.arange(1, nv + 1) ** 1.1
    tok = np.searchsorted(np.cumsum(p) / p.sum(), r.random(pool // 5)).clip(0, nv - 1)
    wl = lens[tok] + 1
    ends = np.cumsum(wl)
    text = np.empty(int(ends[-1]), dtype=np.uint8)
    at = np.arange(len(text)) - np.repeat(ends - wl, wl)
    text[:] = letters[np.repeat(tok, wl), np.minimum(at, 11)]
    text[ends - 1] = np.where(r.random(len(tok)) < 0.1, 10, 32)
    sizes = np.exp(np.log(case["median"]) + r.standard_normal(case["files"]))
    sizes = np.clip(sizes, 1, min(8 * MIB, len(text) - 1)).astype(np.int64)
    starts = (r.random(case["files"]) * (len(text) - sizes)).astype(np.int64)
    files = [text[a:a + s] for a, s in zip(starts, sizes)]
    pick = list(dict.fromkeys(vocab[i] for i in
                              np.concatenate([np.arange(40), r.permutation(nv)[:200]])))
    queries = pick[:case["queries"]]
    if len(queries) > 4:
        queries[-1] = b"Absent"
    return files, queries


def _jobs(case, seed, scan_bytes):
    """The case fixes each job's kind and length, the seed the ranges read and
    the bytes written."""
    n = case["jobs"]
    r = np.random.default_rng([n, case["pages_log2"]])
    u = r.random(n)
    kind = np.where(u < 0.1, JOB_SCAN, np.where(u < 0.7, JOB_PWRITE, JOB_RELEASE)).astype(np.uint8)
    scan = np.round(2.0 ** r.uniform(0, case["pages_log2"], n)).astype(np.uint64)
    wr = np.round(2.0 ** r.uniform(0, 6, n)).astype(np.uint64)
    r = _rng(case, seed, 2)
    first = (r.random(n) * (scan_bytes // 4096 - scan.astype(np.int64) + 1)).astype(np.uint64)
    off, ln, con = (np.zeros(n, dtype=np.uint64) for _ in range(3))
    s, w, rel = kind == JOB_SCAN, kind == JOB_PWRITE, kind == JOB_RELEASE
    off[s], ln[s] = first[s] * 4096, scan[s] * 4096
    ln[w] = wr[w] * 4096
    off[w] = np.cumsum(ln[w]) - ln[w]
    con[w] = off[w]
    off[rel] = np.arange(int(rel.sum())) % ARENA_BLOCKS
    ln[rel] = 2 * MIB
    return types.SimpleNamespace(kind=kind, arrival_ns=np.zeros(n, dtype=np.uint64), arg_off=off,
                                 arg_len=ln, content_off=con,
                                 content=_bytes(r, int(ln[w].sum())).copy())


def _scan_bytes(case):
    return max(4 * MIB, min(256 * MIB, 16 << (12 + case["pages_log2"])))


def _kv_inputs(case, seed):
    r = _rng(case, seed)
    n = case["keys"]
    keys = _bytes(r, 16 * n).reshape(n, 16).copy()
    keys[:, :8] = np.arange(n, dtype=np.uint64).view(np.uint8).reshape(n, 8)  # distinct
    vlen = r.integers(32, 1025, n, dtype=np.uint32)
    voff = (np.cumsum(vlen) - vlen).astype(np.uint64)
    heap = _bytes(r, int(vlen.sum()))
    p = 1.0 / np.arange(1, n + 1) ** 0.99
    rank = np.searchsorted(np.cumsum(p) / p.sum(), r.random(case["gets"])).clip(0, n - 1)
    want = keys[r.permutation(n)[rank]].copy()
    want[::64, 15] ^= 0xFF  # misses
    return keys, voff, vlen, heap, want


# -------------------------------------------------------------------- state

_ctx = None


def _context():
    global _ctx
    if _ctx is None:
        soft, hard = resource.getrlimit(resource.RLIMIT_NOFILE)
        resource.setrlimit(resource.RLIMIT_NOFILE, (min(hard, 60000), hard))
        _ctx = g.Context(service_threads=max(1, len(os.sched_getaffinity(0)) - 4),
                         arena_bytes=ARENA_BLOCKS * 2 * MIB, device_timeout_ns=20_000_000_000)
    return _ctx


class _State:
    """What a program holds for one case; everything is given back when it goes."""

    def __init__(self, case):
        self.case = case
        self.ctx = _context()
        self.fds, self.undo, self.folder = [], [], None

    def memory_file(self, data=None, size=0):
        fd = os.memfd_create("gsys_case")
        self.fds.append(fd)
        if data is not None:
            view = memoryview(data)
            while len(view):
                view = view[os.write(fd, view[:1 << 30]):]
        elif size:
            os.ftruncate(fd, size)
        return fd, "/proc/self/fd/%d" % fd

    def directory(self):
        base = "/dev/shm"
        for old in os.listdir(base):  # left by a process that was killed
            if old.startswith("gsys_case_") and not os.path.exists("/proc/" + old.split("_")[2]):
                shutil.rmtree(os.path.join(base, old), ignore_errors=True)
        self.folder = tempfile.mkdtemp(prefix="gsys_case_%d_" % os.getpid(), dir=base)
        return self.folder

    def close(self):
        for f in self.undo:
            f()
        for fd in self.fds:
            os.close(fd)
        if self.folder:
            shutil.rmtree(self.folder, ignore_errors=True)
        self.fds, self.undo, self.folder = [], [], None

    def __del__(self):
        self.close()


class _Held(np.ndarray):
    """A view of a state's registered buffer; it keeps the state."""


def _write_files(folder, files):
    names = ["f%05d.txt" % i for i in range(len(files))]
    for name, data in zip(names, files):
        with open(os.path.join(folder, name), "wb") as f:
            f.write(data)
    return names


def prepare(case, seed):
    s = _State(case)
    ctx, kind = s.ctx, case["kind"]
    if kind == "fnv":
        data, offs = _fnv_file(case, seed)
        _, path = s.memory_file(data)
        ring = 0  # a staging ring of 16 or 1 work-groups' batches where that is smaller
        if case["ring"]:
            pair = 2 * case["wg"] * case["item"]
            ring = next((k * pair for k in (16, 1) if k * pair < case["n"] * case["item"]), 0)
        s.r = FnvRunner(ctx, path, offs, case["item"], case["wg"], staging_bytes=ring)
        s.undo.append(s.r.close)
    elif kind == "split":
        n, item = case["n"], case["item"]
        data = _bytes(_rng(case, seed), n * item)
        if case["where"] == "hbm":
            s.items = torch.from_numpy(data).to("cuda")
            s.addr = s.items.data_ptr()
        else:
            s.buf = ctx.host_alloc(n * item)
            s.buf.array[:] = data
            s.addr = s.buf.dev
            s.undo.append(s.buf.free)
        s.rets = torch.from_numpy(_split_rets(case, seed)).to("cuda")
        s.out = torch.zeros(n, dtype=torch.int64, device="cuda")
    elif kind in ("scan", "wordopen"):
        files, queries = _text(case, seed)
        folder = s.directory()
        names = _write_files(folder, files)
        if kind == "scan":
            s.r = WordScanRunner(ctx, [os.path.join(folder, x) for x in names], queries)
            r = s.r
            s.undo += [r.close, r.staging_p.free,
                       lambda: r.staging_w is not None and r.staging_w.free()]
        else:
            s.r = WordOpenRunner(ctx, folder, names, queries, chunk=case["chunk"], groups=64)
            s.undo.append(s.r.close)
    elif kind == "files":
        names = ["w%03d.bin" % i for i in range(case["files"])]
        s.r = FileRoundtrip(ctx, s.directory(), names)
        data = _bytes(_rng(case, seed), case["files"] * case["size"])
        s.r.prepare(data.reshape(case["files"], case["size"]), case["piece"])
        s.undo.append(s.r.close)
    elif kind == "permute":
        r = _rng(case, seed)
        data = _bytes(r, case["blocks"] * BLOCK).view(np.uint64)
        fd, path = s.memory_file(size=case["blocks"] * BLOCK)
        s.r = PermuteRunner(ctx, path, data, r.permutation(1024), r.permutation(64))
        s.out = np.frombuffer(mmap.mmap(fd, case["blocks"] * BLOCK), dtype=np.uint8)
        s.undo.append(s.r.close)
    elif kind == "serve":
        size = _scan_bytes(case)
        _, path = s.memory_file(_bytes(_rng(case, seed), size))
        fd, out = s.memory_file()
        s.r = ServeRun(ctx, _jobs(case, seed, size), path, out, arena_blocks=ARENA_BLOCKS)
        r = s.r
        size = r.release_base + 128 * int((r.js.kind == JOB_RELEASE).sum())
        os.ftruncate(fd, max(size, 1))
        s.out = np.frombuffer(mmap.mmap(fd, max(size, 1)), dtype=np.uint8)
        r.params(FORMS[case["form"]], staging_bytes=128 * MIB)
        s.undo += [r.close, r.jobs.free, r.staging.free]
    else:
        keys, voff, vlen, heap, want = _kv_inputs(case, seed)
        s.r = KVServer(ctx, keys, voff, vlen, heap, grid=case["grid"], batch=case["batch"],
                       pipelined=case["pipelined"])
        s.reqs = make_requests(want)
        r = s.r
        s.undo += [r.close, r.io.free, r.ctl.free]
    return s


def run(s):
    case, r = s.case, getattr(s, "r", None)
    kind = case["kind"]
    if kind == "fnv":
        f, ret = r.run(*case["cell"].split("/"), form=FORMS[case["form"]])
        return f.view(np.int64), ret
    if kind == "split":
        consume(s.ctx, s.addr, s.rets, case["item"], s.out, case["wg"])
        return s.out
    if kind == "scan":
        return r.run(FORMS[case["form"]], passes=case["passes"]).view(np.int32)
    if kind == "wordopen":
        counts, ret = r.run()
        return counts.view(np.int32), ret
    if kind == "files":
        r.launch(case["order"])
        torch.cuda.synchronize()
        if s.ctx.wait(60_000_000_000):
            raise RuntimeError("drain failed")
        back = r.staging.array[:r.need].reshape(case["files"], 2 * r.a)[:, r.a:r.a + r.fb]
        back = back.view(_Held)
        back.owner = s
        # every result but the two opens' descriptor numbers
        return r.rets[:, 1:r.k + 2], r.rets[:, r.k + 3:], r.mism, back
    if kind == "permute":
        return r.run(case["iters"], *case["cell"].split("/")), s.out
    if kind == "serve":
        res, dig, _ = r.run(FORMS[case["form"]], staging_bytes=128 * MIB)
        return res, dig.view(np.int64), s.out
    r.start()
    got, replies, rlen, _, _ = loadgen(r.port, s.reqs, case["clients"], case["window"])
    r.stop()
    if got != case["gets"]:
        raise RuntimeError("%d of %d GETs answered" % (got, case["gets"]))
    return replies, rlen.view(np.int32)


# -------------------------------------------------------------- what it costs

def work(case):
    """Every byte that has to be read or written once (payload, tables and
    results; a file's write and its read back count one each)."""
    kind = case["kind"]
    if kind == "fnv":
        return {"bytes": case["n"] * (case["item"] + 24), "flops": 0}
    if kind == "split":
        return {"bytes": case["n"] * (case["item"] + 16), "flops": 0}
    if kind in ("scan", "wordopen"):
        total = case["files"] * case["median"] * 1.6  # mean of the log-normal sizes
        out = case["files"] * case["queries"] * 4
        return {"bytes": total * case.get("passes", 1) + out, "flops": 0}
    if kind == "files":
        return {"bytes": 2 * case["files"] * case["size"], "flops": 0}
    if kind == "permute":
        return {"bytes": 2 * case["blocks"] * BLOCK, "flops": 0}
    if kind == "serve":
        pages = 2 ** case["pages_log2"] / max(1.0, case["pages_log2"] * 0.693)
        return {"bytes": case["jobs"] * (0.1 * pages * 4096 + 0.6 * 2 * 15 * 4096 +
                                         0.3 * 2 * MIB), "flops": 0}
    return {"bytes": case["gets"] * (32 + 16 + 528 * 2), "flops": 0}


# ------------------------------------------------------------------- checks

def _fnv(rows, lens):
    """FNV-1a-64 of the first lens[i] bytes of each row of a byte matrix."""
    h = np.full(len(rows), 0xcbf29ce484222325, dtype=np.uint64)
    p = np.uint64(0x100000001b3)
    short = bool((lens < rows.shape[1]).any())
    step = max(1, min(rows.shape[1], (64 << 20) // max(1, len(rows))))
    for a in range(0, rows.shape[1], step):
        cols = np.ascontiguousarray(rows[:, a:a + step].T).astype(np.uint64)
        for k in range(len(cols)):
            v = (h ^ cols[k]) * p
            h = np.where(a + k < lens, v, h) if short else v
    return h.view(np.int64)


def _word_counts(files, queries, passes=1):
    out = np.zeros((len(files), len(queries)), dtype=np.int32)
    at = {q: i for i, q in enumerate(queries)}
    for f, data in enumerate(files):
        for w in bytes(data).replace(b"\n", b" ").split(b" "):
            i = at.get(w)
            if i is not None:
                out[f, i] += passes
    return out


def _permuted(case, seed):
    r = _rng(case, seed)
    x = _bytes(r, case["blocks"] * BLOCK).view(np.uint64).reshape(-1, 1024)
    sigma, tau = r.permutation(1024), r.permutation(64)
    s, t = np.arange(1024), np.arange(64)
    for _ in range(case["iters"]):  # both shuffles composed, then applied once
        s, t = s[sigma], t[tau]
    x = np.ascontiguousarray(x[:, s])
    y = np.zeros_like(x)
    for j in range(64):
        y |= ((x >> np.uint64(t[j])) & np.uint64(1)) << np.uint64(j)
    return y.view(np.uint8).reshape(-1)


def exact(case, seed):
    kind = case["kind"]
    if kind in ("fnv", "split") and case["n"] * case["item"] > 256 * MIB:
        return None
    if kind == "fnv":
        data, offs = _fnv_file(case, seed)
        n, item = case["n"], case["item"]
        lens = np.clip(len(data) - offs.astype(np.int64), 0, item)
        rows = np.zeros((n, item), dtype=np.uint8)
        for i in range(n):
            rows[i, :lens[i]] = data[int(offs[i]):int(offs[i]) + int(lens[i])]
        return _fnv(rows, lens), lens
    if kind == "split":
        data = _bytes(_rng(case, seed), case["n"] * case["item"]).reshape(case["n"], case["item"])
        return _fnv(data, _split_rets(case, seed))
    if kind == "scan":
        files, queries = _text(case, seed)
        if sum(map(len, files)) > 64 * MIB:
            return None
        return _word_counts(files, queries, case["passes"])
    if kind == "wordopen":
        files, queries = _text(case, seed)
        if sum(map(len, files)) > 64 * MIB:
            return None
        return _word_counts(files, queries), np.array([len(f) for f in files], dtype=np.int64)
    if kind == "files":
        data = _bytes(_rng(case, seed), case["files"] * case["size"])
        return None, None, np.zeros(case["files"], dtype=np.int64), data.reshape(case["files"], -1)
    if kind == "permute":
        blocking = case["cell"].endswith("/block")
        ret = np.full(case["blocks"], BLOCK if blocking else g.NOT_WAITED, dtype=np.int64)
        return ret, _permuted(case, seed)
    if kind == "serve":
        size = _scan_bytes(case)
        data = _bytes(_rng(case, seed), size)
        js = _jobs(case, seed, size)
        s, w = js.kind == JOB_SCAN, js.kind == JOB_PWRITE
        res = np.where(s | w, js.arg_len, 0).astype(np.int64)
        if int(js.arg_len[s].sum()) > 256 * MIB:
            return res, None, None
        if not s.any():
            return res, np.zeros(1, dtype=np.int64), None
        rows = np.concatenate([data[int(o):int(o + l)] for o, l in
                               zip(js.arg_off[s], js.arg_len[s])]).reshape(-1, 4096)
        return res, _fnv(rows, np.full(len(rows), 4096)), None
    keys, voff, vlen, heap, want = _kv_inputs(case, seed)
    at = {bytes(k): i for i, k in enumerate(keys)}
    replies = np.zeros((case["gets"], 1040), dtype=np.uint8)
    replies[:, :8] = np.arange(1, case["gets"] + 1, dtype=np.uint64).view(np.uint8).reshape(-1, 8)
    rlen = np.full(case["gets"], 16, dtype=np.int32)
    for k, key in enumerate(want):
        i = at.get(bytes(key))
        replies[k, 8] = i is None
        if i is not None:
            ln = int(vlen[i])
            replies[k, 10:12] = np.array([ln], dtype=np.uint16).view(np.uint8)
            replies[k, 16:16 + ln] = heap[int(voff[i]):int(voff[i]) + ln]
            rlen[k] += ln
    return replies, rlen
