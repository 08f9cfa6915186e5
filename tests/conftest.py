import os
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)


def pytest_configure(config):
    config.addinivalue_line("markers", "gpu: needs an MI355X (gfx950) GPU")
    config.addinivalue_line("markers", "slow: long CPU test")


@pytest.fixture(scope="session")
def tmpdata(tmp_path_factory):
    """A private tmpfs-backed data directory for files a test creates."""
    base = "/dev/shm" if os.path.isdir("/dev/shm") else None
    import tempfile
    d = tempfile.mkdtemp(prefix="gsys_test_", dir=base)
    yield d
    import shutil
    shutil.rmtree(d, ignore_errors=True)


POISON = -54321


def poison(runner):
    """Fill a driver's result tensors, and the pinned copies it returns them
    through, with a value that no call returns."""
    import torch
    for t in runner.back.src:
        t.fill_(POISON)
    for t in runner.back.dst or ():
        t.fill_(POISON)
    torch.cuda.synchronize()


@pytest.fixture(autouse=True)
def poisoned_outputs(request, monkeypatch):
    """The drivers keep their result tensors from one run() to the next and do
    not clear them, so a result that a launch does not store would read as the
    run before's, which is often the right answer.  Every run() that a GPU
    test makes starts from poisoned results."""
    if request.node.get_closest_marker("gpu"):
        from paper_1705_06965_amd.fnv import FnvRunner
        from paper_1705_06965_amd.permute import PermuteRunner
        from paper_1705_06965_amd.wordscan import WordOpenRunner, WordScanRunner
        for cls in (FnvRunner, PermuteRunner, WordOpenRunner, WordScanRunner):
            def run(self, *a, _run=cls.run, **k):
                poison(self)
                return _run(self, *a, **k)
            monkeypatch.setattr(cls, "run", run)
    yield
