import os
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)


def pytest_configure(config):
    config.addinivalue_line("markers", "gpu: needs a real MI355X (run with -m gpu)")


@pytest.fixture(params=["computed", "callers"])
def grid(request, monkeypatch):
    """The test runs on the windows that calls compute, then with every handle held to the caller's own windows: several in a launch, with
    joins, ragged last ones, cuts between groups inside a clip."""
    if request.param == "callers":
        import paper_2605_28657_amd as pa
        for cls in (pa.DemonVAE, pa.DemonVAEEncoder):
            def init(self, *args, _made=cls.__init__, **kw):
                _made(self, *args, **kw)
                self.callers_grid(True)
            monkeypatch.setattr(cls, "__init__", init)
    return request.param


def pytest_collection_modifyitems(config, items):
    # GPU tests are skipped, not failed, when collected on a machine without a GPU
    # and no marker expression was given.
    if config.getoption("-m"):
        return
    try:
        import torch
        has_gpu = torch.cuda.is_available()
    except Exception:
        has_gpu = False
    if has_gpu:
        return
    skip = pytest.mark.skip(reason="no GPU")
    for it in items:
        if "gpu" in it.keywords:
            it.add_marker(skip)
