import os
import re
import sys
import warnings

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)


def pytest_configure(config):
    config.addinivalue_line("markers", "gpu: needs a real MI355X (run with -m gpu)")


@pytest.fixture(scope="session")
def hippo():
    """The HIP library's Python binding; GPU tests fail loudly if it cannot be loaded."""
    import paper_2601_08273_amd as h
    h.load()
    return h


@pytest.fixture
def kernels(tmp_path):
    """The (mangled) names of the kernels that a call launches, in launch order: which route it takes."""
    import torch

    def names(call):
        call()
        graph = torch.cuda.CUDAGraph(keep_graph=True)
        graph.enable_debug_mode()
        with torch.cuda.graph(graph):
            call()
        path = str(tmp_path / "graph.dot")
        with warnings.catch_warnings():
            warnings.simplefilter("ignore")                 # it says that it was called
            graph.debug_dump(path)
        with open(path) as f:
            return [name for _, name in sorted((int(i), name) for i, name in re.findall(r"\{ID \| (\d+) \| (\w+)", f.read()))]

    return names
