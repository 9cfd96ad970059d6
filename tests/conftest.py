import gc
import os
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)


def pytest_configure(config):
    config.addinivalue_line("markers", "gpu: needs a real MI355X (run with -m gpu)")


@pytest.fixture(autouse=True)
def _tensors_of_earlier_tests_are_gone(request):
    """Tests that compare torch.cuda.memory_allocated() before and after a call: tensors in reference cycles (the frames an
    exception keeps) must not be collected in between."""
    if request.module.__name__.endswith("no_alloc"):
        gc.collect()
