import os
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)


def pytest_configure(config):
    config.addinivalue_line("markers", "gpu: needs an MI355X (gfx950) GPU and the built HIP library")
    config.addinivalue_line("markers", "slow: long-running CPU test")


# Tuning entries last as long as the process: the modules that query the built-in
# rules run before any other loads entries for their extents, and the module that
# loads entries for extents which other tests take as untuned runs last.
FIRST = ("test_tune.py", "test_tune_rules.py")
LAST = ("test_gpu_hops.py",)


def pytest_collection_modifyitems(items):
    items.sort(key=lambda item: (item.path.name in LAST) - (item.path.name in FIRST))
