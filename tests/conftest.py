import os
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)


def pytest_configure(config):
    config.addinivalue_line("markers", "gpu: needs an MI355X (gfx950) GPU and the built HIP library")
    config.addinivalue_line("markers", "slow: long-running CPU test")


# Modules that load tuning entries for extents which other tests take as
# untuned.  Entries last as long as the process, so these run after the others.
LEAVES_ENTRIES = ("test_gpu_hops.py",)


def pytest_collection_modifyitems(items):
    items.sort(key=lambda item: item.path.name in LEAVES_ENTRIES)
