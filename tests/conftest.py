import os
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)


def pytest_configure(config):
    config.addinivalue_line("markers", "gpu: needs an MI355X (gfx950) GPU")
    config.addinivalue_line("markers", "slow: long CPU test")


def pytest_collection_modifyitems(items):
    # uses up the process's look-back slots for long scans: the tests of other
    # files come before it and run with a slot
    items.sort(key=lambda item: item.path.name == "test_gpu_scan_long_slots.py")
