import gc
import os
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)


def pytest_configure(config):
    config.addinivalue_line("markers", "gpu: needs a real MI355X (run with -m gpu)")


def pytest_runtest_setup(item):
    # A test that counts allocated device memory around a call: garbage that earlier tests left in reference
    # cycles goes before it, not by a collection that happens to start between its two counts.
    if item.path.name == "test_zz_no_alloc.py":
        gc.collect()
