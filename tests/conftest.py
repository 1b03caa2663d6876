import os
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)


def pytest_configure(config):
    config.addinivalue_line("markers", "gpu: needs a real MI355X (run with -m gpu)")


def load_golden(name="paper_values.txt"):
    """Parse tests/golden/<name>: 'key = value' lines, '#' comments."""
    out = {}
    with open(os.path.join(ROOT, "tests", "golden", name)) as f:
        for line in f:
            line = line.split("#", 1)[0].strip()
            if not line:
                continue
            k, v = line.split("=", 1)
            out[k.strip()] = v.strip()
    return out


@pytest.fixture(scope="session")
def golden():
    return load_golden()


@pytest.fixture(scope="session")
def stub_library(tmp_path_factory):
    """The library for the host only over a stand-in HIP runtime (see stub_library.py)."""
    import stub_library as sl
    if not os.path.exists(sl.CLANGXX):
        pytest.skip("needs the ROCm clang++")
    return sl.StubLibrary(str(tmp_path_factory.mktemp("stub")))
