import sys
from pathlib import Path

import pytest

ROOT = Path(__file__).resolve().parent.parent
if str(ROOT) not in sys.path:
    sys.path.insert(0, str(ROOT))


def pytest_configure(config):
    config.addinivalue_line("markers", "gpu: needs a real MI355X (run with -m gpu)")


@pytest.fixture(params=["rule", "table"])
def accept_tables(request):
    """Accept calls as the library routes them, and with a table of masses wherever one is possible (a hook of the benchmark
    library, whose kernels are the product's): the rule gives tables only to calls too large for most tests."""
    from paper_2506_19830_amd import binding as B
    if request.param == "rule":
        yield request.param
        return
    B.select_library("bench")
    B.la_selftest_force_table(True)
    try:
        yield request.param
    finally:
        B.la_selftest_force_table(False)
        B.select_library("product")


@pytest.fixture(scope="session")
def oracle():
    import oracle as _oracle
    _oracle.build()
    return _oracle
