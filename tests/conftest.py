import os
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)


def pytest_configure(config):
    config.addinivalue_line("markers", "gpu: needs a real MI355X (run with -m gpu where there is one)")


@pytest.fixture(scope="session")
def oracle():
    from oracle import specee_oracle
    specee_oracle.build()
    return specee_oracle
