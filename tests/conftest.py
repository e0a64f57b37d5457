"""Shared pytest configuration: the ``gpu`` marker and common fixtures."""
import os
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)


def pytest_configure(config):
    config.addinivalue_line("markers", "gpu: needs an MI355X (gfx950) GPU and the built HIP library")


@pytest.fixture(scope="session")
def orc():
    """The CPU oracle (built on first use)."""
    import oracle
    oracle.build(force=False)
    return oracle


@pytest.fixture(scope="session")
def plan(tmp_path_factory):
    """What a Log-Int-Softmax call launches (tests/launch_plan.py)."""
    from launch_plan import Launches
    return Launches(tmp_path_factory.mktemp("plan"))
