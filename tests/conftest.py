import os
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)


@pytest.fixture(params=["as dispatched", "two launches"])
def decode_form(request, monkeypatch):
    """Runs a test twice: with the decode form the library picks, and with small steps kept in the two-launch
    form that all larger ones use."""
    from gpu_util import DeviceCase
    monkeypatch.setattr(DeviceCase, "two_launches", request.param == "two launches")
    return request.param


def pytest_configure(config):
    config.addinivalue_line("markers", "gpu: needs a real MI355X (run with -m gpu)")
