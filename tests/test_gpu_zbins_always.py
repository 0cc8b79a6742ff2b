"""The cases of test_gpu_zbins with CPM_SF_ZBIN=2: small systems and batches take the
sums over binned charges also where explicit structure factors would cost less.
"""
import pytest

from test_gpu_zbins import *            # noqa: F401,F403
from test_gpu_zbins import cpm, pytestmark  # noqa: F401


@pytest.fixture(autouse=True)
def always_binned(monkeypatch):
    monkeypatch.setenv("CPM_SF_ZBIN", "2")
