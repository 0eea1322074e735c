"""No library source captures a stream: while one does, another thread's wait for the
whole device is refused and ends the capture."""
import os

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1509_08267_amd", "csrc")


@pytest.mark.parametrize("name", sorted(f for f in os.listdir(CSRC) if f.endswith((".hip", ".h"))))
def test_source_begins_no_capture(name):
    with open(os.path.join(CSRC, name)) as f:
        assert "hipStreamBeginCapture" not in f.read()
