import os
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)

# Passes of 9 to 32 rows of wide models are one kernel wherever there is one for them: the hidden states of the tests' models are too
# narrow for the library's own choice (read when a state is created).
os.environ.setdefault("BILD_WIDE_ROWS", "32")


def pytest_configure(config):
    config.addinivalue_line("markers", "gpu: needs a real MI355X (run with -m gpu)")
