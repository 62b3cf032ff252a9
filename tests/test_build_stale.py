"""A library older than anything that it is made from, the compiler's flags among them, is built again."""
import os

import pytest

from paper_2603_06664_amd import build


@pytest.mark.parametrize("newer", ["build.py", "crope.h", "attention.hip", "crope_internal.h", None])
def test_stale(monkeypatch, newer):
    monkeypatch.setattr(os.path, "exists", lambda p: True)
    monkeypatch.setattr(os.path, "getmtime", lambda p: 20.0 if p.endswith(".so") else 30.0 if os.path.basename(p) == newer else 10.0)
    assert build._stale() == (newer is not None)
