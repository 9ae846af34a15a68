"""build.is_stale(): a library older than its sources, its headers or the file
that holds the compiler flags is reported as stale."""
import os

import pytest

from paper_2606_26344_amd import build


@pytest.fixture
def times(monkeypatch):
    t = {f: 100.0 for f in [build.__file__, build.MFMA_CEILING_SOURCE] + build.SOURCES + build.HEADERS}
    t.update({build.LIBRARY: 200.0, build.MFMA_CEILING: 200.0})
    monkeypatch.setattr(os.path, "getmtime", lambda f: t[f])
    monkeypatch.setattr(os.path, "exists", lambda f: f in t)
    return t


def test_fresh(times):
    assert not build.is_stale()


def test_each_input_and_output(times):
    for f in list(times):
        was = times[f]
        times[f] = 150.0 if f in (build.LIBRARY, build.MFMA_CEILING) else 300.0
        assert build.is_stale() == (was == 100.0), f
        times[f] = was
    for f in (build.LIBRARY, build.MFMA_CEILING):
        was = times.pop(f)
        assert build.is_stale(), f
        times[f] = was
