"""The Python binding on its own (no GPU): which libraries it accepts, and what it asks of
torch and of the library in calls that a GPU test could only catch by chance."""
import ctypes

import pytest


def _vclb():
    from paper_2505_10899_amd import vclb
    return vclb


class _Fn:
    def __init__(self, result=0):
        self.result = result

    def __call__(self, *a):
        return self.result


class _OldLibrary:
    """A library of an earlier minor version: no entry points but these."""

    def __init__(self, version):
        self.vclb_version = _Fn(version)
        self.vclb_strerror = _Fn(b"")


@pytest.mark.parametrize("version", [20100, 10000, 30000])
def test_other_version_is_refused_by_its_number(monkeypatch, version):
    """Not by the first symbol that it lacks."""
    v = _vclb()
    monkeypatch.setattr(v, "_lib", None)
    monkeypatch.setattr(ctypes, "CDLL", lambda path: _OldLibrary(version))
    with pytest.raises(ImportError, match=str(version)):
        v.lib()


def test_adjoint_store_came_with_a_new_minor_version():
    v = _vclb()
    assert "vclb_adjoint_set_store" in v.exported_symbols()
    assert v.lib().vclb_version() == v.VERSION >= 20200
