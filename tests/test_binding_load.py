"""Loading the binding where only the library was built."""
import sys

import pytest

import paper_2506_04985_amd
from paper_2506_04985_amd import binding as fptq


def test_the_library_serves_without_the_native_fast_path(monkeypatch):
    monkeypatch.setattr(fptq, "_lib", None)
    monkeypatch.setattr(fptq, "_native", None)
    monkeypatch.delattr(paper_2506_04985_amd, "_native", raising=False)
    monkeypatch.setitem(sys.modules, "paper_2506_04985_amd._native", None)       # importing it raises ImportError
    with pytest.warns(RuntimeWarning, match="native fast path"):
        fptq.lib()
    assert fptq._native is None and fptq.fptq_packed_bytes(10, 129) == 1280
    with pytest.raises(fptq.FptqError):
        fptq.fptq_packed_bytes(0, 1)
