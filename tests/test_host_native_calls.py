"""Which torch the binding's native calls are taken for: the one that they were built with, and no other."""
import sys

import torch

import paper_1608_01409_amd
from paper_1608_01409_amd import binding as B


def test_built_for_this_torch():
    calls = B._native_calls(torch)
    assert calls is not None and calls.torch_version == str(torch.__version__)


def test_built_for_another_torch_or_not_at_all(monkeypatch):
    """The Python lines then serve every call."""
    B._native_calls(torch)
    module = sys.modules["paper_1608_01409_amd._sconv_call"]
    monkeypatch.setattr(module, "torch_version", "0.0")
    assert B._native_calls(torch) is None
    monkeypatch.delattr(module, "torch_version")
    assert B._native_calls(torch) is None
    monkeypatch.delattr(paper_1608_01409_amd, "_sconv_call")
    monkeypatch.setitem(sys.modules, "paper_1608_01409_amd._sconv_call", None)   # what an import that fails looks like
    assert B._native_calls(torch) is None
