"""The native marshalling is optional: without a binding that was built from
these sources for the torch that runs, the Python code takes every call."""
import importlib

import pytest
import torch

import paper_2608_03447_amd as asd
from paper_2608_03447_amd import build


def _missing(monkeypatch):
    monkeypatch.setattr(asd, "BINDING", asd.BINDING + ".missing")


def _unloadable(monkeypatch):
    def fails(name, package=None):
        raise ImportError("undefined symbol: _ZN2at")
    monkeypatch.setattr(importlib, "import_module", fails)


def _stale(monkeypatch):
    monkeypatch.setattr(asd, "binding_hash", lambda: "0123456789abcdef")


@pytest.mark.parametrize("fault", [_missing, _unloadable, _stale])
def test_without_a_usable_binding_the_python_code_takes_the_calls(fault, monkeypatch):
    monkeypatch.setattr(asd, "_fast", None)
    fault(monkeypatch)
    with pytest.warns(RuntimeWarning, match="Python marshalling"):
        fast = asd._load_fast()
    assert fast is asd._fast
    for name in ("verify", "verify_static", "verify_ex", "verify_commit", "verify_partials",
                 "lmhead_verify", "shard_argmax", "opportunity"):
        assert getattr(fast, name)(1, 2, 3) is None
    with pytest.raises(RuntimeError, match="build"):
        asd._load_binding()


def test_the_built_binding_loads_and_its_hash_names_the_torch(monkeypatch):
    assert asd._load_binding().source_hash() == build.binding_hash()
    now = build.binding_hash()
    monkeypatch.setattr(torch, "__version__", "0.0.0")
    assert build.binding_hash() != now
