"""The native part of the Python binding is a shortcut: without it, or with
one built against another torch (whose objects it would misread), the checks
in Python run instead, with a warning (no GPU)."""
from __future__ import annotations

import ctypes

import pytest

import paper_2603_11438_amd as ar


@pytest.fixture
def fresh(monkeypatch):
    monkeypatch.setattr(ar, "_native_path", None)
    return monkeypatch


def _plan():
    """A plan's Python side alone (no device)."""
    p = object.__new__(ar.Plan)
    p._h = ctypes.c_void_p(0)
    p.info = {"nranks": 2, "count": 8, "coll": ar.AR_COLL_ALLREDUCE, "dtype": ar.AR_FLOAT32}
    p._expect = (2, 8, 8, 0)
    return p


def _refused_in_python():
    import torch

    ts = [torch.ones(8), torch.ones(8)]
    with pytest.raises(ValueError):
        ar.run_noalloc(ts)
    plan = _plan()
    for call in (lambda: plan.run(ts), lambda: plan.run_oop(ts, ts), lambda: plan.bind(ts)):
        with pytest.raises(ValueError):
            call()


def test_built_against_the_loaded_torch(fresh):
    import torch

    native = ar._native()
    assert native is not None and native.torch_version == str(torch.__version__)
    _refused_in_python()


def test_not_built(fresh, tmp_path):
    fresh.setattr(ar, "TENSOR_ARGS_PATH", str(tmp_path / "absent.so"))
    with pytest.warns(RuntimeWarning, match="not built"):
        assert ar._native() is None
    _refused_in_python()


def test_built_against_another_torch(fresh):
    import torch

    fresh.setattr(torch, "__version__", "0.0.1")
    with pytest.warns(RuntimeWarning, match="0.0.1"):
        assert ar._native() is None
    _refused_in_python()


def test_cannot_be_loaded(fresh, tmp_path):
    bad = tmp_path / "_tensor_args.so"
    bad.write_bytes(b"not a library")
    fresh.setattr(ar, "TENSOR_ARGS_PATH", str(bad))
    with pytest.warns(RuntimeWarning):
        assert ar._native() is None
    _refused_in_python()
