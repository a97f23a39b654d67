"""The native module that marshals arguments against the same through ctypes: statuses and refusals (no GPU needed: nothing is launched); and what
happens where it cannot be built or loaded."""
import os
import subprocess
import sys
import warnings

import pytest
import torch

from paper_1909_08053_amd import binding as B
from paper_1909_08053_amd import build as BLD

D = B.make_dims(1, 8, 64, 1, 64, 64, 1, 0, B.MLM_BF16)
DROP = B.make_dropout(0.1, 1, 2)
CPU = torch.zeros(8)
CALLS = [
    ("mlm_deferred_sums_flush", (7,)), ("mlm_deferred_sums_begin", (None,)), ("mlm_combine", (D, [], None, None, None, 0)),
    ("mlm_combine", (D, (CPU,), None, None, None, 0)), ("mlm_layernorm_fwd", (D, None, None, None, None, None, None, 0)),
    ("mlm_layernorm_fwd", (D, CPU, None, None, None, None, None, 0)), ("mlm_vocab_ce_merge", (D, None, None, None, 1, None, None, None, None, None, 0)),
    ("mlm_mlp_shard_fwd", (D, None, None, None, None, None, None, None, None, 0)), ("mlm_combine_dropout", (D, [], None, 1, DROP, None, None, 0)),
    ("mlm_embed_bwd_replicated", (D, None, DROP, None, None, 0)), ("mlm_rows_gather", (D, None, None, 1, 2, None, 0)),
]


def outcome(f, args):
    try:
        return f(*args)
    except Exception as e:
        return type(e), str(e)


def native():
    """Not built is a reason to skip; built and not loaded is not."""
    if isinstance(B._call, B._Marshalled):
        assert not os.path.exists(BLD.MODULE), "the native module is built and was not loaded"
        pytest.skip("the native module is not built")


@pytest.mark.parametrize("name,args", CALLS, ids=[f"{n}-{i}" for i, (n, _) in enumerate(CALLS)])
def test_native_marshalling_is_that_of_ctypes(name, args):
    native()
    got, want = outcome(getattr(B._call, name), args), outcome(B._marshalled(name), args)
    assert got == want and got != 0


@pytest.mark.parametrize("args", [(), (D,), (D, None, None, None, None, None, None, 0, 0), (None, None, None, None, None, None, None, 0),
                                  (DROP, None, None, None, None, None, None, 0), (D, 3.5, None, None, None, None, None, 0)])
def test_wrong_arguments_are_refused(args):
    native()
    with pytest.raises(TypeError):
        B._call.mlm_layernorm_fwd(*args)


def test_module_that_cannot_be_built_leaves_the_library(tmp_path, monkeypatch, capsys):
    """No torch headers, say: the library is linked, an older module goes, and a message says what the calls will take."""
    def no_module():
        raise ImportError("no torch")
    monkeypatch.setattr(BLD, "SOURCES", [])
    monkeypatch.setattr(BLD, "OBJ", str(tmp_path))
    monkeypatch.setattr(BLD, "LIB", str(tmp_path / "lib.so"))
    monkeypatch.setattr(BLD, "MODULE", str(tmp_path / "_mlm_call.so"))
    monkeypatch.setattr(BLD, "_module", no_module)
    monkeypatch.setattr(BLD.subprocess, "run", lambda *a, **k: subprocess.CompletedProcess(a, 0, "", ""))
    (tmp_path / "_mlm_call.so").write_text("older")
    assert BLD.build(verbose=False) == str(tmp_path / "lib.so")
    assert not (tmp_path / "_mlm_call.so").exists()
    assert "ctypes: no torch" in capsys.readouterr().err


def test_module_that_cannot_be_loaded_is_said_once(monkeypatch):
    """ctypes takes its place, with a warning where there is a library to call."""
    monkeypatch.setitem(sys.modules, "paper_1909_08053_amd._mlm_call", None)
    monkeypatch.delattr(sys.modules["paper_1909_08053_amd"], "_mlm_call", raising=False)
    monkeypatch.setattr(B, "LIB_PATH", __file__)
    with pytest.warns(RuntimeWarning, match="through ctypes") as said:
        assert isinstance(B._load(), B._Marshalled)
    assert len(said) == 1
    monkeypatch.setattr(B, "LIB_PATH", __file__ + ".absent")
    with warnings.catch_warnings():
        warnings.simplefilter("error")
        assert isinstance(B._load(), B._Marshalled)
