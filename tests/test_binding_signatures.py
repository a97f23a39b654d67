"""Argument types that the binding declares, against the prototypes of include/mlm_shard.h, and the stream it passes (no GPU needed)."""
import os
import re
import types

import pytest
import torch

from paper_1909_08053_amd import binding as B

HEADER = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "include", "mlm_shard.h")
SCALAR = {"int": "i", "int32_t": "i", "int64_t": "l", "uint64_t": "u", "size_t": "z", "float": "f"}


def test_declared_types_are_the_headers():
    text = re.sub(r"/\*.*?\*/|//[^\n]*", "", open(HEADER).read(), flags=re.S)
    protos = dict(re.findall(r"\b(mlm_\w+)\s*\(([^()]*)\)\s*;", text))
    assert set(protos) == set(B._SIGNATURES) == set(B.EXPORTS)
    for name, args in protos.items():
        kinds = "".join("P" if "*" in a else SCALAR[a.replace("const", "").split()[0]] for a in args.split(","))
        assert kinds == B._SIGNATURES[name], name


@pytest.mark.parametrize("missing", ["_raw_stream", "_device"])
def test_current_stream_without_the_short_way(monkeypatch, missing):
    monkeypatch.setattr(B, "_raw_stream", lambda device: 100 + device)
    monkeypatch.setattr(B, "_device", lambda: 3)
    monkeypatch.setattr(torch.cuda, "is_initialized", lambda: True)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: types.SimpleNamespace(cuda_stream=77))
    assert B._st(None) == 103 and B._st(5) == 5
    monkeypatch.setattr(B, missing, None)
    assert B._st(None) == 77
