"""The native module that marshals arguments against the same through ctypes: statuses and refusals (no GPU needed: nothing is launched)."""
import pytest
import torch

from paper_1909_08053_amd import binding as B

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


@pytest.mark.parametrize("name,args", CALLS, ids=[f"{n}-{i}" for i, (n, _) in enumerate(CALLS)])
def test_native_marshalling_is_that_of_ctypes(name, args):
    if isinstance(B._call, B._Marshalled):
        pytest.skip("the native module is not built")
    got, want = outcome(getattr(B._call, name), args), outcome(B._marshalled(name), args)
    assert got == want and got != 0


@pytest.mark.parametrize("args", [(), (D,), (D, None, None, None, None, None, None, 0, 0), (None, None, None, None, None, None, None, 0),
                                  (DROP, None, None, None, None, None, None, 0), (D, 3.5, None, None, None, None, None, 0)])
def test_wrong_arguments_are_refused(args):
    if isinstance(B._call, B._Marshalled):
        pytest.skip("the native module is not built")
    with pytest.raises(TypeError):
        B._call.mlm_layernorm_fwd(*args)
