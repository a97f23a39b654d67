"""Thin ctypes binding of libmlm_shard.so: same names as include/mlm_shard.h, argument marshalling only.

Tensors are torch CUDA tensors (PyTorch is used for device memory and streams, nothing else); every
call is enqueued on torch's current stream.  There is no fallback: if the HIP library is missing the
import of a function raises, loudly.
"""
from __future__ import annotations

import ctypes
import os
import warnings
from typing import Optional, Sequence

import torch

MLM_F32, MLM_BF16 = 0, 1
(WS_LAYERNORM_BWD, WS_ATTN_FWD, WS_ATTN_BWD, WS_MLP_FWD, WS_MLP_BWD, WS_COLSUM,
 WS_VOCAB_CE_FWD, WS_VOCAB_CE_BWD) = range(8)

LIB_PATH = os.path.join(os.path.dirname(os.path.abspath(__file__)), "libmlm_shard.so")

# Argument types, one letter each: P pointer, i int32, l int64, u uint64, z size_t, f float.  They are declared once, so that
# a call passes plain integers.
_SIGNATURES = dict(item.split("=") for item in """
mlm_shard_range=liiPP mlm_workspace_bytes=PiP mlm_status_string=i mlm_layernorm_fwd=PPPPPPPP
mlm_layernorm_bwd=PPPPPPPPPPPzP mlm_combine=PPiPPPP mlm_combine_layernorm_fwd=PPiPPPPPPPPP
mlm_combine_layernorm_bwd=PPiPPPPPPPPPPPzP mlm_colsum=PPPPzP mlm_colsum_noalloc=PPPP mlm_deferred_sums_bytes=PP
mlm_deferred_sums_begin=Pz mlm_deferred_sums_flush=P mlm_attn_shard_fwd=PPPPPPPPPPPzP mlm_attn_shard_bwd=PPPPPPPPPPPPPPzP
mlm_mlp_shard_fwd=PPPPPPPPPzP mlm_mlp_shard_bwd=PPPPPPPPPPPPzP mlm_vocab_ce_shard_fwd=PPPPPPPPPzP
mlm_vocab_ce_merge=PPPPiPPPPPP mlm_vocab_ce_shard_bwd=PPPPPPPPPPPPzP mlm_gemm=iiilllPPPPP mlm_grad_sqnorm=iPPiPPPzP
mlm_adamw_step=ilPPPPPPffffffiP mlm_adamw_step_multi=iiPPPPPPPPfffffiP mlm_rng_stream_seed=uiiP
mlm_combine_dropout=PPiPiPPPP mlm_combine_layernorm_fwd_dropout=PPiPPPPPPPPPP
mlm_combine_layernorm_bwd_dropout=PPiPPPPPPPPPPPPPzP mlm_attn_keep_words=PP mlm_attn_shard_fwd_dropout=PPPPPPPPPPPPPzP
mlm_attn_shard_bwd_dropout=PPPPPPPPPPPPPPPPzP mlm_embed_shard_fwd=PPPPPP mlm_embed_bwd_replicated=PPPPPP
mlm_embed_shard_bwd=PPPPPP mlm_rows_gather=PPPiiPP mlm_rows_scatter=PPPiPP mlm_mlp_shard_bwd_input=PPPPPPPPPzP
mlm_attn_shard_bwd_input=PPPPPPPPPPPPPPzP mlm_layer_shard_wgrads=PPPPPPPPPPPPPPzP
""".split())
EXPORTS = tuple(_SIGNATURES)
_CTYPES = {"P": ctypes.c_void_p, "i": ctypes.c_int32, "l": ctypes.c_int64, "u": ctypes.c_uint64, "z": ctypes.c_size_t,
           "f": ctypes.c_float}
STREAM_REPLICATED, STREAM_MODEL_PARALLEL = 0, 1


class MlmError(RuntimeError):
    def __init__(self, code: int, where: str):
        self.code = code
        super().__init__(f"{where}: {status_string(code)} ({code})")


class Dims(ctypes.Structure):
    _fields_ = [("b", ctypes.c_int32), ("s", ctypes.c_int32), ("H", ctypes.c_int32), ("h", ctypes.c_int32),
                ("F", ctypes.c_int32), ("V", ctypes.c_int32), ("p", ctypes.c_int32), ("r", ctypes.c_int32),
                ("dtype", ctypes.c_int32), ("causal", ctypes.c_int32), ("gelu_tanh", ctypes.c_int32),
                ("ln_eps", ctypes.c_float)]


class Dropout(ctypes.Structure):
    """One dropout site: probability, stream seed (mlm_rng_stream_seed) and the 64-bit offset that names the site."""
    _fields_ = [("p", ctypes.c_float), ("seed", ctypes.c_uint64), ("offset", ctypes.c_uint64)]


def make_dropout(p: float, seed: int, offset: int) -> Dropout:
    return Dropout(float(p), int(seed) & 0xFFFFFFFFFFFFFFFF, int(offset) & 0xFFFFFFFFFFFFFFFF)


_lib = None


def lib() -> ctypes.CDLL:
    global _lib
    if _lib is None:
        if not os.path.exists(LIB_PATH):
            raise RuntimeError(f"{LIB_PATH} is not built; run `python -m paper_1909_08053_amd.build` "
                               "(there is no fallback path)")
        L = ctypes.CDLL(LIB_PATH)
        for name, sig in _SIGNATURES.items():
            f = getattr(L, name)
            f.argtypes = [_CTYPES[c] for c in sig]
            f.restype = ctypes.c_char_p if name == "mlm_status_string" else ctypes.c_int
        _lib = L
    return _lib


def status_string(code: int) -> str:
    return lib().mlm_status_string(int(code)).decode()


def make_dims(b, s, H, h, F, V, p, r, dtype, causal=True, gelu_tanh=True, ln_eps=1e-5) -> Dims:
    return Dims(int(b), int(s), int(H), int(h), int(F), int(V), int(p), int(r), int(dtype), int(bool(causal)),
                int(bool(gelu_tanh)), float(ln_eps))


def _p(t: Optional[torch.Tensor]):
    if t is None:
        return None
    if not t.is_cuda or not t.is_contiguous():
        raise ValueError("expected a contiguous CUDA tensor")
    return t.data_ptr()


# The raw handle of torch.cuda.current_stream(), without building the object; a torch without these two goes through the object.
_raw_stream, _device = (getattr(torch._C, n, None) for n in ("_cuda_getCurrentRawStream", "_cuda_getDevice"))


def _st(stream):
    if stream is not None:
        return int(stream)
    if _raw_stream and _device and torch.cuda.is_initialized():
        return _raw_stream(_device())
    return torch.cuda.current_stream().cuda_stream


def _ws(ws: Optional[torch.Tensor]):
    if ws is None:
        return None, 0
    return _p(ws), ws.numel() * ws.element_size()


def _chk(rc: int, where: str):
    if rc != 0:
        raise MlmError(rc, where)


def _marshalled(name: str):
    """The entry point as the native module has it: (tensors, structures, lists of tensors, ..., stream) -> status.  A list stands for an
    array and the count behind it, a tensor ahead of a size for both."""
    sig = _SIGNATURES[name]

    def f(*args):
        out, it, nbytes, count = [], iter(args), 0, None
        for at, kind in enumerate(sig):
            if kind == "z":
                out.append(nbytes)
                continue
            if kind == "i" and count is not None:
                out.append(count)
                count = None
                continue
            a = next(it)
            if kind == "P" and at == len(sig) - 1:
                a = _st(a)
            elif isinstance(a, ctypes.Structure):
                a = ctypes.byref(a)
            elif isinstance(a, (list, tuple)):
                count, a = len(a), (ctypes.c_void_p * max(len(a), 1))(*[_p(t) for t in a])
            elif kind == "P":
                a, nbytes = _ws(a)
            out.append(a)
        return getattr(lib(), name)(*out)
    return f


class _Marshalled:
    """Every entry point through ctypes, for a torch that the native module does not load into."""
    def __getattr__(self, name):
        f = _marshalled(name)
        setattr(self, name, f)
        return f


def _load():
    """What marshals the calls: the native module or, with a warning that says why, ctypes."""
    try:
        from . import _mlm_call
        return _mlm_call
    except ImportError as e:
        if os.path.exists(LIB_PATH):     # (else nothing is built yet: lib() says so)
            warnings.warn(f"arguments are marshalled through ctypes, not by the native module: {e}", RuntimeWarning, stacklevel=2)
        return _Marshalled()


# Arguments are marshalled natively (csrc/py_call.cpp): in Python that was 69 of 178 us of the host time of a step of 40 launches, now 149 us in
# all (bf16, 400 tokens x 192, two shards; the GPU needs 161).
_call = _load()


def mlm_shard_range(n: int, p: int, r: int):
    b, e = ctypes.c_int64(0), ctypes.c_int64(0)
    _chk(lib().mlm_shard_range(n, p, r, ctypes.byref(b),
                               ctypes.byref(e)), "mlm_shard_range")
    return b.value, e.value


def mlm_workspace_bytes(dims: Dims, which: int) -> int:
    n = ctypes.c_size_t(0)
    _chk(lib().mlm_workspace_bytes(ctypes.byref(dims), which, ctypes.byref(n)), "mlm_workspace_bytes")
    return n.value


def mlm_layernorm_fwd(dims, x, gamma, beta, y, mean, rstd, stream=None):
    _chk(_call.mlm_layernorm_fwd(dims, x, gamma, beta, y, mean, rstd, stream), "mlm_layernorm_fwd")


def mlm_layernorm_bwd(dims, dy, x, gamma, mean, rstd, residual_grad, dx, dgamma, dbeta, ws, stream=None):
    _chk(_call.mlm_layernorm_bwd(dims, dy, x, gamma, mean, rstd, residual_grad, dx, dgamma, dbeta, ws, stream),
         "mlm_layernorm_bwd")


def mlm_combine(dims, partials: Sequence[torch.Tensor], bias, residual, out, stream=None):
    _chk(_call.mlm_combine(dims, partials, bias, residual, out, stream), "mlm_combine")


def mlm_combine_layernorm_fwd(dims, partials: Sequence[torch.Tensor], bias, residual, x_out, gamma, beta, y, mean, rstd,
                              stream=None):
    _chk(_call.mlm_combine_layernorm_fwd(dims, partials, bias, residual, x_out, gamma, beta, y, mean, rstd, stream),
         "mlm_combine_layernorm_fwd")


def mlm_combine_layernorm_bwd(dims, partials: Sequence[torch.Tensor], x, gamma, mean, rstd, residual_grad, dy_out, dx,
                              dgamma, dbeta, dx_colsum, ws, stream=None):
    _chk(_call.mlm_combine_layernorm_bwd(dims, partials, x, gamma, mean, rstd, residual_grad, dy_out, dx, dgamma, dbeta,
                                         dx_colsum, ws, stream), "mlm_combine_layernorm_bwd")


def mlm_colsum(dims, dy, dbias, ws, stream=None):
    _chk(_call.mlm_colsum(dims, dy, dbias, ws, stream), "mlm_colsum")


def mlm_colsum_noalloc(dims, dy, dbias, stream=None):
    _chk(_call.mlm_colsum_noalloc(dims, dy, dbias, stream), "mlm_colsum_noalloc")


def mlm_deferred_sums_bytes(dims) -> int:
    n = ctypes.c_size_t(0)
    _chk(lib().mlm_deferred_sums_bytes(ctypes.byref(dims), ctypes.byref(n)), "mlm_deferred_sums_bytes")
    return int(n.value)


def mlm_deferred_sums_begin(buf):
    _chk(_call.mlm_deferred_sums_begin(buf), "mlm_deferred_sums_begin")


def mlm_deferred_sums_flush(stream=None):
    _chk(_call.mlm_deferred_sums_flush(stream), "mlm_deferred_sums_flush")


def mlm_attn_shard_fwd(dims, u, Wqkv_r, bqkv_r, Wo_r, key_len, qkv_r, ctx_r, lse_r, partial_r, ws=None, stream=None):
    _chk(_call.mlm_attn_shard_fwd(dims, u, Wqkv_r, bqkv_r, Wo_r, key_len, qkv_r, ctx_r, lse_r, partial_r, ws, stream),
         "mlm_attn_shard_fwd")


def mlm_attn_shard_bwd(dims, dx1, u, Wqkv_r, Wo_r, key_len, qkv_r, ctx_r, lse_r, dWqkv_r, dbqkv_r, dWo_r,
                       du_partial_r, ws, stream=None):
    _chk(_call.mlm_attn_shard_bwd(dims, dx1, u, Wqkv_r, Wo_r, key_len, qkv_r, ctx_r, lse_r, dWqkv_r, dbqkv_r, dWo_r,
                                  du_partial_r, ws, stream), "mlm_attn_shard_bwd")


def mlm_mlp_shard_fwd(dims, u2, A_r, a_r, B_r, g_r, y_r, partial_r, ws=None, stream=None):
    _chk(_call.mlm_mlp_shard_fwd(dims, u2, A_r, a_r, B_r, g_r, y_r, partial_r, ws, stream), "mlm_mlp_shard_fwd")


def mlm_mlp_shard_bwd(dims, dx2, u2, A_r, B_r, g_r, y_r, dA_r, da_r, dB_r, du2_partial_r, ws, stream=None):
    _chk(_call.mlm_mlp_shard_bwd(dims, dx2, u2, A_r, B_r, g_r, y_r, dA_r, da_r, dB_r, du2_partial_r, ws, stream),
         "mlm_mlp_shard_bwd")


def mlm_vocab_ce_shard_fwd(dims, hf, E_r, targets, m_r, s_r, t_r, logits_r, ws, stream=None):
    _chk(_call.mlm_vocab_ce_shard_fwd(dims, hf, E_r, targets, m_r, s_r, t_r, logits_r, ws, stream),
         "mlm_vocab_ce_shard_fwd")


def mlm_vocab_ce_merge(dims, m, s, t, n_shards, loss_w, ce, M, S, loss_out, stream=None):
    _chk(_call.mlm_vocab_ce_merge(dims, m, s, t, n_shards, loss_w, ce, M, S, loss_out, stream), "mlm_vocab_ce_merge")


def mlm_vocab_ce_shard_bwd(dims, hf, E_r, targets, loss_w, M, S, loss_stats, logits_r, dE_r, dhf_partial_r, ws,
                           stream=None):
    _chk(_call.mlm_vocab_ce_shard_bwd(dims, hf, E_r, targets, loss_w, M, S, loss_stats, logits_r, dE_r, dhf_partial_r,
                                      ws, stream), "mlm_vocab_ce_shard_bwd")


def mlm_gemm(dtype, trans_a, trans_b, M, N, K, A, B, C, bias=None, stream=None):
    _chk(lib().mlm_gemm(dtype, trans_a, trans_b, M,
                        N, K, _p(A), _p(B), _p(C), _p(bias), _st(stream)), "mlm_gemm")


def mlm_grad_sqnorm(dtype, grads: Sequence[torch.Tensor], other_sqnorm, sqnorm_out, ws, stream=None):
    n = len(grads)
    for t in grads:
        _p(t)
    arr = (ctypes.c_void_p * max(n, 1))(*[t.data_ptr() for t in grads])
    cnt = (ctypes.c_int64 * max(n, 1))(*[t.numel() for t in grads])
    _chk(lib().mlm_grad_sqnorm(dtype, arr, cnt, n, _p(other_sqnorm), _p(sqnorm_out),
                               *_ws(ws), _st(stream)), "mlm_grad_sqnorm")


def mlm_adamw_step(dtype, grad, master, m, v, weight_out, total_sqnorm, max_norm, lr, beta1, beta2, eps, weight_decay,
                   step, stream=None):
    _chk(lib().mlm_adamw_step(dtype, grad.numel(), _p(grad), _p(master), _p(m), _p(v),
                              _p(weight_out), _p(total_sqnorm), max_norm, lr, beta1, beta2, eps,
                              weight_decay, step, _st(stream)), "mlm_adamw_step")


def mlm_adamw_step_multi(dtype, grads, masters, ms, vs, weights_out, weight_decays, total_sqnorm, max_norm, lr, beta1,
                         beta2, eps, step, stream=None):
    n = len(grads)
    ptrs = lambda ts: (ctypes.c_void_p * n)(*[(_p(t) or 0) for t in ts])
    cnt = (ctypes.c_int64 * n)(*[t.numel() for t in grads])
    wds = (ctypes.c_float * n)(*[float(x) for x in weight_decays])
    _chk(lib().mlm_adamw_step_multi(dtype, n, cnt, ptrs(grads), ptrs(masters), ptrs(ms),
                                    ptrs(vs), ptrs(weights_out), wds, _p(total_sqnorm), max_norm, lr, beta1,
                                    beta2, eps, step, _st(stream)), "mlm_adamw_step_multi")


# ---- dropout (two random streams) and the input embedding -------------------------------------------------------
def mlm_rng_stream_seed(base_seed: int, stream: int, r: int) -> int:
    out = ctypes.c_uint64(0)
    _chk(lib().mlm_rng_stream_seed(base_seed & 0xFFFFFFFFFFFFFFFF, stream,
                                   r, ctypes.byref(out)), "mlm_rng_stream_seed")
    return out.value


def mlm_combine_dropout(dims, partials, bias, bias_rows, drop, residual, out, stream=None):
    _chk(_call.mlm_combine_dropout(dims, partials, bias, bias_rows, drop, residual, out, stream), "mlm_combine_dropout")


def mlm_combine_layernorm_fwd_dropout(dims, partials, bias, drop, residual, x_out, gamma, beta, y, mean, rstd,
                                      stream=None):
    _chk(_call.mlm_combine_layernorm_fwd_dropout(dims, partials, bias, drop, residual, x_out, gamma, beta, y, mean,
                                                 rstd, stream), "mlm_combine_layernorm_fwd_dropout")


def mlm_combine_layernorm_bwd_dropout(dims, partials, x, gamma, mean, rstd, residual_grad, drop, dy_out, dx, dz_out,
                                      dgamma, dbeta, dx_colsum, ws, stream=None):
    _chk(_call.mlm_combine_layernorm_bwd_dropout(dims, partials, x, gamma, mean, rstd, residual_grad, drop, dy_out, dx,
                                                 dz_out, dgamma, dbeta, dx_colsum, ws, stream),
         "mlm_combine_layernorm_bwd_dropout")


def mlm_attn_keep_words(dims) -> int:
    n = ctypes.c_size_t(0)
    _chk(lib().mlm_attn_keep_words(ctypes.byref(dims), ctypes.byref(n)), "mlm_attn_keep_words")
    return n.value


def mlm_attn_shard_fwd_dropout(dims, u, Wqkv_r, bqkv_r, Wo_r, key_len, drop, qkv_r, ctx_r, lse_r, keep_bits_r,
                               partial_r, ws=None, stream=None):
    _chk(_call.mlm_attn_shard_fwd_dropout(dims, u, Wqkv_r, bqkv_r, Wo_r, key_len, drop, qkv_r, ctx_r, lse_r,
                                          keep_bits_r, partial_r, ws, stream), "mlm_attn_shard_fwd_dropout")


def mlm_attn_shard_bwd_dropout(dims, dx1, u, Wqkv_r, Wo_r, key_len, drop, qkv_r, ctx_r, lse_r, keep_bits_r, dWqkv_r,
                               dbqkv_r, dWo_r, du_partial_r, ws, stream=None):
    _chk(_call.mlm_attn_shard_bwd_dropout(dims, dx1, u, Wqkv_r, Wo_r, key_len, drop, qkv_r, ctx_r, lse_r, keep_bits_r,
                                          dWqkv_r, dbqkv_r, dWo_r, du_partial_r, ws, stream),
         "mlm_attn_shard_bwd_dropout")


def mlm_embed_shard_fwd(dims, ids, E_r, perm_r, partial_r, stream=None):
    _chk(_call.mlm_embed_shard_fwd(dims, ids, E_r, perm_r, partial_r, stream), "mlm_embed_shard_fwd")


def mlm_embed_bwd_replicated(dims, dx0, drop, dz0, dpos, stream=None):
    _chk(_call.mlm_embed_bwd_replicated(dims, dx0, drop, dz0, dpos, stream), "mlm_embed_bwd_replicated")


def mlm_embed_shard_bwd(dims, ids, perm_r, dz0, dE_r, stream=None):
    _chk(_call.mlm_embed_shard_bwd(dims, ids, perm_r, dz0, dE_r, stream), "mlm_embed_shard_bwd")


def mlm_rows_gather(dims, x, row_idx, n, n_out, out, stream=None):
    _chk(_call.mlm_rows_gather(dims, x, row_idx, n, n_out, out, stream), "mlm_rows_gather")


def mlm_rows_scatter(dims, y, row_idx, n, out, stream=None):
    _chk(_call.mlm_rows_scatter(dims, y, row_idx, n, out, stream), "mlm_rows_scatter")


# ---- backward with the weight gradients deferred to one grouped launch -------------------------------------------
def mlm_mlp_shard_bwd_input(dims, dx2, A_r, B_r, g_r, dg_r, da_r, du2_partial_r, ws, stream=None):
    _chk(_call.mlm_mlp_shard_bwd_input(dims, dx2, A_r, B_r, g_r, dg_r, da_r, du2_partial_r, ws, stream),
         "mlm_mlp_shard_bwd_input")


def mlm_attn_shard_bwd_input(dims, dx1, Wqkv_r, Wo_r, key_len, drop, qkv_r, ctx_r, lse_r, keep_bits_r, dqkv_r, dbqkv_r,
                             du_partial_r, ws, stream=None):
    _chk(_call.mlm_attn_shard_bwd_input(dims, dx1, Wqkv_r, Wo_r, key_len, drop, qkv_r, ctx_r, lse_r, keep_bits_r,
                                        dqkv_r, dbqkv_r, du_partial_r, ws, stream), "mlm_attn_shard_bwd_input")


def mlm_layer_shard_wgrads(dims, u, dqkv_r, ctx_r, dz1, u2, dg_r, y_r, dz2, dWqkv_r, dWo_r, dA_r, dB_r, ws, stream=None):
    _chk(_call.mlm_layer_shard_wgrads(dims, u, dqkv_r, ctx_r, dz1, u2, dg_r, y_r, dz2, dWqkv_r, dWo_r, dA_r, dB_r, ws, stream),
         "mlm_layer_shard_wgrads")
