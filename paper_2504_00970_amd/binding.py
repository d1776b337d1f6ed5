"""Thin Python binding of libsentencekv (see include/sentencekv.h).

Argument marshalling only: every function here forwards the device pointers of caller-allocated
torch tensors to the C entry point of the same name and raises on a non-zero status.  Nothing is
computed in Python and there is no fallback: if the HIP library is missing or fails, calls raise.
The calls of a serving loop go through a native module (csrc/calls.cpp), set-up calls through ctypes; where the module
cannot be built, all of them do.
"""
from __future__ import annotations

import ctypes
import operator
import os
from dataclasses import dataclass
from typing import Optional

import torch

from . import _build

SKV_F32, SKV_BF16, SKV_FP8_E4M3 = 0, 1, 2
SKV_OK, SKV_EINVAL, SKV_ECAPACITY, SKV_EHIP, SKV_ENOMEM = 0, -1, -2, -3, -4


class SkvError(RuntimeError):
    def __init__(self, status: int, what: str):
        self.status = status
        super().__init__(f"{what}: {_lib().skv_strerror(status).decode()} ({status})")


class _Desc(ctypes.Structure):
    _fields_ = [(n, ctypes.c_int32) for n in ("n_layers", "n_q_heads", "n_kv_heads", "head_dim", "kv_dtype",
                                              "max_tokens", "max_sentences", "max_budget", "max_batch", "semvec_dtype")]


_LIB = None
_CALLS = None
_vp, _i32, _int, _i64 = ctypes.c_void_p, ctypes.c_int32, ctypes.c_int, ctypes.c_int64

_SIGNATURES = {
    "skv_create": (_int, [ctypes.POINTER(_vp), ctypes.POINTER(_Desc), _vp]),
    "skv_destroy": (None, [_vp]),
    "skv_set_stream": (_int, [_vp, _vp]),
    "skv_strerror": (ctypes.c_char_p, [_int]),
    "skv_workspace_bytes": (_i64, [_vp]),
    "skv_set_wait_limit": (_int, [_vp, _i32]),
    "skv_set_single_launch": (_int, [_vp, _i32]),
    "skv_set_budget_hint": (_int, [_vp, _i32]),
    "skv_segment": (_int, [_vp, _vp, _i32, _vp, _i32, _vp, _vp, _vp, _vp, _vp]),
    "skv_build_semvec": (_int, [_vp, _vp, _i32, _vp, _i32, _vp]),
    "skv_build_semvec_layers": (_int, [_vp, _vp, _i32, _vp, _i32, _vp]),
    "skv_token_importance_work_bytes": (_i64, [_vp, _i32, _i32]),
    "skv_token_importance": (_int, [_vp, _vp, _vp, _i32, _i32, _vp, _vp, _i64]),
    "skv_retain": (_int, [_vp, _vp, _i32, _i32, _vp, _i32, _vp, _vp, _vp, _vp]),
    "skv_compact_pool": (_int, [_vp, _vp, _vp, _i32, _vp, _i32, _vp, _vp, _vp]),
    "skv_query_update": (_int, [_vp, _i32, _vp, _vp, _vp, _i32, _vp, _vp, _vp]),
    "skv_score": (_int, [_vp, _i32, _vp, _vp, _i32, _vp]),
    "skv_select": (_int, [_vp, _vp, _vp, _vp, _i32, _i32, _vp, _vp, _vp, _vp]),
    "skv_gather": (_int, [_vp, _i32, _vp, _vp, _i32, _int, _vp, _vp, _i32, _vp, _vp]),
    "skv_attend": (_int, [_vp, _vp, _vp, _vp, _vp, _i32, _vp, _vp]),
    "skv_merge_lse": (_int, [_vp, _i32, _vp, _vp, _vp, _vp, _vp, _vp]),
    "skv_decode_step": (_int, [_vp, _i32, _i32, _vp, _vp, _vp, _vp, _i32, _vp, _i32, _vp, _vp, _vp, _vp, _vp, _vp,
                               _vp, _vp, _vp]),
    "skv_decode_step_noalloc": (_int, [ctypes.POINTER(_Desc), _vp, _i32, _i32, _vp, _vp, _vp, _vp, _i32, _vp, _i32, _vp, _vp,
                                       _vp, _vp, _vp, _vp, _vp, _vp, _vp]),
}
EXPORTS = tuple(_SIGNATURES)


def lib_path() -> str:
    return _build.LIB


class _CtypesCalls:
    """The call module's functions by ctypes, for machines that cannot build it: the same arguments, several times the time per call."""

    def __init__(self, lib):
        for name, (res, kinds) in _SIGNATURES.items():
            if res is _int and kinds[0] is _vp:
                setattr(self, name, self._function(getattr(lib, name), kinds, 9 if name == "skv_segment" else 0))

    @staticmethod
    def _function(fn, kinds, address):
        def call(*args):
            if len(args) != len(kinds):
                raise TypeError("wrong number of arguments")
            return fn(*(_address(a) if k is _vp and i in (0, address) else _p(a) if k is _vp else _number(a)
                        for i, (a, k) in enumerate(zip(args, kinds))))
        return call


def _address(a):
    if a is None or isinstance(a, int):
        return a
    raise TypeError(f"an address or None expected, got {type(a).__name__}")


def _number(a):
    if isinstance(a, torch.Tensor):
        raise TypeError("a number expected, got a tensor")
    return operator.index(a)


def _p(t: Optional[torch.Tensor]):
    if t is None:
        return None
    if not isinstance(t, torch.Tensor):
        raise TypeError(f"a tensor or None expected, got {type(t).__name__}")
    assert t.is_contiguous(), "tensors handed to libsentencekv must be contiguous"
    return t.data_ptr()


def _lib():
    """Load the built library and the module that calls it; build what is not there at all, or does not run with this Python and torch."""
    global _LIB, _CALLS
    if _LIB is None:
        if not os.path.exists(_build.LIB):
            _build.build(force=True)
        lib = ctypes.CDLL(_build.LIB)
        for name, (res, args) in _SIGNATURES.items():
            fn = getattr(lib, name)
            fn.restype, fn.argtypes = res, args
        if _build.calls_fit() or _build.build_calls():
            from . import _calls
            _calls.load(_build.LIB)
            _CALLS = _calls
        else:
            _CALLS = _CtypesCalls(lib)
        _LIB = lib
    return _LIB


def _check(status: int, what: str) -> None:
    if status != SKV_OK:
        raise SkvError(status, what)


@dataclass
class Desc:
    n_layers: int
    n_q_heads: int
    n_kv_heads: int
    head_dim: int = 128
    kv_dtype: int = SKV_BF16
    max_tokens: int = 1
    max_sentences: int = 1
    max_budget: int = 1
    max_batch: int = 1
    semvec_dtype: int = SKV_F32

    @property
    def max_sel(self) -> int:
        return min(self.max_sentences, self.max_budget)


def dtype_code(dt: torch.dtype) -> int:
    if dt == torch.float32:
        return SKV_F32
    if dt == torch.bfloat16:
        return SKV_BF16
    raise TypeError(f"K/V/q must be float32 or bfloat16, got {dt}")


class Context:
    """Owns one skv_ctx.  Methods mirror the C entry points one to one."""

    def __init__(self, desc: Desc, stream: Optional[int] = None):
        lib = _lib()
        self.desc = desc
        d = _Desc(desc.n_layers, desc.n_q_heads, desc.n_kv_heads, desc.head_dim, desc.kv_dtype, desc.max_tokens,
                  desc.max_sentences, desc.max_budget, desc.max_batch, desc.semvec_dtype)
        h = _vp()
        if stream is None:
            stream = torch.cuda.current_stream().cuda_stream if torch.cuda.is_available() else 0
        _check(lib.skv_create(ctypes.byref(h), ctypes.byref(d), _vp(stream)), "skv_create")
        self._h = h
        self._handle = h.value

    def close(self) -> None:
        if getattr(self, "_h", None):
            _lib().skv_destroy(self._h)
            self._h = self._handle = None

    def __del__(self):
        try:
            self.close()
        except Exception:
            pass

    def set_stream(self, stream: int) -> None:
        _check(_lib().skv_set_stream(self._h, _vp(stream)), "skv_set_stream")

    def workspace_bytes(self) -> int:
        return int(_lib().skv_workspace_bytes(self._h))

    def set_budget_hint(self, budget: int) -> None:
        _check(_lib().skv_set_budget_hint(self._h, budget), "skv_set_budget_hint")

    def set_wait_limit(self, polls: int) -> None:
        _check(_lib().skv_set_wait_limit(self._h, polls), "skv_set_wait_limit")

    def set_single_launch(self, enable: bool) -> None:
        _check(_lib().skv_set_single_launch(self._h, 1 if enable else 0), "skv_set_single_launch")

    # ---- (1) prefill ----------------------------------------------------------------------------
    def segment(self, tok, term_bitmap, vocab: int, seg_id, sent_off, sent_len, n_sent_dev, sync: bool = True,
                T: Optional[int] = None) -> Optional[int]:
        host = ctypes.c_int32(-1)
        T = tok.shape[0] if T is None else T
        rc = _CALLS.skv_segment(self._handle, tok, T, term_bitmap, vocab, seg_id, sent_off,
                                sent_len, n_sent_dev, ctypes.addressof(host) if sync else None)
        _check(rc, "skv_segment")
        return int(host.value) if sync else None

    def build_semvec(self, K_pool, sent_off, S: int, semvec) -> None:
        T = K_pool.shape[2]
        _check(_CALLS.skv_build_semvec(self._handle, K_pool, T, sent_off, S, semvec), "skv_build_semvec")

    def build_semvec_layers(self, K_pool, sent_off, S: int, semvec) -> None:
        T = K_pool.shape[2]
        _check(_CALLS.skv_build_semvec_layers(self._handle, K_pool, T, sent_off, S, semvec), "skv_build_semvec_layers")

    # ---- prefill-side token retention (Sec. 4.1) ---------------------------------------------------------
    def token_importance_work_bytes(self, T: int, N: int) -> int:
        return int(_lib().skv_token_importance_work_bytes(self._h, T, N))

    def token_importance(self, q_obs, K_pool, T: int, N: int, alpha, work) -> None:
        _check(_CALLS.skv_token_importance(self._handle, q_obs, K_pool, T, N, alpha, work,
                                           work.numel() * work.element_size()), "skv_token_importance")

    def retain(self, alpha, Tp: int, k: int, seg_id, S: int, keep_idx, n_keep, ret_off, ret_len) -> None:
        _check(_CALLS.skv_retain(self._handle, alpha, Tp, k, seg_id, S, keep_idx, n_keep, ret_off,
                                 ret_len), "skv_retain")

    def compact_pool(self, K_pool, V_pool, T: int, keep_idx, k: int, n_keep, K_ret, V_ret) -> None:
        _check(_CALLS.skv_compact_pool(self._handle, K_pool, V_pool, T, keep_idx, k, n_keep, K_ret,
                                       V_ret), "skv_compact_pool")

    # ---- sentence query cache (Eq. 2) ----------------------------------------------------------------
    def query_update(self, B: int, q_t, tok_t, term_bitmap, vocab: int, q_sum, q_cnt, q_bar) -> None:
        _check(_CALLS.skv_query_update(self._handle, B, q_t, tok_t, term_bitmap, vocab, q_sum, q_cnt,
                                       q_bar), "skv_query_update")

    # ---- (2)-(5) decode, one layer, one sequence ---------------------------------------------------
    def score(self, layer: int, q_score, semvec, S: int, score) -> None:
        _check(_CALLS.skv_score(self._handle, layer, q_score, semvec, S, score), "skv_score")

    def select(self, score, sent_off, sent_len, S: int, budget: int, sel_sent, n_sel, tok_idx, n_tok) -> None:
        _check(_CALLS.skv_select(self._handle, score, sent_off, sent_len, S, budget, sel_sent, n_sel,
                                 tok_idx, n_tok), "skv_select")

    def gather(self, layer: int, K_pool, V_pool, T: int, tok_idx, n_tok, budget: int, K_sel, V_sel,
               pool_in_host: bool = False) -> None:
        _check(_CALLS.skv_gather(self._handle, layer, K_pool, V_pool, T, int(pool_in_host), tok_idx, n_tok,
                                 budget, K_sel, V_sel), "skv_gather")

    def attend(self, q_attn, K_sel, V_sel, n_tok, budget: int, out, lse=None) -> None:
        _check(_CALLS.skv_attend(self._handle, q_attn, K_sel, V_sel, n_tok, budget, out, lse),
               "skv_attend")

    # ---- fused, ragged batch -----------------------------------------------------------------------
    def decode_step(self, layer: int, B: int, q_score, q_attn, K_pool, V_pool, T_total: int, semvec, S_total: int,
                    cu_tok, cu_sent, sent_off, sent_len, budget, out, lse=None, tok_idx_out=None, n_tok_out=None) -> None:
        _check(_CALLS.skv_decode_step(self._handle, layer, B, q_score, q_attn, K_pool, V_pool, T_total,
                                      semvec, S_total, cu_tok, cu_sent, sent_off, sent_len,
                                      budget, out, lse, tok_idx_out, n_tok_out), "skv_decode_step")

    def merge_lse(self, n_heads: int, out_a, lse_a, out_b, lse_b, out, lse=None) -> None:
        _check(_CALLS.skv_merge_lse(self._handle, n_heads, out_a, lse_a, out_b, lse_b, out, lse),
               "skv_merge_lse")


NOALLOC_SCRATCH_BYTES = 8 * 1024 * 1024


def decode_step_noalloc(desc: Desc, layer: int, B: int, q_score, q_attn, K_pool, V_pool, T_total: int, semvec, S_total: int,
                        cu_tok, cu_sent, sent_off, sent_len, budget, out, lse=None, tok_idx_out=None, n_tok_out=None,
                        stream: Optional[int] = None) -> None:
    """skv_decode_step_noalloc: the decode step without a context, on the library's static device scratch."""
    d = _Desc(desc.n_layers, desc.n_q_heads, desc.n_kv_heads, desc.head_dim, desc.kv_dtype, desc.max_tokens,
              desc.max_sentences, desc.max_budget, desc.max_batch, desc.semvec_dtype)
    if stream is None:
        stream = torch.cuda.current_stream().cuda_stream if torch.cuda.is_available() else 0
    _check(_lib().skv_decode_step_noalloc(ctypes.byref(d), _vp(stream), layer, B, _p(q_score), _p(q_attn), _p(K_pool),
                                          _p(V_pool), T_total, _p(semvec), S_total, _p(cu_tok), _p(cu_sent), _p(sent_off),
                                          _p(sent_len), _p(budget), _p(out), _p(lse), _p(tok_idx_out), _p(n_tok_out)),
           "skv_decode_step_noalloc")
