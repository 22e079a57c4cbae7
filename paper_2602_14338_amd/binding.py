"""ctypes binding of the C ABI: argument marshalling only, same names as the C entry points.

Tensors must live on the GPU; pointers are taken with ``data_ptr()`` and work is enqueued
on torch's current stream for that device.  Nothing here computes anything.
"""
from __future__ import annotations

import ctypes as C
import os
from dataclasses import dataclass
from typing import Optional

import torch

AERO_F32, AERO_BF16, AERO_F16, AERO_F8E4M3 = 0, 1, 2, 3
AERO_ROW_PADDING, AERO_ROW_UNTOUCHED = -1, -2
AERO_DW_ACCUMULATE = 0x100
OP_GROUP_ADVANTAGE, OP_LOGPROB_FWD, OP_GRPO_LOSS_BWD, OP_LMHEAD_FUSED = 0, 1, 2, 3

_LIB_PATH = os.path.join(os.path.dirname(os.path.abspath(__file__)), "libaero_hip.so")


class AeroError(RuntimeError):
    pass


class _AdvParamsC(C.Structure):
    _fields_ = [("k_ratio", C.c_int32), ("s_rescue", C.c_int32), ("tau_num", C.c_int32),
                ("tau_den", C.c_int32), ("zero_keep", C.c_int32), ("reject_enable", C.c_int32),
                ("posterior_mode", C.c_int32), ("alpha0", C.c_float), ("beta0", C.c_float)]


@dataclass
class AdvParams:
    k_ratio: int = 1
    s_rescue: int = 0
    tau_num: int = 1
    tau_den: int = 2
    zero_keep: int = 4
    reject_enable: int = 0
    posterior_mode: int = 0
    alpha0: float = 1.0
    beta0: float = 1.0

    def to_c(self) -> _AdvParamsC:
        return _AdvParamsC(self.k_ratio, self.s_rescue, self.tau_num, self.tau_den, self.zero_keep,
                           self.reject_enable, self.posterior_mode, self.alpha0, self.beta0)


def library_path() -> str:
    return _LIB_PATH


def _load() -> C.CDLL:
    if not os.path.exists(_LIB_PATH):
        raise AeroError(f"{_LIB_PATH} is missing: build it with `python -m paper_2602_14338_amd.build` "
                        "(there is no fallback path)")
    lib = C.CDLL(_LIB_PATH)
    p, i32, i64, f32, sz = C.c_void_p, C.c_int32, C.c_int64, C.c_float, C.c_size_t
    lib.aero_status_string.restype = C.c_char_p
    lib.aero_status_string.argtypes = [i32]
    lib.aero_workspace_bytes.restype = sz
    lib.aero_workspace_bytes.argtypes = [i32, i64, i32, i32, i32, i32]
    lib.aero_group_advantage.restype = i32
    lib.aero_group_advantage.argtypes = [p, p, p, p, i32, i32, C.POINTER(_AdvParamsC)] + [p] * 7 + [p, p]
    lib.aero_logprob_fwd.restype = i32
    lib.aero_logprob_fwd.argtypes = [p, i32, i64, i32, i64, p, p, p, p, p, p, p]
    lib.aero_grpo_loss_bwd.restype = i32
    lib.aero_grpo_loss_bwd.argtypes = [p, i32, i64, i32, i64, p, p, p, p, p, p, p, i32, f32, f32, f32, f32, f32, p,
                                       p, p, p, p, p, p, p, p, sz, p]
    lib.aero_grpo_loss_bwd_noalloc.restype = i32
    lib.aero_grpo_loss_bwd_noalloc.argtypes = lib.aero_grpo_loss_bwd.argtypes[:-3] + [p]
    lib.aero_lmhead_logprob_fused.restype = i32
    lib.aero_lmhead_logprob_fused.argtypes = [p, p, i64, i32, i32, p, p, p, p, p, p, p, p, i32, f32, f32, f32, f32,
                                              f32, p, p, p, p, p, i32, p, p, sz, p]
    return lib


class _Lazy:
    """Loads the library on first use so that the package can be imported to build it."""
    _cdll = None

    def __getattr__(self, name):   # first use of an entry point: kept as a plain attribute from then on
        if _Lazy._cdll is None:
            _Lazy._cdll = _load()
        fn = getattr(_Lazy._cdll, name)
        setattr(self, name, fn)
        return fn


_lib = _Lazy()


def _check(status: int, what: str) -> None:
    if status != 0:
        raise AeroError(f"{what}: {_lib.aero_status_string(status).decode()} (status {status})")


def _ptr(t: Optional[torch.Tensor], dtype=None, name: str = "") -> Optional[int]:
    if t is None:
        return None
    if not t.is_cuda:
        raise AeroError(f"{name}: expected a GPU tensor")
    if dtype is not None and t.dtype != dtype:
        raise AeroError(f"{name}: expected dtype {dtype}, got {t.dtype}")
    if not t.is_contiguous():
        raise AeroError(f"{name}: expected a contiguous tensor")
    return t.data_ptr()


class _Marshal:
    """The native module (csrc/marshal.cpp).  ``pointers(t, dtype, name, ...)``: `_ptr` of every triple in one call;
    ``group_advantage`` and the others: a whole call whose arguments are all plain, NotImplemented for any other."""

    def __getattr__(self, name):
        if name not in ("pointers", "group_advantage", "logprob_fwd", "loss_bwd", "fused"):
            raise AttributeError(name)
        try:
            from . import _marshal
        except ImportError as e:
            raise AeroError("the package's _marshal module is missing: build it with "
                            "`python -m paper_2602_14338_amd.build` (there is no fallback path)") from e
        if name == "pointers":
            _marshal.setup(AeroError, _ptr)
        else:
            entries = (_lib.aero_group_advantage, _lib.aero_logprob_fwd, _lib.aero_grpo_loss_bwd,
                       _lib.aero_grpo_loss_bwd_noalloc, _lib.aero_lmhead_logprob_fused)
            _marshal.bind(torch._C._cuda_getCurrentRawStream, AdvParams, *(C.cast(f, C.c_void_p).value for f in entries))
        fn = getattr(_marshal, name)
        setattr(self, name, fn)
        return fn


_m = _Marshal()
_F32, _I32, _U8, _BF16 = torch.float32, torch.int32, torch.uint8, torch.bfloat16


def _stream(t: torch.Tensor) -> int:
    """Handle of torch's current stream on the tensor's device (a GPU tensor: its pointer was taken before)."""
    return torch._C._cuda_getCurrentRawStream(t.get_device())


_DTYPE_CODES = {torch.bfloat16: AERO_BF16, torch.float32: AERO_F32, torch.float16: AERO_F16,
                torch.float8_e4m3fn: AERO_F8E4M3}


def _dtype_code(t: torch.Tensor) -> int:
    code = _DTYPE_CODES.get(t.dtype)
    if code is None:
        raise AeroError(f"unsupported dtype {t.dtype}")
    return code


def aero_workspace_bytes(op: int, T: int = 0, V: int = 0, H: int = 0, R: int = 0, Q: int = 0) -> int:
    return int(_lib.aero_workspace_bytes(op, T, V, H, R, Q))


def aero_group_advantage(rewards, lengths, group_offsets, keep_priority, Q: int, R: int, params: AdvParams,
                         adv, weight, keep_mask, kept_index, kept_offsets, group_zero_var, group_category,
                         err_flag=None) -> None:
    st = _m.group_advantage(rewards, lengths, group_offsets, keep_priority, Q, R, params, adv, weight, keep_mask,
                            kept_index, kept_offsets, group_zero_var, group_category, err_flag)
    if st is not NotImplemented:
        return _check(st, "aero_group_advantage")
    pc = params.to_c()
    p = _m.pointers(rewards, _F32, "rewards", lengths, _I32, "lengths", group_offsets, _I32, "group_offsets",
                    keep_priority, None, "keep_priority", adv, _F32, "adv", weight, _F32, "weight",
                    keep_mask, _U8, "keep_mask", kept_index, _I32, "kept_index", kept_offsets, _I32, "kept_offsets",
                    group_zero_var, _U8, "group_zero_var", group_category, _U8, "group_category",
                    err_flag, _I32, "err_flag")
    st = _lib.aero_group_advantage(*p[:4], Q, R, C.byref(pc), *p[4:], _stream(group_offsets))
    _check(st, "aero_group_advantage")


def aero_logprob_fwd(logits, T: int, V: int, ld: int, targets, row_active, logprob, entropy, lse,
                     err_flag=None) -> None:
    st = _m.logprob_fwd(logits, T, V, ld, targets, row_active, logprob, entropy, lse, err_flag)
    if st is not NotImplemented:
        return _check(st, "aero_logprob_fwd")
    z, *p = _m.pointers(logits, None, "logits", targets, _I32, "targets", row_active, _U8, "row_active",
                        logprob, _F32, "logprob", entropy, _F32, "entropy", lse, _F32, "lse",
                        err_flag, _I32, "err_flag")
    st = _lib.aero_logprob_fwd(z, _dtype_code(logits), T, V, ld, *p, _stream(logits))
    _check(st, "aero_logprob_fwd")


def _loss_pointers(logits, targets, lse, entropy, old_logprob, token_rollout, adv, weight, ref_logprob, loss, clip_frac,
                   logprob_out, entropy_out, lse_out, dlogits, err_flag):
    if dlogits is not None and dlogits.dtype != logits.dtype:
        raise AeroError("dlogits must have the dtype of logits")
    return _m.pointers(
        logits, None, "logits", targets, _I32, "targets", lse, _F32, "lse", entropy, _F32, "entropy",
        old_logprob, _F32, "old_logprob", token_rollout, _I32, "token_rollout", adv, _F32, "adv",
        weight, _F32, "weight", ref_logprob, _F32, "ref_logprob", loss, _F32, "loss", clip_frac, _F32, "clip_frac",
        logprob_out, _F32, "logprob_out", entropy_out, _F32, "entropy_out", lse_out, _F32, "lse_out",
        dlogits, None, "dlogits", err_flag, _I32, "err_flag")


def aero_grpo_loss_bwd(logits, T: int, V: int, ld: int, targets, lse, old_logprob, token_rollout, adv, weight,
                       R: int, eps_lo: float, eps_hi: float, grad_scale: float, loss, clip_frac, logprob_out,
                       dlogits, workspace, err_flag=None, entropy_out=None, lse_out=None,
                       entropy_coef: float = 0.0, entropy=None, kl_coef: float = 0.0, ref_logprob=None) -> None:
    st = _m.loss_bwd(logits, T, V, ld, targets, lse, entropy, old_logprob, token_rollout, adv, weight, R, eps_lo, eps_hi,
                     grad_scale, entropy_coef, kl_coef, ref_logprob, loss, clip_frac, logprob_out, entropy_out, lse_out,
                     dlogits, err_flag, workspace)
    if st is not NotImplemented:
        return _check(st, "aero_grpo_loss_bwd")
    z, *p = _loss_pointers(logits, targets, lse, entropy, old_logprob, token_rollout, adv, weight, ref_logprob, loss,
                           clip_frac, logprob_out, entropy_out, lse_out, dlogits, err_flag)
    ws, = _m.pointers(workspace, None, "workspace")
    st = _lib.aero_grpo_loss_bwd(
        z, _dtype_code(logits), T, V, ld, *p[:7], R, eps_lo, eps_hi, grad_scale, entropy_coef, kl_coef, *p[7:], ws,
        workspace.numel() * workspace.element_size() if workspace is not None else 0, _stream(logits))
    _check(st, "aero_grpo_loss_bwd")


def aero_grpo_loss_bwd_noalloc(logits, T: int, V: int, ld: int, targets, lse, old_logprob, token_rollout, adv, weight,
                               R: int, eps_lo: float, eps_hi: float, grad_scale: float, loss, clip_frac,
                               logprob_out, dlogits, err_flag=None, entropy_out=None, lse_out=None,
                               entropy_coef: float = 0.0, entropy=None, kl_coef: float = 0.0,
                               ref_logprob=None) -> None:
    """aero_grpo_loss_bwd without a workspace argument: the library's own fixed scratch is used."""
    st = _m.loss_bwd(logits, T, V, ld, targets, lse, entropy, old_logprob, token_rollout, adv, weight, R, eps_lo, eps_hi,
                     grad_scale, entropy_coef, kl_coef, ref_logprob, loss, clip_frac, logprob_out, entropy_out, lse_out,
                     dlogits, err_flag)
    if st is not NotImplemented:
        return _check(st, "aero_grpo_loss_bwd_noalloc")
    z, *p = _loss_pointers(logits, targets, lse, entropy, old_logprob, token_rollout, adv, weight, ref_logprob, loss,
                           clip_frac, logprob_out, entropy_out, lse_out, dlogits, err_flag)
    st = _lib.aero_grpo_loss_bwd_noalloc(z, _dtype_code(logits), T, V, ld, *p[:7], R, eps_lo, eps_hi, grad_scale,
                                         entropy_coef, kl_coef, *p[7:], _stream(logits))
    _check(st, "aero_grpo_loss_bwd_noalloc")


def aero_lmhead_logprob_fused(hidden, weight, T: int, H: int, V: int, targets, logprob, entropy, lse,
                              old_logprob=None, token_rollout=None, adv=None, weight_rollout=None, R: int = 0,
                              eps_lo: float = 0.2, eps_hi: float = 0.2, grad_scale: float = 1.0,
                              loss=None, clip_frac=None, dhidden=None, dweight=None, workspace=None,
                              err_flag=None, entropy_coef: float = 0.0, kl_coef: float = 0.0,
                              ref_logprob=None, dweight_accumulate: bool = False) -> None:
    st = _m.fused(hidden, weight, T, H, V, targets, logprob, entropy, lse, old_logprob, token_rollout, adv, weight_rollout,
                  R, eps_lo, eps_hi, grad_scale, entropy_coef, kl_coef, ref_logprob, loss, clip_frac, dhidden, dweight,
                  dweight_accumulate, err_flag, workspace)
    if st is not NotImplemented:
        return _check(st, "aero_lmhead_logprob_fused")
    p = _m.pointers(
        hidden, _BF16, "hidden", weight, _BF16, "weight", targets, _I32, "targets", logprob, _F32, "logprob",
        entropy, _F32, "entropy", lse, _F32, "lse", old_logprob, _F32, "old_logprob",
        token_rollout, _I32, "token_rollout", adv, _F32, "adv", weight_rollout, _F32, "weight_rollout",
        ref_logprob, _F32, "ref_logprob", loss, _F32, "loss", clip_frac, _F32, "clip_frac", dhidden, _BF16, "dhidden",
        dweight, None, "dweight", err_flag, _I32, "err_flag", workspace, None, "workspace")
    dweight_dtype = (_dtype_code(dweight) if dweight is not None else AERO_F32) | \
        (AERO_DW_ACCUMULATE if dweight_accumulate else 0)
    st = _lib.aero_lmhead_logprob_fused(
        *p[:2], T, H, V, *p[2:10], R, eps_lo, eps_hi, grad_scale, entropy_coef, kl_coef, *p[10:15], dweight_dtype,
        *p[15:], workspace.numel() * workspace.element_size() if workspace is not None else 0, _stream(hidden))
    _check(st, "aero_lmhead_logprob_fused")
