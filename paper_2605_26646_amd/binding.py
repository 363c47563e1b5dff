"""Binding of libumas.so: the entry points, whose argument marshalling is native (csrc/umas_torch.cpp), and the C ABI through ctypes."""
from __future__ import annotations

import ctypes as C
import importlib.util
import os
from dataclasses import dataclass
from typing import Optional

import numpy as np
import torch

PLACE_LAST, PLACE_ALL = 0, 1
SEG_TURN, SEG_TRAJ = 0, 1
UMAS_F32, UMAS_BF16 = 0, 1

_HERE = os.path.dirname(os.path.abspath(__file__))


class UmasError(RuntimeError):
    def __init__(self, code: int, message: str):
        super().__init__(f"libumas status {code}: {message}")
        self.code = code


class _Graph(C.Structure):
    _fields_ = [("n_roles", C.c_int32), ("n_models", C.c_int32), ("n_traj", C.c_int32), ("n_turns", C.c_int32),
                ("n_tokens", C.c_int64), ("role_to_model", C.c_void_p), ("traj_turn_off", C.c_void_p),
                ("turn_role", C.c_void_p), ("turn_tok_off", C.c_void_p), ("turn_pred_off", C.c_void_p),
                ("turn_pred", C.c_void_p), ("traj_group", C.c_void_p)]


class _Rewards(C.Structure):
    _fields_ = [("role_reward", C.c_void_p), ("turn_reward", C.c_void_p), ("traj_reward", C.c_void_p),
                ("w_role", C.c_void_p), ("w_turn", C.c_void_p), ("w_traj", C.c_void_p),
                ("place_mode", C.c_int32), ("norm_eps", C.c_float)]


_STREAM_FIELDS = ["model_tok_off", "perm", "tok_turn", "tok_role", "tok_mask", "tok_reward", "turn_seg_off",
                  "seg_turn", "model_turn_off", "traj_seg_off", "model_trajrun_off", "rowsel",
                  "model_rowsel_off", "turn_scalar", "turn_step", "tok_flags"]


class _Streams(C.Structure):
    _fields_ = [(name, C.c_void_p) for name in _STREAM_FIELDS]


STATS_DTYPE = np.dtype([("loss", "<f4"), ("clip_frac", "<f4"), ("entropy_mean", "<f4"), ("approx_kl", "<f4"),
                        ("n_scored", "<i8"), ("n_invalid_ids", "<i8")])


@dataclass
class Streams:
    """Device tensors written by umas_assign_token_rewards (model-local order)."""
    n_tokens: int
    n_turns: int
    n_models: int
    model_tok_off: torch.Tensor
    perm: torch.Tensor
    tok_turn: torch.Tensor
    tok_role: torch.Tensor
    tok_mask: torch.Tensor
    tok_reward: torch.Tensor
    turn_seg_off: torch.Tensor
    seg_turn: torch.Tensor
    model_turn_off: torch.Tensor
    traj_seg_off: torch.Tensor
    model_trajrun_off: torch.Tensor
    rowsel: torch.Tensor
    model_rowsel_off: torch.Tensor
    turn_scalar: torch.Tensor
    turn_step: torch.Tensor
    tok_flags: torch.Tensor

    def _c(self) -> _Streams:
        s = _Streams()
        for name in _STREAM_FIELDS:
            t = getattr(self, name)
            # an empty tensor has no storage; the ABI wants non-NULL pointers even for size 0
            setattr(s, name, t.data_ptr() or _dummy(t.device).data_ptr())
        return s


_LIB = None
_DUMMY = {}


def _dummy(device) -> torch.Tensor:
    key = str(device)
    if key not in _DUMMY:
        _DUMMY[key] = torch.zeros(256, dtype=torch.uint8, device=device)
    return _DUMMY[key]


def lib_path() -> str:
    return os.path.join(_HERE, "libumas.so")


def load_library():
    """Load libumas.so built in-tree; there is no fallback when it is missing."""
    global _LIB
    if _LIB is not None:
        return _LIB
    path = lib_path()
    if not os.path.exists(path):
        raise FileNotFoundError(f"{path} is missing: build it with `python -c 'import __graft_entry__ as g; g.build()'`")
    lib = C.CDLL(path)
    lib.umas_last_error.restype = C.c_char_p
    for name in ("umas_assign_workspace_bytes", "umas_advantages_workspace_bytes",
                 "umas_policy_logprobs_workspace_bytes", "umas_ppo_loss_workspace_bytes",
                 "umas_ppo_loss_workspace_bytes_min", "umas_ppo_loss_workspace_bytes_entropy"):
        getattr(lib, name).restype = C.c_size_t
    lib.umas_assign_workspace_bytes.argtypes = [C.c_void_p]
    lib.umas_advantages_workspace_bytes.argtypes = [C.c_int64]
    lib.umas_policy_logprobs_workspace_bytes.argtypes = [C.c_int64, C.c_int32, C.c_int32, C.c_int]
    lib.umas_ppo_loss_workspace_bytes.argtypes = [C.c_int64, C.c_int32, C.c_int32, C.c_int, C.c_int32]
    lib.umas_ppo_loss_workspace_bytes_min.argtypes = [C.c_int64, C.c_int32, C.c_int32, C.c_int, C.c_int32]
    lib.umas_ppo_loss_workspace_bytes_entropy.argtypes = [C.c_int64, C.c_int32, C.c_int32, C.c_int, C.c_int32]
    lib.umas_assign_token_rewards.restype = C.c_int
    lib.umas_assign_token_rewards.argtypes = [C.c_void_p, C.c_void_p, C.c_void_p, C.c_void_p, C.c_void_p,
                                              C.c_size_t, C.c_void_p]
    lib.umas_advantages.restype = C.c_int
    lib.umas_advantages.argtypes = [C.c_void_p, C.c_int64, C.c_int32, C.c_void_p, C.c_float, C.c_float, C.c_float,
                                    C.c_int32, C.c_void_p, C.c_void_p, C.c_void_p, C.c_size_t, C.c_void_p]
    lib.umas_policy_logprobs.restype = C.c_int
    lib.umas_policy_logprobs.argtypes = [C.c_void_p, C.c_void_p, C.c_int, C.c_int64, C.c_int32, C.c_int32,
                                         C.c_void_p, C.c_void_p, C.c_int64, C.c_void_p, C.c_void_p, C.c_void_p,
                                         C.c_void_p, C.c_size_t, C.c_void_p]
    lib.umas_ppo_loss_fwd_bwd.restype = C.c_int
    lib.umas_ppo_loss_fwd_bwd.argtypes = [C.c_void_p, C.c_void_p, C.c_int, C.c_int64, C.c_int32, C.c_int32,
                                          C.c_void_p, C.c_void_p, C.c_int64, C.c_void_p, C.c_void_p, C.c_void_p,
                                          C.c_int32, C.c_float, C.c_float, C.c_float, C.c_int32, C.c_int64, C.c_void_p,
                                          C.c_float, C.c_void_p, C.c_void_p, C.c_void_p, C.c_void_p, C.c_void_p, C.c_size_t,
                                          C.c_void_p]
    lib.umas_policy_logprobs_static.restype = C.c_int
    lib.umas_policy_logprobs_static.argtypes = [C.c_void_p, C.c_void_p, C.c_int, C.c_int64, C.c_int32, C.c_int32,
                                                C.c_void_p, C.c_void_p, C.c_int64, C.c_void_p, C.c_void_p, C.c_void_p,
                                                C.c_void_p]
    lib.umas_values.restype = C.c_int
    lib.umas_values.argtypes = [C.c_void_p, C.c_void_p, C.c_float, C.c_int, C.c_int64, C.c_int32, C.c_void_p, C.c_int64,
                                C.c_void_p, C.c_void_p]
    lib.umas_value_workspace_bytes.restype = C.c_size_t
    lib.umas_value_workspace_bytes.argtypes = [C.c_int64, C.c_int32, C.c_int, C.c_int32]
    lib.umas_value_loss_fwd_bwd.restype = C.c_int
    lib.umas_value_loss_fwd_bwd.argtypes = [C.c_void_p, C.c_void_p, C.c_float, C.c_int, C.c_int64, C.c_int32, C.c_void_p,
                                            C.c_int64, C.c_void_p, C.c_void_p, C.c_void_p, C.c_int32, C.c_float, C.c_int32,
                                            C.c_int32, C.c_int64, C.c_void_p, C.c_void_p, C.c_void_p, C.c_void_p, C.c_void_p,
                                            C.c_void_p, C.c_size_t, C.c_void_p]
    lib.umas_kl_rewards_workspace_bytes.restype = C.c_size_t
    lib.umas_kl_rewards_workspace_bytes.argtypes = [C.c_int64]
    lib.umas_kl_rewards.restype = C.c_int
    lib.umas_kl_rewards.argtypes = [C.c_void_p, C.c_void_p, C.c_void_p, C.c_void_p, C.c_int64, C.c_float, C.c_void_p,
                                    C.c_void_p, C.c_void_p, C.c_size_t, C.c_void_p]
    lib.umas_whiten_workspace_bytes.restype = C.c_size_t
    lib.umas_whiten_workspace_bytes.argtypes = [C.c_int64, C.c_int32, C.c_int32]
    lib.umas_whiten_advantages.restype = C.c_int
    lib.umas_whiten_advantages.argtypes = [C.c_void_p, C.c_void_p, C.c_void_p, C.c_void_p, C.c_int32, C.c_int32, C.c_int64,
                                           C.c_int32, C.c_float, C.c_void_p, C.c_void_p, C.c_size_t, C.c_void_p]
    lib.umas_ready_batch_workspace_bytes.restype = C.c_size_t
    lib.umas_ready_batch_workspace_bytes.argtypes = [C.c_int32, C.c_int32]
    for fn in (lib.umas_ready_batch, lib.umas_ready_batch_balanced):
        fn.restype = C.c_int
        fn.argtypes = [C.c_void_p, C.c_int32, C.c_int32, C.c_void_p, C.c_int32, C.c_void_p, C.c_void_p,
                       C.c_int32, C.c_void_p, C.c_void_p, C.c_void_p, C.c_size_t, C.c_void_p]
    lib.umas_ready_batch_packed.restype = C.c_int
    lib.umas_ready_batch_packed.argtypes = [C.c_void_p, C.c_int32, C.c_int32, C.c_void_p, C.c_int32, C.c_void_p, C.c_void_p,
                                            C.c_int64, C.c_void_p, C.c_void_p, C.c_void_p, C.c_void_p, C.c_size_t, C.c_void_p]
    _LIB = lib
    return lib


_NATIVE = None


def _native():
    """The native half of this module (csrc/umas_torch.cpp), built next to libumas.so; there is no fallback when it is missing."""
    global _NATIVE
    if _NATIVE is None:
        load_library()
        path = os.path.join(_HERE, "_umas_torch.so")
        if not os.path.exists(path):
            raise FileNotFoundError(f"{path} is missing: build it with `python -c 'import __graft_entry__ as g; g.build()'`")
        spec = importlib.util.spec_from_file_location("_umas_torch", path)
        module = importlib.util.module_from_spec(spec)
        spec.loader.exec_module(module)
        _NATIVE = module
    return _NATIVE


def _check(lib, status: int):
    if status != 0:
        raise UmasError(status, lib.umas_last_error().decode())


def _done(result):
    """The native module returns the outputs, or the status when the library refuses."""
    if type(result) is int:
        _check(load_library(), result)
    return result


def _stream():
    return torch._C._cuda_getCurrentRawStream(torch.cuda.current_device())


# Row selections are device data that the library cannot check.  With CHECK_ROWS on (the test suite switches it on)
# every call that takes one first reads its range back and refuses entries outside [0, n_rows): a mistake in a caller
# then raises here instead of sending a kernel out of bounds.  It waits for the stream, so it stays off by default
# and is skipped under graph capture.
CHECK_ROWS = False


def _check_rows(rowsel: Optional[torch.Tensor], H: torch.Tensor):
    if not CHECK_ROWS or rowsel is None or rowsel.numel() == 0 or torch.cuda.is_current_stream_capturing():
        return
    lo, hi, n_rows = int(rowsel.min().item()), int(rowsel.max().item()), H.shape[0]
    if lo < 0 or hi >= n_rows:
        raise UmasError(-1, f"row selection holds entries from {lo} to {hi}, outside [0, {n_rows})")


def umas_assign_token_rewards(*, n_roles, n_models, role_to_model, traj_turn_off, turn_role, turn_tok_off,
                              tok_mask_global: torch.Tensor, turn_pred_off=None, turn_pred=None, traj_group=None,
                              role_reward=None, turn_reward=None, traj_reward=None, w_role=None, w_turn=None,
                              w_traj=None, place_mode=PLACE_LAST, norm_eps=1e-6) -> Streams:
    return Streams(*_done(_native().assign(n_roles, n_models, role_to_model, traj_turn_off, turn_role, turn_tok_off, tok_mask_global,
                                           turn_pred_off, turn_pred, traj_group, role_reward, turn_reward, traj_reward, w_role,
                                           w_turn, w_traj, place_mode, norm_eps, _stream())))


def umas_advantages(streams: Streams, value: Optional[torch.Tensor], gamma, lam, gamma_turn=1.0, seg_mode=SEG_TURN):
    return _done(_native().advantages(streams, value, gamma, lam, gamma_turn, seg_mode, _stream()))


def umas_policy_logprobs(H: torch.Tensor, W: torch.Tensor, ids: torch.Tensor, rowsel: Optional[torch.Tensor] = None,
                         want_entropy=True, workspace: Optional[torch.Tensor] = None):
    _check_rows(rowsel, H)
    return _done(_native().policy_logprobs(H, W, ids, rowsel, want_entropy, workspace, _stream()))


STATIC_SCRATCH_BYTES = 32 << 20


def umas_policy_logprobs_static(H: torch.Tensor, W: torch.Tensor, ids: torch.Tensor, rowsel: Optional[torch.Tensor] = None,
                                logp=None, lse=None, entropy=None):
    """umas_policy_logprobs without a workspace (the library's static scratch); the outputs may be passed in, so that
    the call itself allocates nothing."""
    _check_rows(rowsel, H)
    return _done(_native().policy_logprobs_static(H, W, ids, rowsel, logp, lse, entropy, _stream()))


def ppo_workspace_bytes(n_sel, d, V, dtype: torch.dtype, n_roles, minimum=False, entropy_bonus=True) -> int:
    """The size for updates with or without an entropy bonus; entropy_bonus=False leaves out what only one with a bonus uses (up
    to half of the bytes)."""
    lib = load_library()
    code = UMAS_BF16 if dtype == torch.bfloat16 else UMAS_F32
    f = (lib.umas_ppo_loss_workspace_bytes_min if minimum else
         lib.umas_ppo_loss_workspace_bytes_entropy if entropy_bonus else lib.umas_ppo_loss_workspace_bytes)
    return int(f(n_sel, d, V, code, n_roles))


def umas_ppo_loss_fwd_bwd(H, W, ids, rowsel, logp_old, adv, tok_role, n_roles, clip_eps, *, entropy_coef=0.0,
                          dual_clip=0.0, accumulate_dW=False, norm_rows=0, logp_ref=None, kl_coef=0.0, dW=None, dH=None,
                          logp_new=None, stats=None, workspace=None):
    _check_rows(rowsel, H)
    return _done(_native().ppo_loss(H, W, ids, rowsel, logp_old, adv, tok_role, n_roles, clip_eps, entropy_coef, dual_clip, accumulate_dW,
                                    norm_rows, logp_ref, kl_coef, dW, dH, logp_new, stats, workspace, _stream()))


VALUE_STATS_DTYPE = np.dtype([("loss", "<f4"), ("clip_frac", "<f4"), ("value_mean", "<f4"), ("reserved", "<f4"),
                              ("n_scored", "<i8")])


def umas_values(H, w, bias=0.0, rowsel=None, value=None):
    _check_rows(rowsel, H)
    return _done(_native().values(H, w, bias, rowsel, value, _stream()))


def umas_value_loss_fwd_bwd(H, w, bias, rowsel, value_old, ret, tok_role, n_roles, clip_eps_v, *, accumulate_dH=False,
                            accumulate_dw=False, norm_rows=0, dH=None, dw=None, db=None, value_new=None, stats=None,
                            workspace=None):
    _check_rows(rowsel, H)
    return _done(_native().value_loss(H, w, bias, rowsel, value_old, ret, tok_role, n_roles, clip_eps_v, accumulate_dH, accumulate_dw,
                                      norm_rows, dH, dw, db, value_new, stats, workspace, _stream()))


WHITEN_MODEL, WHITEN_MODEL_ROLE = 0, 1


def umas_kl_rewards(tok_reward, logp, logp_ref, tok_mask, beta, out=None):
    """Returns (penalised rewards, device float[1] mean of logp - logp_ref over the mask=1 tokens)."""
    return _done(_native().kl_rewards(tok_reward, logp, logp_ref, tok_mask, beta, out, _stream()))


def umas_whiten_advantages(adv, tok_mask, tok_role, model_tok_off, n_roles, scope=WHITEN_MODEL, eps=1e-8, out=None):
    return _done(_native().whiten(adv, tok_mask, tok_role, model_tok_off, n_roles, scope, eps, out, _stream()))


def umas_ready_batch(streams: Streams, traj_turn_off, n_minibatch, traj_keep=None, traj_order=None, balance_rows=False):
    """Returns (mb_rowsel device int32, mb_off device int64 [n_models, n_minibatch + 1]); balance_rows selects
    umas_ready_batch_balanced (parts cut by scored rows per model instead of by trajectories)."""
    return _done(_native().ready_batch(streams, traj_turn_off, 1 if balance_rows else 0, n_minibatch, traj_keep, traj_order, _stream()))


def umas_ready_batch_packed(streams: Streams, traj_turn_off, max_rows, traj_keep=None, traj_order=None):
    """Returns (mb_rowsel device int32, mb_off device int64 [n_models, n_traj + 1], n_parts device int32 [n_models]):
    micro-batches of whole trajectories under a budget of max_rows scored rows."""
    return _done(_native().ready_batch(streams, traj_turn_off, 2, max_rows, traj_keep, traj_order, _stream()))


def read_value_stats(stats: torch.Tensor) -> np.ndarray:
    return stats.cpu().numpy().view(VALUE_STATS_DTYPE)


def read_stats(stats: torch.Tensor) -> np.ndarray:
    """Copy the device umas_loss_stats array to a numpy structured array (synchronises)."""
    return stats.cpu().numpy().view(STATS_DTYPE)


def profile_enable(on: bool) -> None:
    """Switch the library's per-kernel event timing on (discarding earlier records) or off."""
    lib = load_library()
    lib.umas_profile_enable.restype = C.c_int
    lib.umas_profile_enable.argtypes = [C.c_int32]
    _check(lib, lib.umas_profile_enable(1 if on else 0))


def profile_read(cap: int = 64) -> dict:
    """{kernel name: (total milliseconds, launches)} since profile_enable(True); synchronises."""
    lib = load_library()
    lib.umas_profile_read.restype = C.c_int32
    lib.umas_profile_read.argtypes = [C.c_void_p, C.c_void_p, C.c_void_p, C.c_int32]
    names = C.create_string_buffer(32 * cap)
    ms = (C.c_float * cap)()
    cnt = (C.c_int32 * cap)()
    n = lib.umas_profile_read(names, ms, cnt, cap)
    if n < 0:
        raise UmasError(-5, "umas_profile_read failed")
    out = {}
    for i in range(n):
        out[names.raw[32 * i:32 * i + 32].split(b"\0")[0].decode()] = (float(ms[i]), int(cnt[i]))
    return out
