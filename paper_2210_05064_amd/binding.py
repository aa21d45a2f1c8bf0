"""ctypes binding of libver.so: argument marshalling only.

Every function has the name of the C entry point it calls (include/ver.h) and
takes torch tensors that already live on the GPU; nothing is computed here and
there is no fallback: importing this module without the built library raises.
"""
from __future__ import annotations

import ctypes as C
import os

import torch

_HERE = os.path.dirname(os.path.abspath(__file__))
LIB_PATH = os.environ.get("VER_LIB", os.path.join(_HERE, "libver.so"))
_NATIVE = os.path.exists(os.path.join(_HERE, "_marshal.so"))   # built with the library; one built elsewhere (VER_LIB) does without
for _path in [LIB_PATH] + ([] if _NATIVE or "VER_LIB" in os.environ else [os.path.join(_HERE, "_marshal.so")]):
    if not os.path.exists(_path):
        raise ImportError(f"{_path} is missing: run `python -m paper_2210_05064_amd.build` "
                          "(or __graft_entry__.build()) first; there is no CPU fallback")
lib = C.CDLL(LIB_PATH)

VER_OK = 0
_vp, _i32, _sz, _f = C.c_void_p, C.c_int32, C.c_size_t, C.c_float


class PackArgs(C.Structure):
    _fields_ = [
        ("dones", _vp), ("env_off", _vp), ("env_started_episode", _vp), ("seq_key", _vp),
        ("N", _i32), ("S", _i32), ("B", _i32), ("b", _i32),
        ("info", _vp), ("seq_first", _vp), ("seq_len", _vp), ("seq_is_ep_start", _vp),
        ("batch_sizes", _vp), ("t_off", _vp), ("gather_idx", _vp),
        ("obs", _vp), ("D", _i32), ("obs_packed", _vp), ("obs_packed_bf16", _i32),
        ("actions", _vp), ("act_bytes", _i32), ("actions_packed", _vp),
        ("logp_old", _vp), ("adv", _vp), ("ret", _vp), ("is_weight", _vp),
        ("logp_old_packed", _vp), ("adv_packed", _vp), ("ret_packed", _vp), ("is_weight_packed", _vp),
        ("rnn_h", _vp), ("rnn_c", _vp), ("n_layers", _i32), ("H", _i32), ("seq_cap", _i32),
        ("h0", _vp), ("c0", _vp),
        ("workspace", _vp), ("workspace_bytes", _sz), ("index_ready", _i32),
    ]


class LstmCfg(C.Structure):
    _fields_ = [("n_layers", _i32), ("input_dim", _i32), ("hidden", _i32), ("act_dim", _i32),
                ("compute", _i32), ("x_bf16", _i32), ("layer_by_layer", _i32)]


class PpoCfg(C.Structure):
    _fields_ = [("clip", _f), ("value_coef", _f), ("entropy_coef", _f), ("dist", _i32), ("act_dim", _i32)]


class AdamCfg(C.Structure):
    _fields_ = [("lr0", _f), ("lr_final", _f), ("total_steps", C.c_int64), ("beta1", _f), ("beta2", _f), ("eps", _f),
                ("max_grad_norm", _f)]


lib.ver_status_string.restype = C.c_char_p
lib.ver_status_string.argtypes = [C.c_int]
lib.ver_gae_workspace_bytes.restype = _sz
lib.ver_gae_workspace_bytes.argtypes = [_i32]
lib.ver_gae.restype = C.c_int
lib.ver_gae.argtypes = [_vp, _vp, _vp, _vp, _vp, _i32, _i32, _f, _f, _vp, _vp, _vp, _sz, _vp]
lib.ver_gae_static.restype = C.c_int
lib.ver_gae_static.argtypes = [_vp, _vp, _vp, _vp, _vp, _i32, _i32, _f, _f, _vp, _vp, _vp]
lib.ver_ingest_workspace_bytes.restype = _sz
lib.ver_ingest_workspace_bytes.argtypes = [_i32, _i32]
lib.ver_ingest.restype = C.c_int
lib.ver_ingest.argtypes = [_vp, _vp, _i32, _i32, _vp, _vp, _vp, _vp, _sz, _vp]
lib.ver_ingest_dense.restype = C.c_int
lib.ver_ingest_dense.argtypes = [_i32, _i32, _vp, _vp, _vp]
lib.ver_ingest_gather.restype = C.c_int
lib.ver_ingest_gather.argtypes = [_vp, _i32, _vp, _i32, _vp, _vp]
lib.ver_ingest_gather_batch.restype = C.c_int
lib.ver_ingest_gather_batch.argtypes = [_vp, _i32, _i32, _vp, _vp, _vp, _vp]
lib.ver_is_weight.restype = C.c_int
lib.ver_is_weight.argtypes = [_vp, _i32, _i32, _f, _vp, _vp]
lib.ver_pack_workspace_bytes.restype = _sz
lib.ver_pack_workspace_bytes.argtypes = [_i32, _i32, _i32]
lib.ver_pack_minibatch.restype = C.c_int
lib.ver_pack_minibatch.argtypes = [C.POINTER(PackArgs), _vp]
lib.ver_pack_index_batch.restype = C.c_int
lib.ver_pack_index_batch.argtypes = [C.POINTER(PackArgs), _i32, _vp]
lib.ver_lstm_workspace_bytes.restype = _sz
lib.ver_lstm_workspace_bytes.argtypes = [C.POINTER(LstmCfg), _i32]
lib.ver_lstm_fwd.restype = C.c_int
lib.ver_lstm_fwd.argtypes = [C.POINTER(LstmCfg), _vp, _i32, _vp, _vp, _vp, _vp, _vp, _i32,
                             C.POINTER(_vp), _vp, _vp, _vp, _sz, _vp]
lib.ver_lstm_bwd.restype = C.c_int
lib.ver_lstm_bwd.argtypes = [C.POINTER(LstmCfg), _vp, _i32, _vp, _vp, _vp, _vp, _vp, _i32,
                             C.POINTER(_vp), _vp, _vp, C.POINTER(_vp), _vp, _vp, _sz, _vp]
lib.ver_ppo_loss_workspace_bytes.restype = _sz
lib.ver_ppo_loss_workspace_bytes.argtypes = [_i32, _i32]
lib.ver_ppo_loss.restype = C.c_int
lib.ver_ppo_loss.argtypes = [C.POINTER(PpoCfg), _i32, _vp, _vp, _vp, _vp, _vp, _vp, _vp, _vp,
                             _vp, _vp, _vp, _vp, _vp, _sz, _vp]
lib.ver_ppo_loss_learned_entropy.restype = C.c_int
lib.ver_ppo_loss_learned_entropy.argtypes = [C.POINTER(PpoCfg), _i32, _vp, _vp, _vp, _vp, _vp, _vp, _vp, _vp,
                                             _vp, _f, _f, _vp, _vp, _vp, _vp, _vp, _vp, _sz, _vp]
lib.ver_adam_workspace_bytes.restype = _sz
lib.ver_adam_workspace_bytes.argtypes = []
lib.ver_adam_step.restype = C.c_int
lib.ver_adam_step.argtypes = [C.POINTER(AdamCfg), _i32, C.POINTER(_vp), C.POINTER(_vp), C.POINTER(_vp), C.POINTER(_vp),
                              C.POINTER(C.c_int64), C.c_int64, _vp, _vp, _sz, _vp]
lib.ver_adam_step_bounded.restype = C.c_int
lib.ver_adam_step_bounded.argtypes = [C.POINTER(AdamCfg), _i32, C.POINTER(_vp), C.POINTER(_vp), C.POINTER(_vp),
                                      C.POINTER(_vp), C.POINTER(C.c_int64), C.POINTER(_f), C.POINTER(_f), C.c_int64,
                                      _vp, _vp, _sz, _vp]

lib.ver_profile_enable.restype = C.c_int
lib.ver_profile_enable.argtypes = [C.c_uint32]
lib.ver_profile_read.restype = C.c_int
lib.ver_profile_read.argtypes = [C.POINTER(C.c_double), C.POINTER(C.c_int64)]
PROF_CLASSES = ["gae", "pack_index", "pack_gather", "lstm_prep", "lstm_gemm_fwd", "lstm_rec_fwd", "heads_fwd",
                "ppo_loss", "heads_bwd", "lstm_rec_bwd", "lstm_gemm_dx", "lstm_gemm_dw", "lstm_dbias", "adam",
                "is_weight", "ingest"]


class VerError(RuntimeError):
    def __init__(self, status: int):
        self.status = status
        super().__init__(f"libver: {lib.ver_status_string(status).decode()} ({status})")


def _check(status: int) -> None:
    if status != VER_OK:
        raise VerError(status)


def _ptr_any(t) -> int | None:
    """What _marshal does for a tensor, for any object (and the place its errors come from)."""
    if t is None:
        return None
    assert t.is_cuda and t.is_contiguous(), "device, contiguous tensors only"
    return t.data_ptr()


if _NATIVE:
    from . import _marshal   # (after torch, whose symbols it uses)
    _marshal.init(_ptr_any)
else:
    class _marshal:
        """The same in Python."""
        ptr = staticmethod(_ptr_any)

        @staticmethod
        def fill(arr, tensors):
            for i, t in enumerate(tensors):
                arr[i] = _ptr_any(t)

        @staticmethod
        def pointers(block, offsets, values):
            return list(values)   # (pack_args takes every field)
_ptr = _marshal.ptr


def _stream() -> int:
    return torch._C._cuda_getCurrentRawStream(torch.cuda.current_device())


def _ws(ws):
    return (_ptr(ws), ws.numel() * ws.element_size()) if ws is not None else (None, 0)


def ver_status_string(status: int) -> str:
    return lib.ver_status_string(status).decode()


def ver_gae_workspace_bytes(S: int) -> int:
    return lib.ver_gae_workspace_bytes(S)


def ver_gae(rewards, values, dones, last_values, env_off, N, S, gamma, lam, adv, ret, workspace):
    p, n = _ws(workspace)
    _check(lib.ver_gae(_ptr(rewards), _ptr(values), _ptr(dones), _ptr(last_values), _ptr(env_off),
                       N, S, gamma, lam, _ptr(adv), _ptr(ret), p, n, _stream()))


def ver_gae_static(rewards, values, dones, last_values, env_off, N, S, gamma, lam, adv, ret):
    _check(lib.ver_gae_static(_ptr(rewards), _ptr(values), _ptr(dones), _ptr(last_values), _ptr(env_off),
                              N, S, gamma, lam, _ptr(adv), _ptr(ret), _stream()))


def ver_ingest_workspace_bytes(N: int, S: int) -> int:
    return lib.ver_ingest_workspace_bytes(N, S)


def ver_ingest(arr_env, arr_t, N, S, env_off, order, info, workspace):
    p, n = _ws(workspace)
    _check(lib.ver_ingest(_ptr(arr_env), _ptr(arr_t), N, S, _ptr(env_off), _ptr(order), _ptr(info), p, n, _stream()))


def ver_ingest_dense(T, N, env_off, order):
    _check(lib.ver_ingest_dense(T, N, _ptr(env_off), _ptr(order), _stream()))


def ver_ingest_gather(order, S, src, dst):
    """dst[k] = src[order[k]] over the leading dimension; src, dst: contiguous tensors of equal shape and dtype."""
    row_bytes = src.element_size() * (src[0].numel() if S > 0 else 1)
    _check(lib.ver_ingest_gather(_ptr(order), S, _ptr(src), row_bytes, _ptr(dst), _stream()))


def ver_ingest_gather_batch(order, S, pairs):
    """dst[k] = src[order[k]] for every (src, dst) pair of contiguous tensors, in one launch."""
    n = len(pairs)
    srcs, dsts = _ptr_array([a for a, _ in pairs]), _ptr_array([b for _, b in pairs])
    rows = (C.c_int32 * n)(*[a.element_size() * (a.numel() // a.shape[0] if S > 0 else 1) for a, _ in pairs])
    _check(lib.ver_ingest_gather_batch(_ptr(order), S, n, srcs, rows, dsts, _stream()))


def ver_is_weight(env_off, N, S, max_is, weight):
    _check(lib.ver_is_weight(_ptr(env_off), N, S, max_is, _ptr(weight), _stream()))


def ver_pack_workspace_bytes(N: int, S: int, B: int) -> int:
    return lib.ver_pack_workspace_bytes(N, S, B)


def pack_args(**kw) -> PackArgs:
    """ver_pack_args from keyword arguments (its fields; tensors or ints)."""
    a = PackArgs()
    for k in _marshal.pointers(a, _PACK_POINTERS, kw):   # what is not a tensor for a pointer field
        if k not in _PACK_NAMES:
            raise TypeError(f"unknown ver_pack_args field {k}")
        v = kw[k]
        if k == "workspace":
            a.workspace, a.workspace_bytes = _ws(v)
        elif isinstance(v, torch.Tensor):
            setattr(a, k, _ptr(v))
        elif v is not None:
            setattr(a, k, v)
    return a


_PACK_NAMES = frozenset(f[0] for f in PackArgs._fields_)
_PACK_POINTERS = {f[0]: getattr(PackArgs, f[0]).offset for f in PackArgs._fields_ if f[1] is _vp and f[0] != "workspace"}


def ver_pack_minibatch(**kw):
    """Keyword arguments are the fields of ver_pack_args; tensors or ints."""
    a = pack_args(**kw)
    _check(lib.ver_pack_minibatch(C.byref(a), _stream()))


def ver_pack_index_batch(arg_blocks):
    """arg_blocks: list of ver_pack_args (see pack_args), one per minibatch."""
    arr = (PackArgs * len(arg_blocks))(*arg_blocks)
    _check(lib.ver_pack_index_batch(arr, len(arg_blocks), _stream()))


def _ptr_array(tensors):
    arr = (_vp * len(tensors))()
    _marshal.fill(arr, tensors)
    return arr


def lstm_cfg(n_layers, input_dim, hidden, act_dim, compute=0, x_bf16=0, layer_by_layer=0) -> LstmCfg:
    return LstmCfg(n_layers, input_dim, hidden, act_dim, compute, x_bf16, layer_by_layer)


def ver_lstm_workspace_bytes(cfg: LstmCfg, M: int) -> int:
    return lib.ver_lstm_workspace_bytes(C.byref(cfg), M)


def ver_lstm_fwd(cfg, x_packed, M, info, batch_sizes, t_off, h0, c0, seq_cap, weights, head_out, value,
                 workspace):
    p, n = _ws(workspace)
    _check(lib.ver_lstm_fwd(C.byref(cfg), _ptr(x_packed), M, _ptr(info), _ptr(batch_sizes), _ptr(t_off),
                            _ptr(h0), _ptr(c0), seq_cap, _ptr_array(weights), _ptr(head_out), _ptr(value),
                            p, n, _stream()))


def ver_lstm_bwd(cfg, x_packed, M, info, batch_sizes, t_off, h0, c0, seq_cap, weights, d_head_out, d_value,
                 weight_grads, d_x, workspace):
    p, n = _ws(workspace)
    _check(lib.ver_lstm_bwd(C.byref(cfg), _ptr(x_packed), M, _ptr(info), _ptr(batch_sizes), _ptr(t_off),
                            _ptr(h0), _ptr(c0), seq_cap, _ptr_array(weights), _ptr(d_head_out), _ptr(d_value),
                            _ptr_array(weight_grads), _ptr(d_x), p, n, _stream()))


def ppo_cfg(clip, value_coef, entropy_coef, dist, act_dim) -> PpoCfg:
    return PpoCfg(clip, value_coef, entropy_coef, dist, act_dim)


def ver_ppo_loss_workspace_bytes(M: int, act_dim: int) -> int:
    return lib.ver_ppo_loss_workspace_bytes(M, act_dim)


def ver_ppo_loss(cfg, M, head_out, value, log_std, actions_packed, logp_old, adv, ret, is_weight,
                 scalars, d_head_out, d_value, d_log_std, workspace):
    p, n = _ws(workspace)
    _check(lib.ver_ppo_loss(C.byref(cfg), M, _ptr(head_out), _ptr(value), _ptr(log_std), _ptr(actions_packed),
                            _ptr(logp_old), _ptr(adv), _ptr(ret), _ptr(is_weight), _ptr(scalars),
                            _ptr(d_head_out), _ptr(d_value), _ptr(d_log_std), p, n, _stream()))


def ver_ppo_loss_learned_entropy(cfg, M, head_out, value, log_std, actions_packed, logp_old, adv, ret, is_weight,
                                 alpha, target_entropy, alpha_sign, scalars, d_head_out, d_value, d_log_std, d_alpha,
                                 workspace):
    p, n = _ws(workspace)
    _check(lib.ver_ppo_loss_learned_entropy(
        C.byref(cfg), M, _ptr(head_out), _ptr(value), _ptr(log_std), _ptr(actions_packed), _ptr(logp_old), _ptr(adv),
        _ptr(ret), _ptr(is_weight), _ptr(alpha), target_entropy, alpha_sign, _ptr(scalars), _ptr(d_head_out),
        _ptr(d_value), _ptr(d_log_std), _ptr(d_alpha), p, n, _stream()))


def adam_cfg(lr0=2.5e-4, lr_final=0.0, total_steps=1, beta1=0.9, beta2=0.999, eps=1e-8, max_grad_norm=0.0) -> AdamCfg:
    return AdamCfg(lr0, lr_final, total_steps, beta1, beta2, eps, max_grad_norm)


def ver_adam_workspace_bytes() -> int:
    return lib.ver_adam_workspace_bytes()


def ver_adam_step(cfg, params, grads, exp_avg, exp_avg_sq, step_index, grad_norm, workspace):
    """params, grads, exp_avg, exp_avg_sq: lists of float32 device tensors of equal shapes."""
    sizes = (C.c_int64 * len(params))(*[t.numel() for t in params])
    p, n = _ws(workspace)
    _check(lib.ver_adam_step(C.byref(cfg), len(params), _ptr_array(params), _ptr_array(grads), _ptr_array(exp_avg),
                             _ptr_array(exp_avg_sq), sizes, step_index, _ptr(grad_norm), p, n, _stream()))


def ver_adam_step_bounded(cfg, params, grads, exp_avg, exp_avg_sq, lower, upper, step_index, grad_norm, workspace):
    """lower, upper: one float per tensor (None = unbounded for all tensors)."""
    sizes = (C.c_int64 * len(params))(*[t.numel() for t in params])
    lo = (C.c_float * len(params))(*lower) if lower is not None else None
    hi = (C.c_float * len(params))(*upper) if upper is not None else None
    p, n = _ws(workspace)
    _check(lib.ver_adam_step_bounded(C.byref(cfg), len(params), _ptr_array(params), _ptr_array(grads),
                                     _ptr_array(exp_avg), _ptr_array(exp_avg_sq), sizes, lo, hi, step_index,
                                     _ptr(grad_norm), p, n, _stream()))


def ver_profile_enable(mask: int) -> None:
    _check(lib.ver_profile_enable(mask))


def ver_profile_read() -> dict:
    """{class name: (total milliseconds, launches)} since the last read."""
    n = len(PROF_CLASSES)
    ms, cnt = (C.c_double * n)(), (C.c_int64 * n)()
    _check(lib.ver_profile_read(ms, cnt))
    return {name: (ms[i], cnt[i]) for i, name in enumerate(PROF_CLASSES)}


def workspace(n_bytes: int) -> torch.Tensor:
    """Device scratch of at least n_bytes (torch owns the memory)."""
    return torch.empty(max(1, (n_bytes + 3) // 4), dtype=torch.int32, device="cuda")
