"""Pruned RNN-T loss (Kuang et al., arXiv 2206.13236) on MI355X (gfx950).

Every stage runs in the hand-written HIP kernels of ``librnnt_pruned.so``;
this package only marshals arguments through its C ABI (ctypes). PyTorch
provides device memory and the current stream. The functions named like the
C entry points (``rnnt_simple_loss`` ...) map one-to-one onto them; the
``PrunedRnntLoss`` helper chains the four stages the way the paper's training
step does (Sec. 3.3: loss = pruned + 0.5 * simple).
"""
from __future__ import annotations

import ctypes
import math
from typing import Optional

import torch

from ._native import (RNNT_BF16, RNNT_EHIP, RNNT_EINVAL, RNNT_EUNSUPPORTED, RNNT_EWORKSPACE,  # noqa: F401
                      RNNT_F32, RNNT_FLAGS, RNNT_OK, RNNT_REDUCE_MEAN, RNNT_REDUCE_SUM, RnntBatch, RnntError, RnntScaled,
                      RnntStep, check, lib)

__all__ = [
    "Batch", "RnntError", "rnnt_simple_loss", "rnnt_simple_loss_backward", "rnnt_prune_ranges",
    "rnnt_pruned_joiner", "pruned_rnnt_loss", "rnnt_full_loss", "full_loss_workspace_size",
    "rnnt_pruned_loss", "rnnt_pruned_joiner_backward", "simple_loss_workspace_size",
    "pruned_joiner_workspace_size", "pruned_loss_workspace_size", "BAND_ALGORITHMS",
    "pruned_joiner_backward_workspace_size", "PrunedRnntLoss", "RNNT_F32", "RNNT_BF16",
    "rnnt_combine_losses", "rnnt_validate_inputs", "RNNT_FLAGS", "rnnt_pruned_loss_noalloc",
    "backward_chunk_rows",
]


def _p(t: Optional[torch.Tensor]):
    return None if t is None else ctypes.c_void_p(t.data_ptr())


def _stream(stream) -> ctypes.c_void_p:
    if stream is None:
        stream = torch.cuda.current_stream()
    if isinstance(stream, torch.cuda.Stream):
        stream = stream.cuda_stream
    return ctypes.c_void_p(int(stream))


def _need(t: torch.Tensor, name: str, dtype: torch.dtype, shape: tuple):
    if not isinstance(t, torch.Tensor):
        raise TypeError(f"{name} must be a tensor")
    if t.device.type != "cuda":
        raise ValueError(f"{name} must be a device (cuda) tensor")
    if t.dtype != dtype:
        raise TypeError(f"{name} must be {dtype}, got {t.dtype}")
    if tuple(t.shape) != tuple(shape):
        raise ValueError(f"{name} must have shape {tuple(shape)}, got {tuple(t.shape)}")
    if not t.is_contiguous():
        raise ValueError(f"{name} must be contiguous")


def _array(t: Optional[torch.Tensor], name: str, dtype: torch.dtype, *shape: int):
    """A caller's array that a kernel reads or writes densely: None, or contiguous device memory that holds the shape
    (in any shape of its own)."""
    if t is None:
        return
    if not isinstance(t, torch.Tensor):
        raise TypeError(f"{name} must be a tensor")
    if t.device.type != "cuda":
        raise ValueError(f"{name} must be a device (cuda) tensor")
    if t.dtype != dtype:
        raise TypeError(f"{name} must be {dtype}, got {t.dtype}")
    if not t.is_contiguous() or t.numel() < math.prod(shape):
        raise ValueError(f"{name} must be contiguous with at least the elements of {shape}, got {tuple(t.shape)}")


def _ws(nbytes: int, device, workspace: Optional[torch.Tensor]) -> torch.Tensor:
    if workspace is not None:
        if workspace.numel() * workspace.element_size() < nbytes:
            raise ValueError(f"workspace has {workspace.numel()} bytes, {nbytes} needed")
        return workspace
    return torch.empty(max(nbytes, 1), dtype=torch.uint8, device=device)


def _jdtype(t: torch.Tensor) -> int:
    if t.dtype == torch.float32:
        return RNNT_F32
    if t.dtype == torch.bfloat16:
        return RNNT_BF16
    raise TypeError(f"joiner tensors must be float32 or bfloat16, got {t.dtype}")


class Batch:
    """Device description of a padded batch (the C ``rnnt_batch``).

    t_len [N], u_len [N] and symbols [N, U] are int32 device tensors;
    symbols[n, u] is y_{u+1}. T and U are the padded maxima.
    """

    def __init__(self, t_len: torch.Tensor, u_len: torch.Tensor, symbols: torch.Tensor,
                 T: int, U: int, blank: int = 0):
        N = int(t_len.shape[0])
        _need(t_len, "t_len", torch.int32, (N,))
        _need(u_len, "u_len", torch.int32, (N,))
        _need(symbols, "symbols", torch.int32, (N, U))
        self.t_len, self.u_len, self.symbols = t_len, u_len, symbols
        self.N, self.T, self.U, self.blank = N, int(T), int(U), int(blank)
        self.device = t_len.device
        self._c = RnntBatch(self.N, self.T, self.U, t_len.data_ptr(), u_len.data_ptr(),
                            symbols.data_ptr() if U > 0 else None, self.blank)

    @property
    def c(self):
        return ctypes.byref(self._c)


# --------------------------------------------------------------------------
# workspace queries
# --------------------------------------------------------------------------

def simple_loss_workspace_size(N, T, U, V) -> int:
    return int(lib().rnnt_simple_loss_workspace_size(N, T, U, V))


def pruned_joiner_workspace_size(N, T, S, J, V, dtype) -> int:
    return int(lib().rnnt_pruned_joiner_workspace_size(N, T, S, J, V, dtype))


def pruned_loss_workspace_size(N, T, U, S, algorithm=None, chunk=0) -> int:
    if algorithm is None:
        return int(lib().rnnt_pruned_loss_workspace_size(N, T, U, S))
    return int(lib().rnnt_pruned_loss_ex_workspace_size(N, T, U, S, BAND_ALGORITHMS[algorithm], chunk))


def pruned_joiner_backward_workspace_size(N, T, U, S, J, V, dtype, chunk_rows: int = 0) -> int:
    if chunk_rows == 0:
        return int(lib().rnnt_pruned_joiner_backward_workspace_size(N, T, U, S, J, V, dtype))
    return int(lib().rnnt_pruned_joiner_backward_ex_workspace_size(N, T, U, S, J, V, dtype, chunk_rows))


# --------------------------------------------------------------------------
# stage wrappers (same names and argument order as the C ABI)
# --------------------------------------------------------------------------

def rnnt_simple_loss(batch: Batch, V: int, am: torch.Tensor, lm: torch.Tensor,
                     scale: Optional[torch.Tensor] = None, loss=None, px_occ=None, py_occ=None,
                     px=None, py=None, am_grad=None, lm_grad=None, workspace=None, stream=None,
                     want_logprobs: bool = False, want_grads: bool = False, lm_only_scale: float = 0.0,
                     am_only_scale: float = 0.0) -> dict:
    N, T, U = batch.N, batch.T, batch.U
    dev = batch.device
    _need(am, "am", torch.float32, (N, T, V))
    _need(lm, "lm", torch.float32, (N, U + 1, V))
    _array(loss, "loss", torch.float32, N)
    for name, t in (("px_occ", px_occ), ("py_occ", py_occ), ("px", px), ("py", py)):
        _array(t, name, torch.float32, N, T, U + 1)
    _array(am_grad, "am_grad", torch.float32, N, T, V)
    _array(lm_grad, "lm_grad", torch.float32, N, U + 1, V)
    f32 = dict(dtype=torch.float32, device=dev)
    loss = torch.empty(N, **f32) if loss is None else loss
    px_occ = torch.empty(N, T, U + 1, **f32) if px_occ is None else px_occ
    py_occ = torch.empty(N, T, U + 1, **f32) if py_occ is None else py_occ
    if want_logprobs and px is None:
        px, py = torch.empty(N, T, U + 1, **f32), torch.empty(N, T, U + 1, **f32)
    if want_grads and am_grad is None:
        am_grad, lm_grad = torch.empty(N, T, V, **f32), torch.empty(N, U + 1, V, **f32)
    if scale is not None:
        _need(scale, "scale", torch.float32, (N,))
    ws = _ws(simple_loss_workspace_size(N, T, U, V), dev, workspace)
    check(lib().rnnt_simple_loss(batch.c, V, _p(am), _p(lm), _p(scale), float(lm_only_scale),
                                 float(am_only_scale), _p(loss), _p(px_occ),
                                 _p(py_occ), _p(px), _p(py), _p(am_grad), _p(lm_grad), _p(ws),
                                 ws.numel(), _stream(stream)))
    return {"loss": loss, "px_occ": px_occ, "py_occ": py_occ, "px": px, "py": py,
            "am_grad": am_grad, "lm_grad": lm_grad}


def rnnt_simple_loss_backward(batch: Batch, V: int, am: torch.Tensor, lm: torch.Tensor, px_occ: torch.Tensor,
                              workspace: torch.Tensor, scale: Optional[torch.Tensor] = None, am_grad=None,
                              lm_grad=None, stream=None, lm_only_scale: float = 0.0,
                              am_only_scale: float = 0.0) -> dict:
    """d am, d lm from the state a preceding rnnt_simple_loss call left in ``workspace``."""
    N, T, U = batch.N, batch.T, batch.U
    dev = batch.device
    _need(am, "am", torch.float32, (N, T, V))
    _need(lm, "lm", torch.float32, (N, U + 1, V))
    _need(px_occ, "px_occ", torch.float32, (N, T, U + 1))
    _array(am_grad, "am_grad", torch.float32, N, T, V)
    _array(lm_grad, "lm_grad", torch.float32, N, U + 1, V)
    if scale is not None:
        _need(scale, "scale", torch.float32, (N,))
    f32 = dict(dtype=torch.float32, device=dev)
    am_grad = torch.empty(N, T, V, **f32) if am_grad is None else am_grad
    lm_grad = torch.empty(N, U + 1, V, **f32) if lm_grad is None else lm_grad
    ws = _ws(simple_loss_workspace_size(N, T, U, V), dev, workspace)
    check(lib().rnnt_simple_loss_backward(batch.c, V, _p(am), _p(lm), _p(scale), float(lm_only_scale),
                                          float(am_only_scale), _p(px_occ), _p(am_grad),
                                          _p(lm_grad), _p(ws), ws.numel(), _stream(stream)))
    return {"am_grad": am_grad, "lm_grad": lm_grad}


def rnnt_prune_ranges(batch: Batch, S: int, px_occ: torch.Tensor, py_occ: torch.Tensor,
                      ranges: Optional[torch.Tensor] = None, stream=None) -> torch.Tensor:
    N, T, U = batch.N, batch.T, batch.U
    _need(px_occ, "px_occ", torch.float32, (N, T, U + 1))
    _need(py_occ, "py_occ", torch.float32, (N, T, U + 1))
    _array(ranges, "ranges", torch.int32, N, T, S)
    ranges = torch.empty(N, T, S, dtype=torch.int32, device=batch.device) if ranges is None else ranges
    check(lib().rnnt_prune_ranges(batch.c, S, _p(px_occ), _p(py_occ), _p(ranges), _stream(stream)))
    return ranges


def backward_chunk_rows(N, T, S, J, V, dtype, chunk_rows: int = 0) -> int:
    """Rows of the joiner backward's chunk (the head's rows)."""
    return int(lib().rnnt_pruned_joiner_backward_chunk_rows(N, T, S, J, V, dtype, chunk_rows))


def rnnt_pruned_joiner(batch: Batch, S: int, enc: torch.Tensor, dec: torch.Tensor, W: torch.Tensor,
                       bias: Optional[torch.Tensor], ranges: torch.Tensor, px=None, py=None, lse=None,
                       logits=None, workspace=None, stream=None, keep_logits: bool = False, head=None,
                       head_rows: int = 0) -> dict:
    """The pruned joiner; with ``head`` ([head_rows, ldl] fp32) it calls
    rnnt_pruned_joiner_ex, which also keeps the first chunk's logits there."""
    N, T, U = batch.N, batch.T, batch.U
    J, V = int(W.shape[0]), int(W.shape[1])
    dt = _jdtype(W)
    _need(enc, "enc", W.dtype, (N, T, J))
    _need(dec, "dec", W.dtype, (N, U + 1, J))
    _need(W, "W", W.dtype, (J, V))
    if bias is not None:
        _need(bias, "bias", W.dtype, (V,))
    _need(ranges, "ranges", torch.int32, (N, T, S))
    for name, t in (("px", px), ("py", py), ("lse", lse)):
        _array(t, name, torch.float32, N, T, S)
    f32 = dict(dtype=torch.float32, device=batch.device)
    px = torch.empty(N, T, S, **f32) if px is None else px
    py = torch.empty(N, T, S, **f32) if py is None else py
    lse = torch.empty(N, T, S, **f32) if lse is None else lse
    if keep_logits and logits is None:
        logits = torch.empty(N, T, S, V, **f32)
    if logits is not None:
        _need(logits, "logits", torch.float32, (N, T, S, V))
    ws = _ws(pruned_joiner_workspace_size(N, T, S, J, V, dt), batch.device, workspace)
    if head is None:
        check(lib().rnnt_pruned_joiner(batch.c, S, J, V, dt, _p(enc), _p(dec), _p(W), _p(bias), _p(ranges),
                                       _p(px), _p(py), _p(lse), _p(logits), _p(ws), ws.numel(), _stream(stream)))
    else:
        _need(head, "head", torch.float32, (head_rows, (V + 7) // 8 * 8))
        check(lib().rnnt_pruned_joiner_ex(batch.c, S, J, V, dt, _p(enc), _p(dec), _p(W), _p(bias), _p(ranges),
                                          _p(px), _p(py), _p(lse), _p(logits), _p(head), int(head_rows), _p(ws),
                                          ws.numel(), _stream(stream)))
    return {"px": px, "py": py, "lse": lse, "logits": logits}


# algorithms of the pruned recursion (rnnt_pruned_loss_ex)
BAND_ALGORITHMS = {"auto": 0, "wavefront": 1, "scan": 2}


def rnnt_pruned_loss(batch: Batch, S: int, px: torch.Tensor, py: torch.Tensor, ranges: torch.Tensor,
                     loss=None, px_occ=None, py_occ=None, workspace=None, stream=None,
                     want_occupations: bool = True, algorithm: str = None, chunk: int = 0) -> dict:
    """The pruned recursion; `algorithm` ("auto", "wavefront" or "scan") and
    `chunk` select rnnt_pruned_loss_ex, None calls rnnt_pruned_loss."""
    N, T = batch.N, batch.T
    _need(px, "px", torch.float32, (N, T, S))
    _need(py, "py", torch.float32, (N, T, S))
    _need(ranges, "ranges", torch.int32, (N, T, S))
    _array(loss, "loss", torch.float32, N)
    _array(px_occ, "px_occ", torch.float32, N, T, S)
    _array(py_occ, "py_occ", torch.float32, N, T, S)
    f32 = dict(dtype=torch.float32, device=batch.device)
    loss = torch.empty(N, **f32) if loss is None else loss
    if want_occupations and px_occ is None:
        px_occ, py_occ = torch.empty(N, T, S, **f32), torch.empty(N, T, S, **f32)
    ws = _ws(pruned_loss_workspace_size(N, T, batch.U, S, algorithm, chunk), batch.device, workspace)
    if algorithm is None:
        check(lib().rnnt_pruned_loss(batch.c, S, _p(px), _p(py), _p(ranges), _p(loss), _p(px_occ), _p(py_occ),
                                     _p(ws), ws.numel(), _stream(stream)))
    else:
        check(lib().rnnt_pruned_loss_ex(batch.c, S, BAND_ALGORITHMS[algorithm], chunk, _p(px), _p(py),
                                        _p(ranges), _p(loss), _p(px_occ), _p(py_occ), _p(ws), ws.numel(),
                                        _stream(stream)))
    return {"loss": loss, "px_occ": px_occ, "py_occ": py_occ}


def rnnt_pruned_loss_noalloc(batch: Batch, S: int, px: torch.Tensor, py: torch.Tensor, ranges: torch.Tensor,
                             loss=None, px_occ=None, py_occ=None, stream=None) -> dict:
    """rnnt_pruned_loss with its workspace in the library's static device
    scratch (no allocation in the call; overlapping calls on one GPU race)."""
    N, T = batch.N, batch.T
    _need(px, "px", torch.float32, (N, T, S))
    _need(py, "py", torch.float32, (N, T, S))
    _need(ranges, "ranges", torch.int32, (N, T, S))
    _array(loss, "loss", torch.float32, N)
    _array(px_occ, "px_occ", torch.float32, N, T, S)
    _array(py_occ, "py_occ", torch.float32, N, T, S)
    f32 = dict(dtype=torch.float32, device=batch.device)
    loss = torch.empty(N, **f32) if loss is None else loss
    check(lib().rnnt_pruned_loss_noalloc(batch.c, S, _p(px), _p(py), _p(ranges), _p(loss), _p(px_occ), _p(py_occ),
                                         _stream(stream)))
    return {"loss": loss, "px_occ": px_occ, "py_occ": py_occ}


def rnnt_pruned_joiner_backward(batch: Batch, S: int, enc, dec, W, bias, ranges, lse, px_occ, py_occ,
                                scale=None, enc_grad=None, dec_grad=None, W_grad=None, bias_grad=None,
                                logits_grad=None, workspace=None, stream=None, want_param_grads=True,
                                want_logits_grad=False, logits=None, chunk_rows: int = 0, head=None,
                                head_rows: int = 0) -> dict:
    """The joiner backward; chunk_rows != 0 (a multiple of 128) or a head
    (the first chunk's logits from rnnt_pruned_joiner with ``head``) selects
    rnnt_pruned_joiner_backward_ex."""
    N, T, U = batch.N, batch.T, batch.U
    J, V = int(W.shape[0]), int(W.shape[1])
    dt = _jdtype(W)
    _need(enc, "enc", W.dtype, (N, T, J))
    _need(dec, "dec", W.dtype, (N, U + 1, J))
    _need(W, "W", W.dtype, (J, V))
    _array(bias, "bias", W.dtype, V)
    _array(scale, "scale", torch.float32, N)
    for name, t, *shape in (("enc_grad", enc_grad, N, T, J), ("dec_grad", dec_grad, N, U + 1, J),
                            ("W_grad", W_grad, J, V), ("bias_grad", bias_grad, V),
                            ("logits_grad", logits_grad, N, T, S, V)):
        _array(t, name, torch.float32, *shape)
    for name, t in (("lse", lse), ("px_occ", px_occ), ("py_occ", py_occ)):
        _need(t, name, torch.float32, (N, T, S))
    _need(ranges, "ranges", torch.int32, (N, T, S))
    if logits is not None:
        _need(logits, "logits", torch.float32, (N, T, S, V))
    f32 = dict(dtype=torch.float32, device=batch.device)
    enc_grad = torch.empty(N, T, J, **f32) if enc_grad is None else enc_grad
    dec_grad = torch.empty(N, U + 1, J, **f32) if dec_grad is None else dec_grad
    if want_param_grads and W_grad is None:
        W_grad, bias_grad = torch.empty(J, V, **f32), torch.empty(V, **f32)
    if want_logits_grad and logits_grad is None:
        logits_grad = torch.empty(N, T, S, V, **f32)
    ws = _ws(pruned_joiner_backward_workspace_size(N, T, U, S, J, V, dt, chunk_rows), batch.device, workspace)
    rest = (_p(enc), _p(dec), _p(W), _p(bias), _p(ranges), _p(lse), _p(logits), _p(px_occ), _p(py_occ), _p(scale),
            _p(enc_grad), _p(dec_grad), _p(W_grad), _p(bias_grad), _p(logits_grad), _p(ws), ws.numel(),
            _stream(stream))
    if chunk_rows == 0 and head is None:
        check(lib().rnnt_pruned_joiner_backward(batch.c, S, J, V, dt, *rest))
    else:
        if head is not None:
            _need(head, "head", torch.float32, (head_rows, (V + 7) // 8 * 8))
        check(lib().rnnt_pruned_joiner_backward_ex(batch.c, S, J, V, dt, int(chunk_rows), *rest[:7], _p(head),
                                                   int(head_rows), *rest[7:]))
    return {"enc_grad": enc_grad, "dec_grad": dec_grad, "W_grad": W_grad, "bias_grad": bias_grad,
            "logits_grad": logits_grad}


_REDUCTIONS = {"sum": RNNT_REDUCE_SUM, "mean": RNNT_REDUCE_MEAN}


def rnnt_combine_losses(simple_loss: Optional[torch.Tensor], pruned_loss: Optional[torch.Tensor],
                        simple_scale: float, pruned_scale: float, reduction: str = "sum", loss=None, total=None,
                        stream=None) -> dict:
    """The training loss of Sec. 3.3 per utterance and summed (or averaged), in the library."""
    ref = simple_loss if simple_loss is not None else pruned_loss
    N = int(ref.shape[0])
    for name, t in (("simple_loss", simple_loss), ("pruned_loss", pruned_loss)):
        if t is not None:
            _need(t, name, torch.float32, (N,))
    _array(loss, "loss", torch.float32, N)
    _array(total, "total", torch.float32)
    f32 = dict(dtype=torch.float32, device=ref.device)
    loss = torch.empty(N, **f32) if loss is None else loss
    total = torch.empty((), **f32) if total is None else total
    check(lib().rnnt_combine_losses(N, _p(simple_loss), _p(pruned_loss), float(simple_scale), float(pruned_scale),
                                    _REDUCTIONS[reduction], _p(loss), _p(total), _stream(stream)))
    return {"loss": loss, "total": total}


def rnnt_validate_inputs(batch: Batch, V: int, S: int = 0, am=None, lm=None, enc=None, dec=None, flags=None,
                         stream=None) -> dict:
    """Synchronous check of a batch (Sec. 2's problem statement; the band
    condition for S > 0). Returns the per-utterance flag tensor, the number of
    flagged utterances and, per flagged utterance, the names of its flags."""
    N, T, U = batch.N, batch.T, batch.U
    if am is not None:
        _need(am, "am", torch.float32, (N, T, V))
    if lm is not None:
        _need(lm, "lm", torch.float32, (N, U + 1, V))
    J, dt = 0, RNNT_F32
    if enc is not None or dec is not None:
        ref = enc if enc is not None else dec
        J, dt = int(ref.shape[-1]), _jdtype(ref)
        if enc is not None:
            _need(enc, "enc", ref.dtype, (N, T, J))
        if dec is not None:
            _need(dec, "dec", ref.dtype, (N, U + 1, J))
    _array(flags, "flags", torch.int32, N)
    flags = torch.empty(N, dtype=torch.int32, device=batch.device) if flags is None else flags
    n_bad = ctypes.c_int32(0)
    check(lib().rnnt_validate_inputs(batch.c, V, S, J, dt, _p(am), _p(lm), _p(enc), _p(dec), _p(flags),
                                     ctypes.byref(n_bad), _stream(stream)))
    fl = flags.cpu().tolist()
    bad = {n: [k for k, bit in RNNT_FLAGS.items() if f & bit] for n, f in enumerate(fl) if f}
    return {"flags": flags, "n_bad": int(n_bad.value), "bad": bad}


def full_loss_workspace_size(N, T, U, J, V, dtype) -> int:
    return int(lib().rnnt_full_loss_workspace_size(N, T, U, J, V, dtype))


def rnnt_full_loss(batch: Batch, enc, dec, W, bias=None, scale=None, keep_logits: bool = False, loss=None,
                   enc_grad=None, dec_grad=None, W_grad=None, bias_grad=None, logits=None, workspace=None,
                   stream=None) -> dict:
    """The unpruned RNN-T loss with the same joiner at every (t, u), and its gradients."""
    N, T, U = batch.N, batch.T, batch.U
    J, V = int(W.shape[0]), int(W.shape[1])
    dt = _jdtype(W)
    _need(enc, "enc", W.dtype, (N, T, J))
    _need(dec, "dec", W.dtype, (N, U + 1, J))
    _need(W, "W", W.dtype, (J, V))
    if bias is not None:
        _need(bias, "bias", W.dtype, (V,))
    if scale is not None:
        _need(scale, "scale", torch.float32, (N,))
    for name, t, *shape in (("loss", loss, N), ("enc_grad", enc_grad, N, T, J), ("dec_grad", dec_grad, N, U + 1, J),
                            ("W_grad", W_grad, J, V), ("bias_grad", bias_grad, V), ("logits", logits, N, T, U + 1, V)):
        _array(t, name, torch.float32, *shape)
    f32 = dict(dtype=torch.float32, device=batch.device)
    loss = torch.empty(N, **f32) if loss is None else loss
    enc_grad = torch.empty(N, T, J, **f32) if enc_grad is None else enc_grad
    dec_grad = torch.empty(N, U + 1, J, **f32) if dec_grad is None else dec_grad
    W_grad = torch.empty(J, V, **f32) if W_grad is None else W_grad
    bias_grad = torch.empty(V, **f32) if bias_grad is None else bias_grad
    if keep_logits and logits is None:
        logits = torch.empty(N, T, U + 1, V, **f32)
    ws = _ws(full_loss_workspace_size(N, T, U, J, V, dt), batch.device, workspace)
    check(lib().rnnt_full_loss(batch.c, J, V, dt, _p(enc), _p(dec), _p(W), _p(bias), _p(scale), _p(loss),
                               _p(enc_grad), _p(dec_grad), _p(W_grad), _p(bias_grad), _p(logits), _p(ws),
                               ws.numel(), _stream(stream)))
    return {"loss": loss, "enc_grad": enc_grad, "dec_grad": dec_grad, "W_grad": W_grad, "bias_grad": bias_grad,
            "logits": logits}


class PrunedRnntLoss:
    """The paper's training loss on one batch: pruned_scale * pruned + simple_scale * simple (Sec. 3.3).

    Holds the intermediate tensors and two workspaces between calls, so that
    repeated steps on same-shaped batches allocate nothing new. ``step``
    enqueues the whole path on the caller's stream: the simple loss and its
    occupations, the pruning bounds, the pruned joiner, the pruned recursion
    and the joiner backward. The simple loss's own gradients (two
    contractions that only the caller needs) run on a second stream at the
    default priority, forked after the joiner forward so that they overlap
    the pruned recursion, which occupies a few workgroups per utterance; the
    combined loss follows them there once the pruned loss is final (beside
    the joiner backward), and the stream is joined back before ``step``
    returns (in stream order). Small batches stay on the caller's stream.

    With ``pruned_scale == 0`` (the warm-up of Sec. 4: the pruned part is
    disabled until the simple loss gives useful bounds) the pruned stages are
    skipped and their loss and gradients are zero.

    By default no [N, T, S, V] array is kept: the backward recomputes the
    logits in chunks of rows whose size does not depend on N or T. With
    ``keep_logits`` the pruned logits [N, T, S, V] are stored by the forward
    and streamed by the backward instead, in one chunk of all rows (one GEMM
    less, the logits' memory more). ``bwd_chunk_rows`` (a multiple of 128, 0 = the library's choice)
    sets the backward's chunk. With ``keep_head`` (default) the forward keeps
    the logits of the backward's first chunk only (at most 16,384 rows, a
    buffer whose size does not depend on N or T), so that the backward
    streams that chunk instead of recomputing it.

    ``step`` also returns the training loss per utterance (``loss``) and its
    sum or mean (``total``), formed by the library (rnnt_combine_losses).

    ``lm_only_scale`` and ``am_only_scale`` smooth the simple loss's joiner
    (Sec. 3.3.1); both 0 gives the plain trivial joiner.
    """

    def __init__(self, S: int, simple_scale: float = 0.5, pruned_scale: float = 1.0,
                 keep_logits: bool = False, overlap: bool = True, lm_only_scale: float = 0.0,
                 am_only_scale: float = 0.0, bwd_chunk_rows: int = 0, keep_head: bool = True):
        self.S = int(S)
        self.simple_scale = float(simple_scale)
        self.pruned_scale = float(pruned_scale)
        self.lm_only_scale = float(lm_only_scale)
        self.am_only_scale = float(am_only_scale)
        self.keep_logits = bool(keep_logits)
        self.overlap = bool(overlap)
        self.bwd_chunk_rows = int(bwd_chunk_rows)
        self.keep_head = bool(keep_head)
        self._cache = {}
        self._size_cache = {}
        self._side = {}

    def _buf(self, key, shape, dtype, device):
        t = self._cache.get(key)
        if t is None or tuple(t.shape) != tuple(shape) or t.dtype != dtype or t.device != device:
            t = torch.empty(shape, dtype=dtype, device=device)
            self._cache[key] = t
        return t

    def _side_stream(self, device):
        key = device.index if device.index is not None else torch.cuda.current_device()
        if key not in self._side:
            stream = torch.cuda.Stream(device=device)
            events = [torch.cuda.Event() for _ in range(3)]
            for e in events:
                e.record(stream)  # creates the event, whose handle the step passes on
            self._side[key] = (stream, events)
        return self._side[key]

    def _sizes(self, key):
        """Workspace bytes, the backward's chunk request and the head's rows: functions of the key's sizes and options."""
        got = self._size_cache.get(key)
        if got is None:
            N, T, U, V, S, J, dt, keep_logits, keep_head, chunk = key
            if keep_logits and chunk == 0:
                # the caller keeps all the logits anyway: one chunk of every row
                # (fewer, fuller launches) unless that breaks the 32-bit limit
                whole = (N * T * S + 127) // 128 * 128
                chunk = whole if backward_chunk_rows(N, T, S, J, V, dt, whole) else 0
            head = not keep_logits and keep_head
            got = (simple_loss_workspace_size(N, T, U, V),
                   max(pruned_joiner_workspace_size(N, T, S, J, V, dt), pruned_loss_workspace_size(N, T, U, S),
                       pruned_joiner_backward_workspace_size(N, T, U, S, J, V, dt, chunk)),
                   chunk, backward_chunk_rows(N, T, S, J, V, dt, chunk) if head else 0)
            if len(self._size_cache) >= 256:
                self._size_cache.clear()
            self._size_cache[key] = got
        return got

    def step(self, batch: Batch, am, lm, enc, dec, W, bias=None, stream=None, out=None,
             reduction: str = "sum") -> dict:
        """Run one step; ``out`` optionally maps output names to caller-owned
        tensors; ``reduction`` ("sum" or "mean") is that of ``total``."""
        N, T, U, S = batch.N, batch.T, batch.U, self.S
        V = int(am.shape[2])
        J = int(W.shape[0])
        dev = batch.device
        dt = _jdtype(W)
        f32 = torch.float32
        out = {} if out is None else out
        main = torch.cuda.current_stream(dev) if stream is None else stream
        reduce = _REDUCTIONS[reduction]

        def o(key, shape, dtype=f32):
            t = out.get(key)
            return t if t is not None else self._buf(key, shape, dtype, dev)

        _need(am, "am", f32, (N, T, V))
        _need(lm, "lm", f32, (N, U + 1, V))
        lat, band = (N, T, U + 1), (N, T, S)
        if self.pruned_scale != 0.0:
            _need(enc, "enc", W.dtype, (N, T, J))
            _need(dec, "dec", W.dtype, (N, U + 1, J))
            _need(W, "W", W.dtype, (J, V))
            if bias is not None:
                _need(bias, "bias", W.dtype, (V,))
            # arrays that a later stage reads back have their shape, the others room for what is written
            back = {"simple_loss": (N,), "pruned_loss": (N,), "simple_px_occ": lat, "simple_py_occ": lat, "ranges": band,
                    "px": band, "py": band, "lse": band, "pruned_px_occ": band, "pruned_py_occ": band}
            if self.keep_logits:
                back["logits"] = (N, T, S, V)
            written = {"am_grad": (N, T, V), "lm_grad": (N, U + 1, V), "enc_grad": (N, T, J), "dec_grad": (N, U + 1, J),
                       "W_grad": (J, V), "bias_grad": (V,), "loss": (N,), "total": ()}
            for name, t in out.items():
                if name in written:
                    _array(t, name, f32, *written[name])
                elif name in back and t is not None:
                    _need(t, name, torch.int32 if name == "ranges" else f32, back[name])
        key = (N, T, U, V, S, J, dt, self.keep_logits, self.keep_head, self.bwd_chunk_rows)
        sizes, kept = self._size_cache.get(key), self._cache.get("ws_pruned")
        # a module's first step, or its first of these sizes: the stages up to the joiner are enqueued one by one, so
        # that what the later ones need is allocated, and the second stream set up, beside them and not before them
        # (N = 32, T = 500, U = 100, V = 500, nothing allocated yet: 957 us with all of it before them, 763 so; a small
        # batch, whose device time hides nothing, has fewer calls without: 206 against 222 at N = 2, T = 20, V = 16)
        large = N * T * (U + 1) * V >= _OVERLAP_WORK
        fresh = large and (sizes is None or kept is None or kept.numel() != sizes[1] or kept.device != dev)
        n_simple = simple_loss_workspace_size(N, T, U, V) if fresh else self._sizes(key)[0]
        ws_s = self._buf("ws_simple", (n_simple,), torch.uint8, dev)
        ssc = self._buf("ssc", (N,), f32, dev)
        psc = self._buf("psc", (N,), f32, dev)
        if self._cache.get("scales") != (N, dev, self.simple_scale, self.pruned_scale):
            with torch.cuda.stream(main):
                ssc.fill_(self.simple_scale)
                psc.fill_(self.pruned_scale)
            self._cache["scales"] = (N, dev, self.simple_scale, self.pruned_scale)
        res = {"simple_loss": o("simple_loss", (N,)), "simple_px_occ": o("simple_px_occ", lat),
               "simple_py_occ": o("simple_py_occ", lat)}
        if fresh or self.pruned_scale == 0.0:
            rnnt_simple_loss(
                batch, V, am, lm, ssc, loss=res["simple_loss"], px_occ=res["simple_px_occ"],
                py_occ=res["simple_py_occ"], workspace=ws_s, stream=main, lm_only_scale=self.lm_only_scale,
                am_only_scale=self.am_only_scale)
        if self.pruned_scale != 0.0:
            _, n_pruned, chunk, head_rows = self._sizes(key)
            res["ranges"] = o("ranges", band, torch.int32)
            if fresh:
                rnnt_prune_ranges(batch, S, res["simple_px_occ"], res["simple_py_occ"], res["ranges"], stream=main)
            ws_p = self._buf("ws_pruned", (n_pruned,), torch.uint8, dev)
            res.update(px=o("px", band), py=o("py", band), lse=o("lse", band))
            logits = o("logits", (N, T, S, V)) if self.keep_logits else None
            head = self._buf("head", (head_rows, (V + 7) // 8 * 8), f32, dev) if head_rows else None
            if fresh:
                rnnt_pruned_joiner(batch, S, enc, dec, W, bias, res["ranges"], px=res["px"], py=res["py"], lse=res["lse"],
                                   logits=logits, workspace=ws_p, stream=main, head=head, head_rows=head_rows)
        res.update(am_grad=o("am_grad", (N, T, V)), lm_grad=o("lm_grad", (N, U + 1, V)), enc_grad=o("enc_grad", (N, T, J)),
                   dec_grad=o("dec_grad", (N, U + 1, J)), W_grad=o("W_grad", (J, V)), bias_grad=o("bias_grad", (V,)))

        if self.pruned_scale == 0.0:
            # warm-up: the pruned part carries no weight and is not evaluated
            rnnt_simple_loss_backward(
                batch, V, am, lm, res["simple_px_occ"], ws_s, scale=ssc, am_grad=res["am_grad"],
                lm_grad=res["lm_grad"], stream=main, lm_only_scale=self.lm_only_scale,
                am_only_scale=self.am_only_scale)
            with torch.cuda.stream(main):
                pl = o("pruned_loss", (N,))
                for t in (pl, res["enc_grad"], res["dec_grad"], res["W_grad"], res["bias_grad"]):
                    t.zero_()
            res["pruned_loss"] = pl
            res.update(rnnt_combine_losses(res["simple_loss"], None, self.simple_scale, 0.0, reduction,
                                           loss=o("loss", (N,)), total=o("total", ()), stream=main))
            return res

        res.update(pruned_loss=o("pruned_loss", (N,)), pruned_px_occ=o("pruned_px_occ", band),
                   pruned_py_occ=o("pruned_py_occ", band), loss=o("loss", (N,)), total=o("total", ()))
        # the second stream's events cost more than what it would overlap on small batches
        overlap = self.overlap and large
        side, (fork, lossev, join) = self._side_stream(dev) if overlap else (None, (None,) * 3)
        ptr = torch.Tensor.data_ptr
        p = RnntStep(
            S, J, V, dt, chunk, head_rows, reduce,
            self.simple_scale, self.pruned_scale, self.lm_only_scale, self.am_only_scale,
            ptr(am), ptr(lm), ptr(enc), ptr(dec), ptr(W), None if bias is None else ptr(bias), ptr(ssc), ptr(psc),
            ptr(res["simple_loss"]), ptr(res["simple_px_occ"]), ptr(res["simple_py_occ"]), ptr(res["am_grad"]),
            ptr(res["lm_grad"]), ptr(res["ranges"]), ptr(res["px"]), ptr(res["py"]), ptr(res["lse"]),
            None if logits is None else ptr(logits), None if head is None else ptr(head),
            ptr(res["pruned_loss"]), ptr(res["pruned_px_occ"]), ptr(res["pruned_py_occ"]), ptr(res["enc_grad"]),
            ptr(res["dec_grad"]), ptr(res["W_grad"]), ptr(res["bias_grad"]), ptr(res["loss"]), ptr(res["total"]),
            ptr(ws_s), n_simple, ptr(ws_p), n_pruned,
            side.cuda_stream if overlap else None, fork.cuda_event if overlap else None,
            lossev.cuda_event if overlap else None, join.cuda_event if overlap else None)
        run = lib().rnnt_train_step_rest if fresh else lib().rnnt_train_step
        check(run(batch.c, ctypes.byref(p), _stream(main)))
        return res


# The least N T (U+1) V for which the simple loss's gradients go to a second
# stream: its three events cost the host 36 us a step, while on one stream the
# gradients add 11 us at the tiny test batch and 29 us at the BPE batch
# (1.2e8), where the host is ahead of the device.
_OVERLAP_WORK = 1 << 24


def _scaled_gradients(g, divisor: float, saved, dtypes, has_bias: bool):
    """The stored gradients times g / divisor in their inputs' dtypes, in one launch (g: the loss's gradient, a
    device scalar)."""
    ed, dd, wd = dtypes
    f32 = torch.float32
    grads = [torch.empty_like(t, dtype=d) for t, d in zip(saved, (f32, f32, ed, dd, wd, wd))]
    g = g.to(f32).contiguous()
    n = 6 if has_bias else 5
    arrays = (RnntScaled * 6)(*[(t.data_ptr(), r.data_ptr(), t.numel(), RNNT_BF16 if r.dtype == torch.bfloat16 else RNNT_F32)
                                for t, r in zip(saved, grads)])
    check(lib().rnnt_scale_gradients(n, arrays, g.data_ptr(), divisor, _stream(None)))
    return grads if has_bias else grads[:5] + [None]


def _readable(t: torch.Tensor) -> bool:
    """Whether a kernel can read t through its address and nothing of it is lost by that: a plain CUDA tensor, no
    subclass, no vmap or functorch wrapper (which have no storage) and no forward-mode dual."""
    if type(t) is not torch.Tensor or not t.is_cuda or torch.autograd.forward_ad.unpack_dual(t).tangent is not None:
        return False
    try:
        t.data_ptr()
    except RuntimeError:
        return False
    return True


class _PrunedRnntFunction(torch.autograd.Function):
    """Forward computes the loss and every gradient at once (the kernels are
    fused forward-backward); backward scales the stored gradients."""

    @staticmethod
    def forward(ctx, am, lm, enc, dec, W, bias, module, batch, reduction):
        N, T, U, V, J = batch.N, batch.T, batch.U, int(am.shape[2]), int(W.shape[0])
        f32 = dict(dtype=torch.float32, device=am.device)
        fresh = {"am_grad": torch.empty(N, T, V, **f32), "lm_grad": torch.empty(N, U + 1, V, **f32),
                 "enc_grad": torch.empty(N, T, J, **f32), "dec_grad": torch.empty(N, U + 1, J, **f32),
                 "W_grad": torch.empty(J, V, **f32), "bias_grad": torch.empty(V, **f32)}
        fresh["total"] = torch.empty((), **f32)
        r = module.step(batch, am, lm, enc, dec, W, bias, out=fresh, reduction=reduction)
        loss = r["total"]
        ctx.reduction = reduction
        ctx.N = N
        ctx.has_bias = bias is not None
        ctx.dtypes = (enc.dtype, dec.dtype, W.dtype)
        ctx.save_for_backward(fresh["am_grad"], fresh["lm_grad"], fresh["enc_grad"], fresh["dec_grad"],
                              fresh["W_grad"], fresh["bias_grad"])
        return loss

    @staticmethod
    def backward(ctx, g):
        saved = ctx.saved_tensors
        # (a saved-tensor hook may have replaced the stored arrays)
        plain = _readable(g) and all(_readable(t) and t.device == g.device and t.dtype == torch.float32 and
                                    t.is_contiguous() for t in saved)
        if plain and not (torch.is_grad_enabled() and g.requires_grad):
            return (*_scaled_gradients(g, float(ctx.N) if ctx.reduction == "mean" else 1.0, saved, ctx.dtypes,
                                       ctx.has_bias), None, None, None)
        # differentiated again (with respect to g), or not where the kernel could read them: torch's own products
        am_g, lm_g, enc_g, dec_g, W_g, b_g = saved
        if ctx.reduction == "mean":
            g = g / ctx.N
        ed, dd, wd = ctx.dtypes
        return (am_g * g, lm_g * g, (enc_g * g).to(ed), (dec_g * g).to(dd), (W_g * g).to(wd),
                (b_g * g).to(wd) if ctx.has_bias else None, None, None, None)


def pruned_rnnt_loss(am, lm, enc, dec, W, bias, batch: Batch, S: int, simple_scale: float = 0.5,
                     pruned_scale: float = 1.0, reduction: str = "sum", module: Optional[PrunedRnntLoss] = None,
                     lm_only_scale: float = 0.0, am_only_scale: float = 0.0):
    """Differentiable training loss: sum (or mean) over utterances of
    simple_scale * simple_loss + pruned_scale * pruned_loss (Sec. 3.3), the
    simple loss optionally with the smoothed joiner (Sec. 3.3.1)."""
    if reduction not in ("sum", "mean"):
        raise ValueError("reduction must be 'sum' or 'mean'")
    if module is None:
        module = PrunedRnntLoss(S, simple_scale=simple_scale, pruned_scale=pruned_scale,
                                lm_only_scale=lm_only_scale, am_only_scale=am_only_scale)
    return _PrunedRnntFunction.apply(am, lm, enc, dec, W, bias, module, batch, reduction)
