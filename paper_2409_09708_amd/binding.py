"""ctypes binding of libnm_sparse.so.  Argument marshalling only: every step of the path runs in the
HIP kernels behind the C ABI (include/nm_sparse.h).  torch provides device memory and the stream.  The calls made per
layer go through the native marshalling of csrc/nm_calls.cpp first, which declines what is not in the ordinary form.

Tensor conventions: weights / activations / packed values are torch.bfloat16 CUDA tensors; index and
mask words are torch.int32 tensors holding the uint32 bit patterns.
"""
from __future__ import annotations

import ctypes
import importlib.machinery
import importlib.util
import os
import struct
import sysconfig
from ctypes import c_char_p, c_int32, c_int64, c_size_t, c_void_p
from typing import List, Optional, Sequence, Tuple

_LIB = None
_CALLS = None
_PKG_DIR = os.path.dirname(os.path.abspath(__file__))

NM_OK = 0
NM_OUT_F32, NM_OUT_BF16, NM_OUT_I32 = 0, 1, 2

EXPORTS = (
    "nm_status_string", "nm_last_hip_error", "nm_values_bytes", "nm_index_bytes", "nm_mask_bytes",
    "nm_spmm_workspace_bytes", "nm_prune", "nm_pack", "nm_pack_batched", "nm_unpack", "nm_mask_check",
    "nm_spmm", "nm_linear_forward", "nm_spmm_prepare", "nm_linear_forward_prepared",
    "nm_static_scratch_bytes", "nm_linear_forward_static",
    "nm_probe_sink_bytes", "nm_probe_matrix_rate", "nm_probe_copy",
    "nm_values_i8_bytes", "nm_pack_i8", "nm_unpack_i8", "nm_linear_forward_i8_packed", "nm_i8_prepare_packed",
    "nm_linear_forward_i8_packed_prepared",
    "nm_rank_bytes", "nm_rank", "nm_rank_batched", "nm_rank_mask", "nm_pack_ranked", "nm_pack_ranked_batched", "nm_pack_prepare_batched",
    "nm_config_cost", "nm_sample_config",
    "nm_backward_input_workspace_bytes", "nm_backward_weight_workspace_bytes", "nm_linear_backward_input", "nm_backward_input_scratch_bytes", "nm_backward_input_scratch_pays", "nm_linear_backward_input_scratch", "nm_linear_backward_weight",
    "nm_backward_weight_scratch_bytes", "nm_linear_backward_weight_scratch",
    "nm_linear_forward_prepared_batched", "nm_prepared_scratch_bytes", "nm_linear_forward_prepared_scratch",
    "nm_prepared_batched_scratch_bytes", "nm_linear_forward_prepared_batched_scratch", "nm_prune_scored", "nm_i8_workspace_bytes", "nm_linear_forward_i8", "nm_i8_prepare", "nm_linear_forward_i8_prepared",
)


class NmError(RuntimeError):
    def __init__(self, status: int, text: str):
        super().__init__(f"nm_sparse status {status}: {text}")
        self.status = status


class PackDesc(ctypes.Structure):
    _fields_ = [("W", c_void_p), ("values", c_void_p), ("indices", c_void_p),
                ("O", c_int64), ("K", c_int64), ("N", c_int32), ("M", c_int32)]
    packer = struct.Struct("QQQqqii")


class PackRankedDesc(ctypes.Structure):
    _fields_ = [("W", c_void_p), ("rank", c_void_p), ("values", c_void_p), ("indices", c_void_p),
                ("O", c_int64), ("K", c_int64), ("N", c_int32), ("M", c_int32)]
    packer = struct.Struct("QQQQqqii")


class LayerDesc(ctypes.Structure):
    _fields_ = [("W", c_void_p), ("values", c_void_p), ("indices", c_void_p),
                ("O", c_int64), ("K", c_int64), ("N", c_int32), ("M", c_int32),
                ("T", c_int64), ("workspace", c_void_p), ("workspace_bytes", c_size_t)]
    packer = struct.Struct("QQQqqiiqQQ")


class RankDesc(ctypes.Structure):
    _fields_ = [("W", c_void_p), ("rank", c_void_p), ("O", c_int64), ("K", c_int64), ("M", c_int32),
                ("reserved", c_int32)]
    packer = struct.Struct("QQqqii")


def _desc_array(kind, rows):
    """Host array of descriptors of one kind from their packed rows (a quarter of the time of building the structures
    one by one, and these calls describe a whole model)."""
    return (kind * len(rows)).from_buffer_copy(b"".join(rows))


class ForwardDesc(ctypes.Structure):
    _fields_ = [("values", c_void_p), ("indices", c_void_p), ("O", c_int64), ("K", c_int64), ("N", c_int32),
                ("M", c_int32), ("X", c_void_p), ("T", c_int64), ("ldx", c_int64), ("bias", c_void_p), ("Y", c_void_p),
                ("ldy", c_int64), ("out_dtype", c_int32), ("reserved", c_int32), ("workspace", c_void_p),
                ("workspace_bytes", c_size_t)]


def library_path() -> str:
    return os.path.join(_PKG_DIR, "libnm_sparse.so")


def calls_path() -> str:
    """The native marshalling reads torch's C++ objects as they lie, so it serves the Python and the torch that it was built
    against, and its file name says which."""
    return os.path.join(_PKG_DIR, f"_nm_calls.{sysconfig.get_config_var('SOABI')}.torch-{_torch().__version__}.so")


def load_library() -> ctypes.CDLL:
    """Load the HIP library (once).  There is no fallback: a missing library is an error."""
    global _LIB
    if _LIB is not None:
        return _LIB
    path = library_path()
    if not os.path.exists(path):
        raise RuntimeError(f"{path} is missing: build it with `python -m paper_2409_09708_amd.build`")
    lib = ctypes.CDLL(path)
    lib.nm_status_string.restype = c_char_p
    lib.nm_status_string.argtypes = [c_int32]
    lib.nm_last_hip_error.restype = c_int32
    lib.nm_last_hip_error.argtypes = []
    for name in ("nm_values_bytes", "nm_index_bytes"):
        getattr(lib, name).restype = c_size_t
        getattr(lib, name).argtypes = [c_int64, c_int64, c_int32, c_int32]
    lib.nm_mask_bytes.restype = c_size_t
    lib.nm_mask_bytes.argtypes = [c_int64, c_int64]
    lib.nm_spmm_workspace_bytes.restype = c_size_t
    lib.nm_spmm_workspace_bytes.argtypes = [c_int64, c_int64, c_int32, c_int32, c_int64]
    lib.nm_prune.restype = c_int32
    lib.nm_prune.argtypes = [c_void_p, c_int64, c_int64, c_int64, c_int32, c_int32, c_void_p, c_void_p, c_void_p]
    lib.nm_pack.restype = c_int32
    lib.nm_pack.argtypes = [c_void_p, c_int64, c_int64, c_int64, c_int32, c_int32, c_void_p, c_void_p, c_void_p,
                            c_void_p]
    lib.nm_pack_batched.restype = c_int32
    lib.nm_pack_batched.argtypes = [ctypes.POINTER(PackDesc), c_int32, c_void_p]
    lib.nm_unpack.restype = c_int32
    lib.nm_unpack.argtypes = [c_void_p, c_void_p, c_int64, c_int64, c_int32, c_int32, c_void_p, c_int64, c_void_p]
    lib.nm_mask_check.restype = c_int32
    lib.nm_mask_check.argtypes = [c_void_p, c_int64, c_int64, c_int32, c_int32, c_void_p, c_void_p]
    lib.nm_spmm.restype = c_int32
    lib.nm_spmm.argtypes = [c_void_p, c_void_p, c_int64, c_int64, c_int32, c_int32, c_void_p, c_int64, c_int64,
                            c_void_p, c_int64, c_int32, c_void_p, c_size_t, c_void_p]
    lib.nm_linear_forward.restype = c_int32
    lib.nm_linear_forward.argtypes = [c_void_p, c_void_p, c_int64, c_int64, c_int32, c_int32, c_void_p, c_int64,
                                      c_int64, c_void_p, c_void_p, c_int64, c_int32, c_void_p, c_size_t, c_void_p]
    lib.nm_spmm_prepare.restype = c_int32
    lib.nm_spmm_prepare.argtypes = [c_void_p, c_void_p, c_int64, c_int64, c_int32, c_int32, c_int64, c_void_p, c_size_t,
                                    c_void_p]
    lib.nm_linear_forward_prepared.restype = c_int32
    lib.nm_linear_forward_prepared.argtypes = lib.nm_linear_forward.argtypes
    lib.nm_prepared_scratch_bytes.restype = c_size_t
    lib.nm_prepared_scratch_bytes.argtypes = [c_int64, c_int64, c_int32, c_int32, c_int64]
    lib.nm_linear_forward_prepared_scratch.restype = c_int32
    lib.nm_linear_forward_prepared_scratch.argtypes = lib.nm_linear_forward.argtypes[:-1] + [c_void_p, c_size_t, c_void_p]
    lib.nm_static_scratch_bytes.restype = c_size_t
    lib.nm_static_scratch_bytes.argtypes = []
    lib.nm_linear_forward_static.restype = c_int32
    lib.nm_linear_forward_static.argtypes = [c_void_p, c_void_p, c_int64, c_int64, c_int32, c_int32, c_void_p, c_int64,
                                             c_int64, c_void_p, c_void_p, c_int64, c_int32, c_void_p]
    lib.nm_probe_sink_bytes.restype = c_size_t
    lib.nm_probe_sink_bytes.argtypes = []
    lib.nm_probe_matrix_rate.restype = c_int32
    lib.nm_probe_matrix_rate.argtypes = [c_int32, c_int32, c_void_p, ctypes.POINTER(c_int64), c_void_p]
    lib.nm_probe_copy.restype = c_int32
    lib.nm_probe_copy.argtypes = [c_void_p, c_void_p, c_size_t, c_void_p]
    lib.nm_pack_prepare_batched.restype = c_int32
    lib.nm_pack_prepare_batched.argtypes = [ctypes.POINTER(LayerDesc), c_int32, c_void_p]
    lib.nm_rank_bytes.restype = c_size_t
    lib.nm_rank_bytes.argtypes = [c_int64, c_int64]
    lib.nm_rank.restype = c_int32
    lib.nm_rank.argtypes = [c_void_p, c_int64, c_int64, c_int64, c_int32, c_void_p, c_void_p]
    c_double_p, c_int32_p = ctypes.POINTER(ctypes.c_double), ctypes.POINTER(c_int32)
    lib.nm_config_cost.restype = ctypes.c_double
    lib.nm_config_cost.argtypes = [c_double_p, c_int32_p, c_int32_p, c_int32, ctypes.c_double]
    lib.nm_sample_config.restype = c_int32
    lib.nm_sample_config.argtypes = [c_double_p, c_int32, ctypes.c_double, c_int32_p, c_int32_p, c_int32, c_double_p,
                                     c_double_p, c_int32, c_double_p, c_int64, c_int32_p, c_int32_p,
                                     ctypes.POINTER(c_int64)]
    lib.nm_rank_batched.restype = c_int32
    lib.nm_rank_batched.argtypes = [ctypes.POINTER(RankDesc), c_int32, c_void_p]
    lib.nm_rank_mask.restype = c_int32
    lib.nm_rank_mask.argtypes = [c_void_p, c_int64, c_int64, c_int32, c_int32, c_void_p, c_void_p]
    lib.nm_pack_ranked.restype = c_int32
    lib.nm_pack_ranked.argtypes = [c_void_p, c_void_p, c_int64, c_int64, c_int64, c_int32, c_int32, c_void_p, c_void_p,
                                   c_void_p]
    lib.nm_pack_ranked_batched.restype = c_int32
    lib.nm_pack_ranked_batched.argtypes = [ctypes.POINTER(PackRankedDesc), c_int32, c_void_p]
    lib.nm_backward_weight_workspace_bytes.restype = c_size_t
    lib.nm_backward_weight_workspace_bytes.argtypes = [c_int64, c_int64, c_int64]
    lib.nm_linear_backward_input.restype = c_int32
    lib.nm_backward_input_scratch_bytes.restype = c_size_t
    lib.nm_backward_input_scratch_bytes.argtypes = [c_int64, c_int64, c_int64]
    lib.nm_backward_input_scratch_pays.restype = c_int32
    lib.nm_backward_input_scratch_pays.argtypes = [c_int64, c_int64, c_int64, c_int32, c_void_p]
    lib.nm_backward_input_workspace_bytes.restype = c_size_t
    lib.nm_backward_input_workspace_bytes.argtypes = [c_int64, c_int64, c_int64]
    lib.nm_linear_backward_input.argtypes = [c_void_p, c_int64, c_int64, c_int64, c_void_p, c_int64, c_int64, c_void_p,
                                             c_int64, c_int32, c_void_p, c_size_t, c_void_p]
    lib.nm_linear_backward_input_scratch.restype = c_int32
    lib.nm_linear_backward_input_scratch.argtypes = lib.nm_linear_backward_input.argtypes
    lib.nm_backward_weight_scratch_bytes.restype = c_size_t
    lib.nm_backward_weight_scratch_bytes.argtypes = [c_int64, c_int64, c_int64]
    lib.nm_linear_backward_weight.restype = c_int32
    lib.nm_linear_backward_weight.argtypes = [c_void_p, c_int64, c_int64, c_int64, c_void_p, c_int64, c_int64, c_void_p,
                                              c_void_p, c_int64, c_int32, c_void_p, c_size_t, c_void_p]
    lib.nm_linear_backward_weight_scratch.restype = c_int32
    lib.nm_linear_backward_weight_scratch.argtypes = lib.nm_linear_backward_weight.argtypes
    lib.nm_linear_forward_prepared_batched.restype = c_int32
    lib.nm_linear_forward_prepared_batched.argtypes = [ctypes.POINTER(ForwardDesc), c_int32, c_void_p]
    lib.nm_prepared_batched_scratch_bytes.restype = c_size_t
    lib.nm_prepared_batched_scratch_bytes.argtypes = [ctypes.POINTER(ForwardDesc), c_int32]
    lib.nm_linear_forward_prepared_batched_scratch.restype = c_int32
    lib.nm_linear_forward_prepared_batched_scratch.argtypes = [ctypes.POINTER(ForwardDesc), c_int32, c_void_p, c_size_t, c_void_p]
    lib.nm_prune_scored.restype = c_int32
    lib.nm_prune_scored.argtypes = [c_void_p, c_int64, c_int64, c_int64, c_int32, c_int32, c_void_p, c_void_p]
    lib.nm_i8_workspace_bytes.restype = c_size_t
    lib.nm_i8_workspace_bytes.argtypes = [c_int64, c_int64, c_int32, c_int32, c_int64]
    i8_args = [c_void_p, c_int64, c_int64, c_int64, c_void_p, c_int32, c_int32, c_void_p, c_int64, c_int64,
               ctypes.c_float, c_void_p, c_void_p, c_void_p, c_int64, c_int32, c_void_p, c_size_t, c_void_p]
    lib.nm_linear_forward_i8.restype = c_int32
    lib.nm_linear_forward_i8.argtypes = i8_args
    lib.nm_linear_forward_i8_prepared.restype = c_int32
    lib.nm_linear_forward_i8_prepared.argtypes = i8_args
    lib.nm_i8_prepare.restype = c_int32
    lib.nm_i8_prepare.argtypes = [c_void_p, c_int64, c_int64, c_int64, c_void_p, c_int32, c_int32, c_int64, c_void_p, c_size_t,
                                  c_void_p]
    lib.nm_values_i8_bytes.restype = c_size_t
    lib.nm_values_i8_bytes.argtypes = [c_int64, c_int64, c_int32, c_int32]
    lib.nm_pack_i8.restype = c_int32
    lib.nm_pack_i8.argtypes = [c_void_p, c_int64, c_int64, c_int64, c_int32, c_int32, c_void_p, c_void_p, c_void_p, c_void_p]
    lib.nm_unpack_i8.restype = c_int32
    lib.nm_unpack_i8.argtypes = [c_void_p, c_void_p, c_int64, c_int64, c_int32, c_int32, c_void_p, c_int64, c_void_p]
    i8p_args = [c_void_p, c_void_p, c_int64, c_int64, c_int32, c_int32, c_void_p, c_int64, c_int64, ctypes.c_float,
                c_void_p, c_void_p, c_void_p, c_int64, c_int32, c_void_p, c_size_t, c_void_p]
    lib.nm_linear_forward_i8_packed.restype = c_int32
    lib.nm_linear_forward_i8_packed.argtypes = i8p_args
    lib.nm_linear_forward_i8_packed_prepared.restype = c_int32
    lib.nm_linear_forward_i8_packed_prepared.argtypes = i8p_args
    lib.nm_i8_prepare_packed.restype = c_int32
    lib.nm_i8_prepare_packed.argtypes = [c_void_p, c_void_p, c_int64, c_int64, c_int32, c_int32, c_int64, c_void_p, c_size_t,
                                         c_void_p]
    _LIB = lib
    return lib


def _native():
    """The native marshalling, bound to the loaded library.  As with the library there is no fallback for a missing build."""
    global _CALLS
    lib = load_library()
    path = calls_path()
    if not os.path.exists(path):
        raise RuntimeError(f"{path} is missing: build it with `python -m paper_2409_09708_amd.build`")
    loader = importlib.machinery.ExtensionFileLoader("_nm_calls", path)
    calls = importlib.util.module_from_spec(importlib.util.spec_from_loader("_nm_calls", loader))
    loader.exec_module(calls)
    calls.bind({name: ctypes.cast(getattr(lib, name), c_void_p).value for name in EXPORTS}, _check, _workspace, _WORKSPACES)
    _CALLS = calls
    return calls


def nm_status_string(status: int) -> str:
    return load_library().nm_status_string(status).decode()


def _check(status: int) -> None:
    if status != NM_OK:
        raise NmError(status, nm_status_string(status))


def nm_values_bytes(O: int, K: int, N: int, M: int) -> int:
    return int(load_library().nm_values_bytes(O, K, N, M))


def nm_index_bytes(O: int, K: int, N: int, M: int) -> int:
    return int(load_library().nm_index_bytes(O, K, N, M))


def nm_mask_bytes(O: int, K: int) -> int:
    return int(load_library().nm_mask_bytes(O, K))


def nm_spmm_workspace_bytes(O: int, K: int, N: int, M: int, T: int) -> int:
    return int(load_library().nm_spmm_workspace_bytes(O, K, N, M, T))


# ------------------------------------------------------------------------------------------------
# tensor marshalling
# ------------------------------------------------------------------------------------------------
# A call on a small layer costs the host more than the device (one image through a 384 x 384 projection: 4 us of kernel,
# 3 us of launch), so what every call does is kept short: torch is imported once, the current stream is asked for as
# a raw handle (0.1 us; building a Stream object takes 2.9), and a tensor's sizes and strides are read once.
_TORCH = None


def _torch():
    global _TORCH
    if _TORCH is None:
        import torch
        _TORCH = torch
    return _TORCH


def _stream_handle(stream) -> int:
    if stream is not None:
        return int(stream.cuda_stream)
    c = _torch()._C
    return c._cuda_getCurrentRawStream(c._cuda_getDevice())


def _need(t, dtype, what: str) -> None:
    if not t.is_cuda:
        raise ValueError(f"{what} must be a device tensor")
    if t.dtype != dtype:
        raise ValueError(f"{what} must be {dtype}, got {t.dtype}")


def _rows(t, what: str) -> Tuple[int, int, int]:
    """(rows, cols, leading dimension) of a 2-D tensor whose rows are contiguous."""
    shape = t.shape
    if len(shape) == 2:
        rows, cols = shape
        ld, step = t.stride()
        if step == 1 or cols <= 1:
            return rows, cols, ld if rows > 1 else cols
    raise ValueError(f"{what} must be 2-D with unit stride along its rows")


def _contiguous_weight(W, caller: str) -> Tuple[int, int]:
    """(out-features, in-features) of a bfloat16 weight of a batched call."""
    _need(W, _torch().bfloat16, "W")
    if not W.is_contiguous():
        raise ValueError(f"{caller} needs contiguous weights")
    shape = W.shape  # (a weight with trailing dimensions of one is a matrix to these calls)
    return shape[0], shape[1]


def _packed(values, indices, dtype) -> int:
    """Out-features of a packed weight whose tensors have been checked."""
    _need(values, dtype, "values")
    _need(indices, _torch().int32, "indices")
    if not values.is_contiguous() or not indices.is_contiguous():
        raise ValueError("packed tensors must be contiguous")
    return values.shape[0]


def _per_feature(t, O: int, name: str):
    """Device pointer of an optional float32 [O] tensor."""
    if t is None:
        return None
    _need(t, _torch().float32, name)
    if t.numel() != O or not t.is_contiguous():
        raise ValueError(f"{name} must be contiguous [O]")
    return t.data_ptr()


def _mask_words(mask, O: int, K: int):
    _need(mask, _torch().int32, "mask")
    if mask.shape != (O, (K + 31) // 32) or not mask.is_contiguous():
        raise ValueError("mask must be contiguous [O, ceil(K/32)] words")
    return mask.data_ptr()


def _scratch(workspace):
    """(pointer, bytes) of an optional workspace tensor."""
    if workspace is None:
        return None, 0
    return workspace.data_ptr(), workspace.nbytes


def _empty_packed(O: int, K: int, N: int, M: int, W):
    """Uninitialised packed tensors of a weight on W's device."""
    torch = _torch()
    lib = load_library()
    vb = lib.nm_values_bytes(O, K, N, M)
    if vb == 0:  # illegal level or shape: let the library name the error (it returns before touching a pointer)
        _check(lib.nm_pack(16, O, K, K, N, M, None, 16, 16, None))
    values = W.new_empty((O, vb // (2 * O)))
    indices = W.new_empty((O, lib.nm_index_bytes(O, K, N, M) // (4 * O)), dtype=torch.int32)
    return values, indices


def nm_prune(W, N: int, M: int, W_masked=None, stream=None):
    """Mask words [O, ceil(K/32)] (int32) of Eq. (1); optionally writes the pruned weight to W_masked."""
    done = (_CALLS or _native()).prune(W, N, M, W_masked, stream)
    if done is not NotImplemented:
        return done
    torch = _torch()
    _need(W, torch.bfloat16, "W")
    O, K, ldw = _rows(W, "W")
    mask = W.new_empty((O, (K + 31) // 32), dtype=torch.int32)
    wm_ptr = None
    if W_masked is not None:
        _need(W_masked, torch.bfloat16, "W_masked")
        if _rows(W_masked, "W_masked") != (O, K, ldw):
            raise ValueError("W_masked must have the shape and leading dimension of W")
        wm_ptr = W_masked.data_ptr()
    _check(load_library().nm_prune(W.data_ptr(), O, K, ldw, N, M, mask.data_ptr(), wm_ptr, _stream_handle(stream)))
    return mask


def nm_prune_scored(score, N: int, M: int, stream=None):
    """Mask words [O, ceil(K/32)] (int32) keeping the N largest of every M scores (float32 [O, K])."""
    done = (_CALLS or _native()).prune_scored(score, N, M, stream)
    if done is not NotImplemented:
        return done
    torch = _torch()
    _need(score, torch.float32, "score")
    O, K, lds = _rows(score, "score")
    mask = score.new_empty((O, (K + 31) // 32), dtype=torch.int32)
    _check(load_library().nm_prune_scored(score.data_ptr(), O, K, lds, N, M, mask.data_ptr(), _stream_handle(stream)))
    return mask


def _doubles(xs):
    return (ctypes.c_double * len(xs))(*[float(x) for x in xs])


def _ints(xs):
    return (c_int32 * len(xs))(*[int(x) for x in xs])


def nm_config_cost(layer_macs, levels, fixed_cost: float = 0.0) -> float:
    """F(alpha) = fixed_cost + sum_l layer_macs[l] * N_l / M_l (host only)."""
    L = len(layer_macs)
    c = load_library().nm_config_cost(_doubles(layer_macs), _ints([n for n, _ in levels]), _ints([m for _, m in levels]),
                                      L, float(fixed_cost))
    if c < 0:
        raise ValueError("illegal level or layer cost")
    return float(c)


def nm_sample_config(layer_macs, fixed_cost, choices, probs, edges, uniforms):
    """Two-step sampling (host only): (interval, [choice index per layer], uniforms used); raises NmError with
    status NM_ERR_EXHAUSTED when the uniforms run out."""
    L, S = len(layer_macs), len(choices)
    flat = [float(p) for row in probs for p in row]
    choice = (c_int32 * L)()
    interval, used = c_int32(0), c_int64(0)
    _check(load_library().nm_sample_config(_doubles(layer_macs), L, float(fixed_cost), _ints([n for n, _ in choices]),
                                           _ints([m for _, m in choices]), S, _doubles(flat), _doubles(edges),
                                           len(edges), _doubles(uniforms), len(uniforms), choice,
                                           ctypes.byref(interval), ctypes.byref(used)))
    return int(interval.value), [int(c) for c in choice], int(used.value)


def nm_rank_bytes(O: int, K: int) -> int:
    return int(load_library().nm_rank_bytes(O, K))


def nm_rank(W, M: int, stream=None):
    """Ranks (uint8 [O, K/2], two 4-bit ranks per byte) of the weights inside their groups of M."""
    torch = _torch()
    _need(W, torch.bfloat16, "W")
    O, K, ldw = _rows(W, "W")
    rank = torch.empty((O, K // 2), dtype=torch.uint8, device=W.device)
    _check(load_library().nm_rank(W.data_ptr(), O, K, ldw, M, rank.data_ptr(), _stream_handle(stream)))
    return rank


def nm_rank_batched(layers: Sequence[Tuple[object, int]], stream=None, out=None):
    """One launch for many (W, M); returns the rank tensors."""
    torch = _torch()
    descs = []
    outs = []
    for i, (W, M) in enumerate(layers):
        O, K = _contiguous_weight(W, "nm_rank_batched")
        rank = out[i] if out is not None else W.new_empty((O, K // 2), dtype=torch.uint8)
        outs.append(rank)
        descs.append(RankDesc.packer.pack(W.data_ptr(), rank.data_ptr(), O, K, M, 0))
    _check(load_library().nm_rank_batched(_desc_array(RankDesc, descs), len(descs), _stream_handle(stream)))
    return outs


def _need_rank(rank, O: int, K: int) -> None:
    torch = _torch()
    _need(rank, torch.uint8, "rank")
    if rank.shape != (O, K // 2) or not rank.is_contiguous():
        raise ValueError("rank must be contiguous [O, K/2]")


def nm_rank_mask(rank, K: int, N: int, M: int, stream=None):
    """Mask words [O, ceil(K/32)] (int32) of level N:M from stored ranks: bit = rank < N."""
    torch = _torch()
    O = int(rank.shape[0])
    _need_rank(rank, O, K)
    mask = torch.empty((O, (K + 31) // 32), dtype=torch.int32, device=rank.device)
    _check(load_library().nm_rank_mask(rank.data_ptr(), O, K, N, M, mask.data_ptr(), _stream_handle(stream)))
    return mask


def nm_pack_ranked(W, rank, N: int, M: int, stream=None):
    """nm_pack with the selection read from stored ranks."""
    torch = _torch()
    _need(W, torch.bfloat16, "W")
    O, K, ldw = _rows(W, "W")
    _need_rank(rank, O, K)
    values, indices = _empty_packed(O, K, N, M, W)
    _check(load_library().nm_pack_ranked(W.data_ptr(), rank.data_ptr(), O, K, ldw, N, M, values.data_ptr(),
                                         indices.data_ptr(), _stream_handle(stream)))
    return values, indices


def nm_pack_ranked_batched(layers: Sequence[Tuple[object, object, int, int]], stream=None, out=None):
    """One launch for many (W, rank, N, M); returns [(values, indices), ...]."""
    descs = []
    outs: List[Tuple[object, object]] = []
    for i, (W, rank, N, M) in enumerate(layers):
        O, K = _contiguous_weight(W, "nm_pack_ranked_batched")
        _need_rank(rank, O, K)
        values, indices = out[i] if out is not None else _empty_packed(O, K, N, M, W)
        outs.append((values, indices))
        descs.append(PackRankedDesc.packer.pack(W.data_ptr(), rank.data_ptr(), values.data_ptr(), indices.data_ptr(), O, K, N, M))
    _check(load_library().nm_pack_ranked_batched(_desc_array(PackRankedDesc, descs), len(descs), _stream_handle(stream)))
    return outs


def nm_pack(W, N: int, M: int, mask=None, stream=None):
    """(values bf16 [O, K*N/M], indices int32 [O, words]) of W at level N:M."""
    done = (_CALLS or _native()).pack(W, N, M, mask, stream)
    if done is not NotImplemented:
        return done
    torch = _torch()
    _need(W, torch.bfloat16, "W")
    O, K, ldw = _rows(W, "W")
    values, indices = _empty_packed(O, K, N, M, W)
    mask_ptr = None if mask is None else _mask_words(mask, O, K)
    _check(load_library().nm_pack(W.data_ptr(), O, K, ldw, N, M, mask_ptr, values.data_ptr(), indices.data_ptr(),
                                  _stream_handle(stream)))
    return values, indices


def nm_pack_batched(layers: Sequence[Tuple[object, int, int]], stream=None, out=None):
    """One launch for many (W, N, M); returns [(values, indices), ...]."""
    descs = []
    outs: List[Tuple[object, object]] = []
    for i, (W, N, M) in enumerate(layers):
        O, K = _contiguous_weight(W, "nm_pack_batched")
        values, indices = out[i] if out is not None else _empty_packed(O, K, N, M, W)
        outs.append((values, indices))
        descs.append(PackDesc.packer.pack(W.data_ptr(), values.data_ptr(), indices.data_ptr(), O, K, N, M))
    _check(load_library().nm_pack_batched(_desc_array(PackDesc, descs), len(descs), _stream_handle(stream)))
    return outs


def nm_pack_prepare_batched(layers: Sequence[Tuple[object, int, int, int]], stream=None, out=None, workspaces=None):
    """nm_pack + nm_spmm_prepare for many (W, N, M, T); returns ([(values, indices), ...], [workspace or None, ...])."""
    torch = _torch()
    descs = []
    outs: List[Tuple[object, object]] = []
    wss: List[object] = []
    for i, (W, N, M, T) in enumerate(layers):
        O, K = _contiguous_weight(W, "nm_pack_prepare_batched")
        values, indices = out[i] if out is not None else _empty_packed(O, K, N, M, W)
        if workspaces is not None:
            ws = workspaces[i]
        else:
            need = nm_spmm_workspace_bytes(O, K, N, M, T)
            ws = W.new_empty((need,), dtype=torch.uint8) if need else None
        outs.append((values, indices))
        wss.append(ws)
        ws_ptr, ws_bytes = _scratch(ws)
        descs.append(LayerDesc.packer.pack(W.data_ptr(), values.data_ptr(), indices.data_ptr(), O, K, N, M, T, ws_ptr or 0,
                                      ws_bytes))
    _check(load_library().nm_pack_prepare_batched(_desc_array(LayerDesc, descs), len(descs), _stream_handle(stream)))
    return outs, wss


def nm_unpack(values, indices, K: int, N: int, M: int, stream=None):
    done = (_CALLS or _native()).unpack(values, indices, K, N, M, stream)
    if done is not NotImplemented:
        return done
    torch = _torch()
    _need(values, torch.bfloat16, "values")
    _need(indices, torch.int32, "indices")
    O = values.shape[0]
    Wd = values.new_empty((O, K))
    _check(load_library().nm_unpack(values.data_ptr(), indices.data_ptr(), O, K, N, M, Wd.data_ptr(), K,
                                    _stream_handle(stream)))
    return Wd


def nm_mask_check(mask, K: int, N: int, M: int, stream=None) -> int:
    """Number of groups of `mask` that do not hold exactly N ones (synchronises to read it)."""
    torch = _torch()
    _need(mask, torch.int32, "mask")
    O = int(mask.shape[0])
    bad = torch.empty((1,), dtype=torch.int32, device=mask.device)
    _check(load_library().nm_mask_check(mask.data_ptr(), O, K, N, M, bad.data_ptr(), _stream_handle(stream)))
    return int(bad.item()) & 0xFFFFFFFF


def bf16_tensor(bits, device="cuda"):
    """numpy uint16 bf16 bit patterns -> torch.bfloat16 tensor on `device` (a copy of the bits)."""
    import numpy as np
    torch = _torch()
    return torch.from_numpy(np.ascontiguousarray(bits).view(np.int16)).to(device).view(torch.bfloat16)


def bf16_bits(t):
    """torch.bfloat16 tensor -> numpy uint16 bit patterns on the host."""
    import numpy as np
    torch = _torch()
    return t.contiguous().view(torch.int16).cpu().numpy().view(np.uint16)


_WORKSPACES = {}


def _workspace(nbytes: int, device, stream=None):
    """A cached scratch tensor per (device, stream), grown on demand (allocated by torch, not by the library).
    Calls on different streams may overlap, and concurrent calls need distinct workspaces, hence one per
    stream.  A tensor that is replaced may still be read by kernels on its stream: it is marked as in use on
    that stream so that the allocator does not hand its memory out before they finish."""
    torch = _torch()
    index = device.index if device.index is not None else torch.cuda.current_device()
    handle = _stream_handle(stream)
    key = (device.type, index, handle)
    ws = _WORKSPACES.get(key)
    if ws is None or ws.numel() < nbytes:
        if ws is not None:
            ws.record_stream(torch.cuda.ExternalStream(handle, device=index) if handle else torch.cuda.default_stream(index))
        ws = torch.empty((max(nbytes, 1 << 20),), dtype=torch.uint8, device=device)
        _WORKSPACES[key] = ws
    return ws


def _own_scratch(nbytes: int, stream=None):
    """A scratch tensor of one call, allocated on its stream: once dropped, its memory goes to later work of that stream
    only (under graph capture, of that graph)."""
    torch = _torch()
    if stream is None:
        return torch.empty((nbytes,), dtype=torch.uint8, device="cuda")
    if not isinstance(stream, torch.cuda.Stream):
        handle = _stream_handle(stream)
        stream = torch.cuda.ExternalStream(handle) if handle else torch.cuda.default_stream()
    with torch.cuda.stream(stream):
        return torch.empty((nbytes,), dtype=torch.uint8, device="cuda")


def nm_spmm_prepare(values, indices, K: int, N: int, M: int, T: int, workspace=None, stream=None):
    """Fill (and return) the workspace nm_linear_forward_prepared reads; None if the level needs none."""
    torch = _torch()
    _need(values, torch.bfloat16, "values")
    _need(indices, torch.int32, "indices")
    O = int(values.shape[0])
    need = nm_spmm_workspace_bytes(O, K, N, M, T)
    if workspace is None and need:
        workspace = torch.empty((need,), dtype=torch.uint8, device=values.device)
    ws_ptr, ws_bytes = _scratch(workspace)
    _check(load_library().nm_spmm_prepare(values.data_ptr(), indices.data_ptr(), O, K, N, M, T, ws_ptr, ws_bytes,
                                          _stream_handle(stream)))
    return workspace


def nm_linear_forward_prepared(values, indices, K: int, N: int, M: int, X, workspace, bias=None, out_dtype=None,
                               out=None, stream=None):
    """The product alone, from a workspace filled by nm_spmm_prepare."""
    done = (_CALLS or _native()).forward(values, indices, K, N, M, X, bias, out_dtype, out, workspace, stream, 1)
    if done is not NotImplemented:
        return done
    return nm_linear_forward(values, indices, K, N, M, X, bias, out_dtype, out, workspace, stream, _prepared=True)


def nm_linear_forward(values, indices, K: int, N: int, M: int, X, bias=None, out_dtype=None, out=None,
                      workspace=None, stream=None, _prepared=False, from_packed=False):
    """Y = X * W_s^T (+ bias) from the packed weight; Y is float32 (default) or bfloat16 [T, O].
    from_packed: hand the library no workspace, so that a product of up to 208 tokens runs straight from the packed
    format (the library reports a missing workspace for shapes that path does not take)."""
    done = (_CALLS or _native()).forward(values, indices, K, N, M, X, bias, out_dtype, out, workspace, stream,
                                         1 if _prepared else 2 if from_packed else 0)
    if done is not NotImplemented:
        return done
    torch = _torch()
    lib = load_library()
    O = _packed(values, indices, torch.bfloat16)
    _need(X, torch.bfloat16, "X")
    T, KX, ldx = _rows(X, "X")
    if KX != K:
        raise ValueError("X must be [T, K]")
    out, ldy, code = _out_matrix(out, out_dtype, T, O, X, "out")
    if workspace is None and not from_packed:
        need = lib.nm_spmm_workspace_bytes(O, K, N, M, T)
        if need and not _prepared:
            workspace = _workspace(need, X.device, stream)
        elif need and K % 64 == 0:  # (a ragged reduction can do without one)
            raise ValueError("a prepared call needs the workspace nm_spmm_prepare filled")
    ws_ptr, ws_bytes = _scratch(workspace)
    args = (values.data_ptr(), indices.data_ptr(), O, K, N, M, X.data_ptr(), T, ldx, _per_feature(bias, O, "bias"),
            out.data_ptr(), ldy, code, ws_ptr, ws_bytes)
    # partial sums of a prepared layer that is cut (a workspace of the operand part alone asks for the uncut product)
    need = lib.nm_prepared_scratch_bytes(O, K, N, M, T) if _prepared else 0
    if need and ws_bytes >= lib.nm_spmm_workspace_bytes(O, K, N, M, T):
        scratch = _own_scratch(need, stream)
        _check(lib.nm_linear_forward_prepared_scratch(*args, scratch.data_ptr(), need, _stream_handle(stream)))
    else:
        _check((lib.nm_linear_forward_prepared if _prepared else lib.nm_linear_forward)(*args, _stream_handle(stream)))
    return out


def nm_static_scratch_bytes() -> int:
    return int(load_library().nm_static_scratch_bytes())


def nm_linear_forward_static(values, indices, K: int, N: int, M: int, X, bias=None, out_dtype=None, out=None,
                             stream=None):
    """nm_linear_forward on the library's own fixed scratch: the call itself allocates nothing (pass `out`)."""
    done = (_CALLS or _native()).forward(values, indices, K, N, M, X, bias, out_dtype, out, None, stream, 3)
    if done is not NotImplemented:
        return done
    torch = _torch()
    O = _packed(values, indices, torch.bfloat16)
    _need(X, torch.bfloat16, "X")
    T, KX, ldx = _rows(X, "X")
    if KX != K:
        raise ValueError("X must be [T, K]")
    out, ldy, code = _out_matrix(out, out_dtype, T, O, X, "out")
    _check(load_library().nm_linear_forward_static(values.data_ptr(), indices.data_ptr(), O, K, N, M, X.data_ptr(), T,
                                                   ldx, _per_feature(bias, O, "bias"), out.data_ptr(), ldy, code,
                                                   _stream_handle(stream)))
    return out


def nm_probe_matrix_rate(kind: int, iters: int, sink=None, stream=None):
    """Launch the matrix-instruction loop (kind 0: 2:4 sparse bf16, 1: dense bf16); returns (sink, operations)."""
    torch = _torch()
    lib = load_library()
    if sink is None:
        sink = torch.empty((lib.nm_probe_sink_bytes(),), dtype=torch.uint8, device="cuda")
    ops = c_int64(0)
    _check(lib.nm_probe_matrix_rate(kind, iters, sink.data_ptr(), ctypes.byref(ops), _stream_handle(stream)))
    return sink, int(ops.value)


def nm_probe_copy(src, dst, stream=None):
    """dst = src with the library's plain streaming copy kernel (equal-sized contiguous device tensors)."""
    nbytes = src.numel() * src.element_size()
    if not (src.is_contiguous() and dst.is_contiguous()) or dst.numel() * dst.element_size() != nbytes:
        raise ValueError("src and dst must be contiguous and of equal size")
    _check(load_library().nm_probe_copy(src.data_ptr(), dst.data_ptr(), nbytes, _stream_handle(stream)))
    return dst


def _out_matrix(out, out_dtype, rows: int, cols: int, like, name: str, i32: bool = False):
    """(output tensor, its leading dimension, its type code); allocated on `like`'s device when not given."""
    torch = _torch()
    if out is not None:
        out_dtype = out.dtype
    if out_dtype == torch.bfloat16:
        code = NM_OUT_BF16
    elif out_dtype is None or out_dtype == torch.float32:
        code, out_dtype = NM_OUT_F32, torch.float32
    elif i32 and out_dtype == torch.int32:
        code = NM_OUT_I32
    else:
        raise ValueError("out dtype must be float32, bfloat16 or int32" if i32 else "out dtype must be float32 or bfloat16")
    if out is None:
        return like.new_empty((rows, cols), dtype=out_dtype), cols, code
    r, c, ld = _rows(out, name)
    if (r, c) != (rows, cols):
        raise ValueError(f"{name} must be [{rows}, {cols}]")
    return out, ld, code


def nm_backward_input_workspace_bytes(O: int, K: int, T: int) -> int:
    return int(load_library().nm_backward_input_workspace_bytes(O, K, T))


def nm_linear_backward_input(Ws, dY, out_dtype=None, out=None, workspace=None, stream=None):
    """dX = dY * Ws for the masked dense weight Ws [O, K] and dY [T, O]; float32 (default) or bfloat16 [T, K]."""
    done = (_CALLS or _native()).backward_input(Ws, dY, out_dtype, out, workspace, stream)
    if done is not NotImplemented:
        return done
    torch = _torch()
    _need(Ws, torch.bfloat16, "Ws")
    _need(dY, torch.bfloat16, "dY")
    O, K, ldw = _rows(Ws, "Ws")
    T, OY, ldy = _rows(dY, "dY")
    if OY != O:
        raise ValueError("dY must be [T, O]")
    out, ldx, code = _out_matrix(out, out_dtype, T, K, dY, "dX")
    lib = load_library()
    fn = lib.nm_linear_backward_input  # (which leaves a workspace alone that it can do without)
    if workspace is None:
        need = lib.nm_backward_input_workspace_bytes(O, K, T)
        if need:
            workspace = _workspace(need, dY.device, stream)
        else:  # a small layer: what it can use is the call's own, so that such calls may overlap and be captured as without it
            need = lib.nm_backward_input_scratch_bytes(O, K, T)
            if need:
                workspace = _own_scratch(need, stream)
                fn = lib.nm_linear_backward_input_scratch
    ws_ptr, ws_bytes = _scratch(workspace)
    _check(fn(Ws.data_ptr(), O, K, ldw, dY.data_ptr(), T, ldy, out.data_ptr(), ldx, code, ws_ptr, ws_bytes,
              _stream_handle(stream)))
    return out


def nm_backward_weight_workspace_bytes(O: int, K: int, T: int) -> int:
    return int(load_library().nm_backward_weight_workspace_bytes(O, K, T))


def nm_linear_backward_weight(dY, X, mask=None, out_dtype=None, out=None, workspace=None, stream=None):
    """dW = dY^T * X, with pruned positions zeroed when the step's mask words are given; [O, K]."""
    done = (_CALLS or _native()).backward_weight(dY, X, mask, out_dtype, out, workspace, stream)
    if done is not NotImplemented:
        return done
    torch = _torch()
    _need(dY, torch.bfloat16, "dY")
    _need(X, torch.bfloat16, "X")
    T, O, ldy = _rows(dY, "dY")
    TX, K, ldx = _rows(X, "X")
    if TX != T:
        raise ValueError("dY and X must have the same number of rows")
    mask_ptr = None if mask is None else _mask_words(mask, O, K)
    out, lddw, code = _out_matrix(out, out_dtype, O, K, dY, "dW")
    lib = load_library()
    fn = lib.nm_linear_backward_weight
    if workspace is None:
        need = lib.nm_backward_weight_scratch_bytes(O, K, T)
        if need:
            workspace = _workspace(need, dY.device, stream)
        fn = lib.nm_linear_backward_weight_scratch
    ws_ptr, ws_bytes = _scratch(workspace)
    _check(fn(dY.data_ptr(), T, O, ldy, X.data_ptr(), K, ldx, mask_ptr, out.data_ptr(), lddw, code, ws_ptr, ws_bytes,
              _stream_handle(stream)))
    return out


def forward_descs(layers):
    """The descriptor array of nm_linear_forward_prepared_batched for a list of
    (values, indices, K, N, M, X, workspace, bias or None, out); build it once when the buffers stay put."""
    torch = _torch()
    descs = (ForwardDesc * len(layers))()
    for n, (values, indices, K, N, M, X, workspace, bias, out) in enumerate(layers):
        _need(values, torch.bfloat16, "values")
        _need(indices, torch.int32, "indices")
        _need(X, torch.bfloat16, "X")
        if not values.is_contiguous() or not indices.is_contiguous():
            raise ValueError("packed tensors must be contiguous")
        O = int(values.shape[0])
        T, KX, ldx = _rows(X, "X")
        if KX != K:
            raise ValueError("X must be [T, K]")
        if out.dtype not in (torch.float32, torch.bfloat16):
            raise ValueError("out dtype must be float32 or bfloat16")
        TY, OY, ldy = _rows(out, "out")
        if (TY, OY) != (T, O):
            raise ValueError("out must be [T, O]")
        bias_ptr = None
        if bias is not None:
            _need(bias, torch.float32, "bias")
            if bias.numel() != O or not bias.is_contiguous():
                raise ValueError("bias must be contiguous [O]")
            bias_ptr = bias.data_ptr()
        descs[n] = ForwardDesc(values.data_ptr(), indices.data_ptr(), O, K, N, M, X.data_ptr(), T, ldx, bias_ptr,
                               out.data_ptr(), ldy, NM_OUT_F32 if out.dtype == torch.float32 else NM_OUT_BF16, 0,
                               workspace.data_ptr() if workspace is not None else None,
                               workspace.numel() * workspace.element_size() if workspace is not None else 0)
    return descs


def nm_linear_forward_prepared_batched(layers, stream=None):
    """The products of many prepared layers in as few launches as their shapes allow; `layers` is a list of
    (values, indices, K, N, M, X, workspace, bias or None, out) or an array made by forward_descs."""
    descs = layers if isinstance(layers, ctypes.Array) else forward_descs(layers)
    lib = load_library()
    need = lib.nm_prepared_batched_scratch_bytes(descs, len(descs))  # partial sums of the layers that are cut
    scratch = _own_scratch(need, stream) if need else None
    _check(lib.nm_linear_forward_prepared_batched_scratch(descs, len(descs), *_scratch(scratch), _stream_handle(stream)))


def nm_i8_workspace_bytes(O: int, K: int, N: int, M: int, T: int) -> int:
    return int(load_library().nm_i8_workspace_bytes(O, K, N, M, T))


def _i8_weight(Wq, mask):
    torch = _torch()
    _need(Wq, torch.int8, "Wq")
    _need(mask, torch.int32, "mask")
    O, K, ldw = _rows(Wq, "Wq")
    _mask_words(mask, O, K)
    return O, K, ldw


def nm_i8_prepare(Wq, mask, N: int, M: int, T: int, workspace=None, stream=None):
    """Compress the int8 weight into the operand order of the product at T tokens; returns the workspace (None if
    none is needed)."""
    torch = _torch()
    O, K, ldw = _i8_weight(Wq, mask)
    need = nm_i8_workspace_bytes(O, K, N, M, T)
    if workspace is None and need:
        workspace = torch.empty((need,), dtype=torch.uint8, device=Wq.device)
    ws_ptr, ws_bytes = _scratch(workspace)
    _check(load_library().nm_i8_prepare(Wq.data_ptr(), O, K, ldw, mask.data_ptr(), N, M, T, ws_ptr, ws_bytes,
                                        _stream_handle(stream)))
    return workspace


def nm_linear_forward_i8(Wq, mask, N: int, M: int, Xq, x_scale: float = 1.0, w_scale=None, bias=None, out_dtype=None,
                         out=None, workspace=None, stream=None, _prepared=False):
    """Y = x_scale * w_scale[o] * (Xq . (Wq (.) m)^T) + bias from int8 operands: float32 (default), bfloat16, or
    the exact int32 sums (out dtype int32)."""
    done = (_CALLS or _native()).forward_i8(Wq, mask, None, N, M, Xq, x_scale, w_scale, bias, out_dtype, out, workspace, stream,
                                            int(_prepared))
    if done is not NotImplemented:
        return done
    torch = _torch()
    O, K, ldw = _i8_weight(Wq, mask)
    _need(Xq, torch.int8, "Xq")
    T, KX, ldx = _rows(Xq, "Xq")
    if KX != K:
        raise ValueError("Xq must be [T, K]")
    out, ldy, code = _out_matrix(out, out_dtype, T, O, Xq, "out", i32=True)
    lib = load_library()
    workspace = _i8_scratch(lib, workspace, O, K, N, M, T, Xq, stream, _prepared, "nm_i8_prepare")
    ws_ptr, ws_bytes = _scratch(workspace)
    fn = lib.nm_linear_forward_i8_prepared if _prepared else lib.nm_linear_forward_i8
    _check(fn(Wq.data_ptr(), O, K, ldw, mask.data_ptr(), N, M, Xq.data_ptr(), T, ldx, float(x_scale),
              _per_feature(w_scale, O, "w_scale"), _per_feature(bias, O, "bias"), out.data_ptr(), ldy, code, ws_ptr,
              ws_bytes, _stream_handle(stream)))
    return out


def _i8_scratch(lib, workspace, O: int, K: int, N: int, M: int, T: int, Xq, stream, prepared: bool, filler: str):
    if workspace is None:
        need = lib.nm_i8_workspace_bytes(O, K, N, M, T)
        if need:
            if prepared:
                raise ValueError(f"a prepared call needs the workspace {filler} filled")
            workspace = _workspace(need, Xq.device, stream)
    return workspace


def nm_linear_forward_i8_prepared(Wq, mask, N: int, M: int, Xq, workspace, x_scale: float = 1.0, w_scale=None, bias=None,
                                  out_dtype=None, out=None, stream=None):
    """The product alone, from a workspace filled by nm_i8_prepare."""
    return nm_linear_forward_i8(Wq, mask, N, M, Xq, x_scale, w_scale, bias, out_dtype, out, workspace, stream,
                                _prepared=True)


def nm_pack_i8(Wq, mask, N: int, M: int, stream=None):
    """Compressed form of the int8 weight under `mask`: (values int8 [O, K*N/M], indices int32 words)."""
    torch = _torch()
    O, K, ldw = _i8_weight(Wq, mask)
    lib = load_library()
    values = torch.empty((O, K // M * N), dtype=torch.int8, device=Wq.device)
    indices = torch.empty((O, lib.nm_index_bytes(O, K, N, M) // (4 * O)), dtype=torch.int32, device=Wq.device)
    _check(lib.nm_pack_i8(Wq.data_ptr(), O, K, ldw, N, M, mask.data_ptr(), values.data_ptr(), indices.data_ptr(),
                          _stream_handle(stream)))
    return values, indices


def _i8_packed(values, indices):
    return _packed(values, indices, _torch().int8)


def nm_unpack_i8(values, indices, K: int, N: int, M: int, stream=None):
    torch = _torch()
    O = _i8_packed(values, indices)
    out = torch.empty((O, K), dtype=torch.int8, device=values.device)
    _check(load_library().nm_unpack_i8(values.data_ptr(), indices.data_ptr(), O, K, N, M, out.data_ptr(), K,
                                       _stream_handle(stream)))
    return out


def nm_i8_prepare_packed(values, indices, K: int, N: int, M: int, T: int, workspace=None, stream=None):
    """nm_i8_prepare from the compressed form: fills (and returns) the same workspace."""
    torch = _torch()
    O = _i8_packed(values, indices)
    need = nm_i8_workspace_bytes(O, K, N, M, T)
    if workspace is None and need:
        workspace = torch.empty((need,), dtype=torch.uint8, device=values.device)
    ws_ptr, ws_bytes = _scratch(workspace)
    _check(load_library().nm_i8_prepare_packed(values.data_ptr(), indices.data_ptr(), O, K, N, M, T, ws_ptr, ws_bytes,
                                               _stream_handle(stream)))
    return workspace


def nm_linear_forward_i8_packed(values, indices, K: int, N: int, M: int, Xq, x_scale: float = 1.0, w_scale=None, bias=None,
                                out_dtype=None, out=None, workspace=None, stream=None, _prepared=False):
    """nm_linear_forward_i8 with the weight in its compressed form."""
    done = (_CALLS or _native()).forward_i8(values, indices, K, N, M, Xq, x_scale, w_scale, bias, out_dtype, out, workspace, stream,
                                            int(_prepared))
    if done is not NotImplemented:
        return done
    torch = _torch()
    O = _i8_packed(values, indices)
    _need(Xq, torch.int8, "Xq")
    T, KX, ldx = _rows(Xq, "Xq")
    if KX != K:
        raise ValueError("Xq must be [T, K]")
    out, ldy, code = _out_matrix(out, out_dtype, T, O, Xq, "out", i32=True)
    lib = load_library()
    workspace = _i8_scratch(lib, workspace, O, K, N, M, T, Xq, stream, _prepared, "nm_i8_prepare_packed")
    ws_ptr, ws_bytes = _scratch(workspace)
    fn = lib.nm_linear_forward_i8_packed_prepared if _prepared else lib.nm_linear_forward_i8_packed
    _check(fn(values.data_ptr(), indices.data_ptr(), O, K, N, M, Xq.data_ptr(), T, ldx, float(x_scale),
              _per_feature(w_scale, O, "w_scale"), _per_feature(bias, O, "bias"), out.data_ptr(), ldy, code, ws_ptr,
              ws_bytes, _stream_handle(stream)))
    return out


def nm_linear_forward_i8_packed_prepared(values, indices, K: int, N: int, M: int, Xq, workspace, x_scale: float = 1.0,
                                         w_scale=None, bias=None, out_dtype=None, out=None, stream=None):
    return nm_linear_forward_i8_packed(values, indices, K, N, M, Xq, x_scale, w_scale, bias, out_dtype, out, workspace,
                                       stream, _prepared=True)


def nm_spmm(values, indices, K: int, N: int, M: int, X, out_dtype=None, out=None, workspace=None, stream=None,
            from_packed=False):
    return nm_linear_forward(values, indices, K, N, M, X, None, out_dtype, out, workspace, stream,
                             from_packed=from_packed)
