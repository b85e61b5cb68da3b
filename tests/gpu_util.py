"""Helpers shared by the tests: host bit patterns <-> device tensors, acceptance checks, the kernel a shape runs on."""
import ctypes

import numpy as np
import torch

from oracle import nm_oracle as orc


from paper_2409_09708_amd.binding import bf16_bits as host_bits
from paper_2409_09708_amd.binding import bf16_tensor as dev_bf16
from paper_2409_09708_amd.binding import load_library


def host_words(t: torch.Tensor) -> np.ndarray:
    return t.contiguous().cpu().numpy().view(np.uint32)


def dev_words(w: np.ndarray) -> torch.Tensor:
    return torch.from_numpy(np.ascontiguousarray(w).view(np.int32)).cuda()


def host_output(y: torch.Tensor) -> np.ndarray:
    """Y as float64, whatever its storage type."""
    if y.dtype == torch.bfloat16:
        return orc.bf16_bits_to_f64(host_bits(y))
    return y.cpu().numpy().astype(np.float64)


def check_output(Y: np.ndarray, Yref: np.ndarray, B: np.ndarray, terms: int, fp32_out: bool, what=""):
    """Acceptance: every element within 1e-2 * sum_k |x_k w_k|, relative Frobenius error <= 5e-3.
    For fp32 outputs also the rounding bound of an fp32 sum of `terms` exact products in any order,
    (terms + 2) * 2^-24 * B, which is far tighter and catches a single dropped or doubled product."""
    err = np.abs(Y - Yref)
    assert np.all(np.isfinite(Y)), what
    assert np.all(err <= 1e-2 * B + 1e-30), (what, float((err / (B + 1e-30)).max()))
    fro = np.linalg.norm(Y - Yref) / max(np.linalg.norm(Yref), 1e-30)
    assert fro <= 5e-3, (what, fro)
    if fp32_out:
        tight = (terms + 2) * 2.0 ** -24 * B + 1e-30
        assert np.all(err <= tight), (what, float((err / tight).max()))
    return float((err / (B + 1e-30)).max()), float(fro)


PRODUCT_KERNELS = ("general", "tiled", "persistent", "ragged", "direct", "fewtok")


def product_route(call: str, T: int, K: int, O: int, N: int, M: int):
    """(kernel, (out-features, tokens, LDS stages) of its tile) of a product of aligned operands, as the library's own
    dispatch has it; call: "plain", "prepared" or "packed" (no workspace).  No tile but for "tiled" and "persistent"."""
    i64, tile = ctypes.c_int64, (ctypes.c_int32 * 3)()
    call_code = ("plain", "prepared", "packed").index(call)
    r = load_library().nm_internal_product_route(call_code, i64(O), i64(K), N, M, i64(T), tile)
    return (PRODUCT_KERNELS[r] if r >= 0 else "refused"), tuple(tile)


def int8_route(T: int, K: int, O: int, N: int, M: int):
    """(kernel, tokens per tile) of an int8 product of aligned operands: the persistent kernel's operand copy is padded to
    whole 256-row tiles, which tells it from the tiled one's (O off the tile edge)."""
    i64, sparse_form = ctypes.c_int64, N <= 2 and N < M
    lib, stages = load_library(), ctypes.c_int32()
    rows = (O + 255) // 256 * 256
    assert rows != O
    if lib.nm_i8_workspace_bytes(O, K, N, M, T) != (rows * K // 2 + rows * K // 8 if sparse_form else rows * K):
        return "tiled", 0
    return "persistent", lib.nm_internal_stream_tile(1, int(sparse_form), i64(O), i64(T), i64(K // (128 if sparse_form else 64)),
                                                     ctypes.byref(stages))


def weight_grad_plan(T: int, K: int, O: int):
    """(tiles, ranges of the token reduction, partial tiles that the sum over them reads) of a weight gradient; the ranges are
    taken in pairs where there are more of them than partial tiles."""
    i64, ranges, planes = ctypes.c_int64, ctypes.c_int32(), ctypes.c_int32()
    tiles = load_library().nm_internal_weight_grad_plan(i64(O), i64(K), i64(T), ctypes.byref(ranges), ctypes.byref(planes))
    return tiles, ranges.value, planes.value
