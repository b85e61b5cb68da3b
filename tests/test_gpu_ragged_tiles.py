"""The tiles of rows of X at any alignment: an output does not depend on the tile that computes it, over reductions of two to a few
steps in the large tiles, and of whole rounds of the stages loaded ahead and more in the small ones that load four of them."""
import ctypes

import pytest
import torch

import paper_2409_09708_amd as nm
from gpu_util import check_output, dev_bf16, host_output
from paper_2409_09708_amd.binding import load_library
from test_gpu_ragged import layer


def tile(T, K, O, N, dtype):
    i64 = ctypes.c_int64
    bf16 = dtype == torch.bfloat16
    return load_library().nm_internal_ragged_tile(int(N <= 2), i64(O), i64(K), i64(T), int(bf16), int(O % (8 if bf16 else 4) == 0))


# (one list of blocks per unit more for the small tiles; 208 to 336 and past 512 large ones, where those are the second round that is
# nearly empty; rows of the output in whole pieces)
@pytest.mark.parametrize("T,K,O,N,dtype,want", [
    (7410, 84, 1317, 2, torch.bfloat16, 64), (6053, 76, 1774, 2, torch.bfloat16, 64), (10403, 100, 279, 4, torch.float32, 64),
    (33413, 140, 1896, 2, torch.bfloat16, 128), (6061, 116, 6096, 2, torch.bfloat16, 128),
    (9545, 548, 354, 1, torch.float32, 64), (35674, 84, 2697, 2, torch.float32, 128), (15713, 444, 1188, 3, torch.float32, 128),
    (9460, 1764, 324, 1, torch.float32, 128), (926, 2740, 96, 1, torch.bfloat16, 64)])
def test_choice(T, K, O, N, dtype, want):
    assert tile(T, K, O, N, dtype) == want


@pytest.mark.gpu
@pytest.mark.parametrize("N,K", [(1, 68), (2, 124), (3, 132), (4, 188), (1, 196), (3, 260), (2, 316), (4, 324)])
def test_large_tiles_of_short_reductions(N, K):
    T, O = 31001, 1020
    assert tile(T, K, O, N, torch.float32) == 128
    g = torch.Generator(device="cuda")
    g.manual_seed(K)
    W, X = (torch.empty(n, K, dtype=torch.bfloat16, device="cuda").normal_(generator=g) for n in (O, T))
    bias = torch.empty(O, device="cuda").normal_(generator=g)
    v, i = nm.nm_pack(W, N, 4)
    y = nm.nm_linear_forward(v, i, K, N, 4, X, bias=bias)
    for first in (0, 127, 15000, T - 130):
        assert tile(130, K, O, N, torch.float32) == 64
        assert torch.equal(y[first:first + 130], nm.nm_linear_forward(v, i, K, N, 4, X[first:first + 130], bias=bias))


@pytest.mark.gpu
@pytest.mark.parametrize("N", [3, 4])
@pytest.mark.parametrize("steps", [20, 21, 22, 23, 24, 28, 29])
def test_long_reductions_of_dense_levels(N, steps):
    T, O = 70, 66
    for K in (64 * steps - 4, 64 * steps - 60):
        X, v, i, bias, Yref, B = layer(12500 + K + N, T, K, O, N, 4)
        y = nm.nm_linear_forward(v, i, K, N, 4, dev_bf16(X), bias=bias)
        check_output(host_output(y), Yref, B, K // 4 * N + 1, True, (T, K, O, N))
