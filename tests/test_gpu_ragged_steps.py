"""GPU parity of products of rows of X at any alignment over the number of their steps: none past the stages that are loaded ahead, as
many, one more, and whole rounds of them and one more, in the small and in the large tiles and on both sides of their border; a last
piece of four elements, X at the end of its memory and with NaN between its rows."""
import pytest
import torch

import paper_2409_09708_amd as nm
from gpu_util import check_output, dev_bf16, host_output
from test_gpu_ragged import layer

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,O", [(67, 70), (1700, 1900), (3300, 1020)])  # the last two take tiles of 128 x 128 from 6 (1:4) and 9 (3:4) steps on
@pytest.mark.parametrize("N,M", [(1, 4), (3, 4)])
@pytest.mark.parametrize("steps", [2, 3, 4, 5, 6, 8, 9, 10, 12, 13])
def test_steps_of_rows_at_any_alignment(T, O, N, M, steps):
    for K in (64 * steps - 60, 64 * steps - 4):
        X, v, i, bias, Yref, B = layer(12100 + T + K + N, T, K, O, N, M)
        flat = torch.full((T * (K + 2),), float("nan"), dtype=torch.bfloat16, device="cuda")
        Xd = flat.as_strided((T, K), (K + 2, 1), 2)  # the last row ends with the memory
        Xd.copy_(dev_bf16(X))
        y = nm.nm_linear_forward(v, i, K, N, M, Xd, bias=bias)
        check_output(host_output(y), Yref, B, K // M * N + 1, True, (T, K, O, N, M))
        assert torch.equal(y, nm.nm_linear_forward(v, i, K, N, M, dev_bf16(X), bias=bias))
        Xo = torch.full((T * K + 1,), float("nan"), dtype=torch.bfloat16, device="cuda")[1:].view(T, K)
        Xo.copy_(dev_bf16(X))
        assert torch.equal(y, nm.nm_linear_forward(v, i, K, N, M, Xo, bias=bias))


@pytest.mark.parametrize("T,O", [(1600, 1900), (1700, 1900), (2600, 1900), (2700, 2000)])  # 195, 210, 315 and 352 tiles of 128 x 128, taken at 210 and 352
@pytest.mark.parametrize("K", [508, 516])
def test_both_sides_of_the_large_tiles(T, O, K):
    X, v, i, bias, Yref, B = layer(12300 + T + K, T, K, O, 2, 4)
    y = nm.nm_linear_forward(v, i, K, 2, 4, dev_bf16(X), bias=bias)
    check_output(host_output(y), Yref, B, K // 2 + 1, True, (T, K, O))
