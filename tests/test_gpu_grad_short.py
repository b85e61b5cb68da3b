"""Weight gradient of a short reduction, one launch: reductions of less than a step, whole steps and one token more, fewer steps
than stages, single ranges and pairs of an even and an odd number of them; outputs of less than a tile, whole tiles and 8 features
more, more tiles than compute units; pitched rows, gradients in bfloat16 and at addresses without alignment.  And the last
reduction of one launch, the first of two, and pairs of an odd number of ranges over an odd number of tiles in two."""
import ctypes

import pytest
import torch

import paper_2409_09708_amd as nm
from oracle import nm_oracle as orc
from paper_2409_09708_amd.binding import load_library

from gpu_util import check_output, dev_bf16, host_output, weight_grad_plan
from test_gpu_backward import draw

pytestmark = pytest.mark.gpu


def one_launch(T, K, O):
    i64 = ctypes.c_int64
    return bool(load_library().nm_internal_weight_grad_one_launch(i64(O), i64(K), i64(T)))


# ranges of the reduction, and their number or that of their pairs
@pytest.mark.parametrize("T,K,O,ranges,sums", [
    (1, 8, 8, 1, 1), (31, 136, 64, 1, 1), (32, 128, 128, 1, 1), (33, 120, 136, 1, 1), (96, 256, 264, 1, 1), (97, 264, 256, 1, 1),
    (128, 768, 768, 1, 1), (129, 768, 760, 1, 1), (197, 768, 2304, 1, 1), (257, 520, 1032, 2, 2), (394, 1024, 4096, 3, 3),
    (700, 2048, 2056, 3, 2), (788, 768, 3072, 6, 3), (801, 768, 3064, 6, 3), (900, 1664, 1272, 7, 4), (1000, 1152, 504, 8, 8),
    (60, 4224, 4104, 1, 1)])
@pytest.mark.parametrize("masked", [False, True])
def test_weight_gradient_in_one_launch(T, K, O, ranges, sums, masked):
    assert one_launch(T, K, O) and weight_grad_plan(T, K, O)[1:] == (ranges, sums)
    X, W, dY, mask = draw(8100 + T + K, T, K, O, 2, 4)
    _, dWref, _, BW = orc.nm_linear_backward(dY, X, W, mask, masked_grad=masked)
    words = torch.from_numpy(orc.mask_to_words(mask).view("int32")).cuda() if masked else None
    Xp = torch.full((T + 1, K + 8), float("nan"), dtype=torch.bfloat16, device="cuda")  # nothing beside the rows is read
    dYp = torch.full((T + 1, O + 24), float("nan"), dtype=torch.bfloat16, device="cuda")
    Xp[:T, :K], dYp[:T, 16:16 + O] = dev_bf16(X), dev_bf16(dY)
    dW = nm.nm_linear_backward_weight(dYp[:T, 16:16 + O], Xp[:T, :K], mask=words)
    check_output(host_output(dW), dWref, BW, T, True, (T, K, O))
    for dtype in (torch.float32, torch.bfloat16):
        for pad in (0, 8, 1):
            out = torch.full((O, K + 2 * pad), 7.0, dtype=dtype, device="cuda")
            nm.nm_linear_backward_weight(dYp[:T, 16:16 + O], Xp[:T, :K], mask=words, out=out[:, pad:pad + K])
            assert torch.equal(out[:, pad:pad + K], dW.to(dtype)), (dtype, pad)
            assert bool((out[:, :pad] == 7).all()) and bool((out[:, pad + K:] == 7).all())


@pytest.mark.parametrize("K,O,T", [(256, 256, 352), (768, 768, 1568), (768, 2304, 1920), (2944, 768, 2112)])
def test_both_sides_of_one_launch(K, O, T):
    assert K < 2944 or weight_grad_plan(T + 1, K, O) == (69, 7, 4)
    for T in (T, T + 1):
        assert one_launch(T, K, O) == (T % 32 == 0)
        X, W, dY, mask = draw(8200 + T + K, T, K, O, 2, 4)
        _, dWref, _, BW = orc.nm_linear_backward(dY, X, W, mask, masked_grad=True)
        words = torch.from_numpy(orc.mask_to_words(mask).view("int32")).cuda()
        dW = nm.nm_linear_backward_weight(dev_bf16(dY), dev_bf16(X), mask=words)
        check_output(host_output(dW), dWref, BW, T, True, (T, K, O))
