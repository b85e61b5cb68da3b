"""Weight gradient from pairs of token ranges: an odd number of ranges over an odd number of tiles (one half of the last block has
no tile), a pair whose second range is the shorter one or ends in a ragged step, long ranges, and both sides of the shortest reduction
that is paired (16 steps of 32 tokens); operands and gradients in pitched rows, gradients in bfloat16."""
import pytest
import torch

import paper_2409_09708_amd as nm
from oracle import nm_oracle as orc

from gpu_util import check_output, dev_bf16, host_output, weight_grad_plan
from test_gpu_backward import draw

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,K,O,tiles,ranges", [(480, 384, 11008, 129, 3), (481, 384, 11008, 129, 3), (500, 2048, 4096, 256, 2),
                                                (545, 2040, 4088, 256, 2), (1100, 1152, 2304, 81, 6), (1057, 640, 3328, 65, 7)])
@pytest.mark.parametrize("masked", [False, True])
def test_weight_gradient_pairs(T, K, O, tiles, ranges, masked):
    assert nm.nm_backward_weight_workspace_bytes(O, K, T) == tiles * ranges * 128 * 256 * 4
    assert weight_grad_plan(T, K, O) == (tiles, ranges, ranges if T == 480 else (ranges + 1) // 2)
    X, W, dY, mask = draw(7100 + T + K, T, K, O, 2, 4)
    _, dWref, _, BW = orc.nm_linear_backward(dY, X, W, mask, masked_grad=masked)
    words = torch.from_numpy(orc.mask_to_words(mask).view("int32")).cuda() if masked else None
    dW = nm.nm_linear_backward_weight(dev_bf16(dY), dev_bf16(X), mask=words)
    check_output(host_output(dW), dWref, BW, T, True, (T, K, O))
    assert torch.equal(dW, nm.nm_linear_backward_weight(dev_bf16(dY), dev_bf16(X), mask=words))


# pitched rows, and a pair of 57 and 56 steps that ends inside a step
@pytest.mark.parametrize("T,K,O,tiles,ranges", [(1057, 640, 3328, 65, 7), (545, 2040, 4088, 256, 2), (3590, 2040, 4088, 256, 2)])
def test_rows_of_pairs_lie_anywhere(T, K, O, tiles, ranges):
    assert weight_grad_plan(T, K, O) == (tiles, ranges, (ranges + 1) // 2)
    X, W, dY, mask = draw(7200 + T + K, T, K, O, 2, 4)
    _, dWref, _, BW = orc.nm_linear_backward(dY, X, W, mask, masked_grad=True)
    words = torch.from_numpy(orc.mask_to_words(mask).view("int32")).cuda()
    Xp = torch.full((T, K + 8), float("nan"), dtype=torch.bfloat16, device="cuda")  # nothing beside the rows is read
    dYp = torch.full((T, O + 24), float("nan"), dtype=torch.bfloat16, device="cuda")
    Xp[:, :K], dYp[:, 16:16 + O] = dev_bf16(X), dev_bf16(dY)
    dW = nm.nm_linear_backward_weight(dev_bf16(dY), dev_bf16(X), mask=words)
    check_output(host_output(dW), dWref, BW, T, True, (T, K, O))
    for dtype in (torch.float32, torch.bfloat16):
        for pad in (0, 8, 1):
            out = torch.full((O, K + 2 * pad), 7.0, dtype=dtype, device="cuda")
            nm.nm_linear_backward_weight(dYp[:, 16:16 + O], Xp[:, :K], mask=words, out=out[:, pad:pad + K])
            assert torch.equal(out[:, pad:pad + K], dW.to(dtype)), (dtype, pad)
            assert bool((out[:, :pad] == 7).all()) and bool((out[:, pad + K:] == 7).all())
