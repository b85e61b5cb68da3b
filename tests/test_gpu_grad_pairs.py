"""Weight gradient from pairs of token ranges: an odd number of ranges over an odd number of tiles (one half of the last block has
no tile), a pair whose second range is the shorter one or ends in a ragged step, and both sides of the shortest reduction that
is paired (16 steps of 32 tokens)."""
import pytest
import torch

import paper_2409_09708_amd as nm
from oracle import nm_oracle as orc

from gpu_util import check_output, dev_bf16, host_output
from test_gpu_backward import draw

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,K,O,tiles,ranges", [(480, 384, 11008, 129, 3), (481, 384, 11008, 129, 3), (500, 2048, 4096, 256, 2),
                                                (545, 2040, 4088, 256, 2), (1100, 1152, 2304, 81, 6), (1057, 640, 3328, 65, 7)])
@pytest.mark.parametrize("masked", [False, True])
def test_weight_gradient_pairs(T, K, O, tiles, ranges, masked):
    assert nm.nm_backward_weight_workspace_bytes(O, K, T) == tiles * ranges * 128 * 256 * 4
    X, W, dY, mask = draw(7100 + T + K, T, K, O, 2, 4)
    _, dWref, _, BW = orc.nm_linear_backward(dY, X, W, mask, masked_grad=masked)
    words = torch.from_numpy(orc.mask_to_words(mask).view("int32")).cuda() if masked else None
    dW = nm.nm_linear_backward_weight(dev_bf16(dY), dev_bf16(X), mask=words)
    check_output(host_output(dW), dWref, BW, T, True, (T, K, O))
    assert torch.equal(dW, nm.nm_linear_backward_weight(dev_bf16(dY), dev_bf16(X), mask=words))
