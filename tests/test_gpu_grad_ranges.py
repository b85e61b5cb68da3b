"""Weight gradient: the sum over the partial tiles reads them one by one or six at a time by the number of tiles; both sides of each
border, with counts of ranges that are one more than whole sixes and others."""
import pytest
import torch

import paper_2409_09708_amd as nm
from oracle import nm_oracle as orc

from gpu_util import check_output, dev_bf16, host_output
from test_gpu_backward import draw

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,K,O,tiles,ranges", [(900, 1024, 512, 16, 7), (3152, 1024, 512, 16, 24), (1700, 128, 256, 1, 13),
                                                (900, 1152, 512, 18, 7), (1312, 1024, 1280, 40, 10), (1100, 2048, 1000, 64, 8),
                                                (900, 1664, 1272, 65, 7), (900, 768, 3072, 72, 7),
                                                (1500, 1664, 1792, 91, 11)])
def test_weight_gradient_ranges(T, K, O, tiles, ranges):
    assert nm.nm_backward_weight_workspace_bytes(O, K, T) == tiles * ranges * 128 * 256 * 4
    X, W, dY, mask = draw(6400 + tiles + ranges, T, K, O, 2, 4)
    _, dWref, _, BW = orc.nm_linear_backward(dY, X, W, mask, masked_grad=False)
    dW = nm.nm_linear_backward_weight(dev_bf16(dY), dev_bf16(X))
    check_output(host_output(dW), dWref, BW, T, True, (T, K, O))
    assert torch.equal(dW, nm.nm_linear_backward_weight(dev_bf16(dY), dev_bf16(X)))
