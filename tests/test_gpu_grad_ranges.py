"""Weight gradient: the sum over the partial tiles reads them two or six at a time by the number of tiles; both sides of that border
(10 tiles), with counts of partial tiles that are one more than whole sixes and others, of single ranges and of pairs."""
import pytest
import torch

import paper_2409_09708_amd as nm
from oracle import nm_oracle as orc

from gpu_util import check_output, dev_bf16, host_output, weight_grad_plan
from test_gpu_backward import draw

pytestmark = pytest.mark.gpu


# partial tiles: as many as ranges, or one per pair
@pytest.mark.parametrize("T,K,O,tiles,ranges,partial", [
    (900, 1024, 512, 16, 7, 7), (3152, 1024, 512, 16, 24, 24), (1700, 128, 256, 1, 13, 13), (900, 1152, 512, 18, 7, 7),
    (1312, 1024, 1280, 40, 10, 10), (1100, 2048, 1000, 64, 8, 4), (900, 1664, 1272, 65, 7, 4), (900, 768, 3072, 72, 7, 4),
    (1500, 1664, 1792, 91, 11, 6),
    # six at a time: nothing but sixes behind the first, up to five left over, pairs of an odd and an even number of ranges
    (870, 640, 504, 10, 7, 7), (1000, 640, 512, 10, 8, 8), (1500, 376, 760, 9, 11, 11), (6304, 640, 512, 10, 47, 24),
    (6304, 384, 768, 9, 49, 25), (3152, 128, 256, 1, 24, 24),
    # just past the border, and the same counts where the wavefronts are many
    (1000, 768, 512, 12, 8, 8), (1700, 768, 504, 12, 13, 13), (6304, 768, 512, 12, 39, 20), (1920, 640, 3328, 65, 15, 8),
    (1700, 640, 3840, 75, 13, 7)])
def test_weight_gradient_ranges(T, K, O, tiles, ranges, partial):
    assert weight_grad_plan(T, K, O) == (tiles, ranges, partial)
    assert nm.nm_backward_weight_workspace_bytes(O, K, T) == tiles * ranges * 128 * 256 * 4
    X, W, dY, mask = draw(6400 + tiles + ranges, T, K, O, 2, 4)
    _, dWref, _, BW = orc.nm_linear_backward(dY, X, W, mask, masked_grad=False)
    dW = nm.nm_linear_backward_weight(dev_bf16(dY), dev_bf16(X))
    check_output(host_output(dW), dWref, BW, T, True, (T, K, O))
    assert torch.equal(dW, nm.nm_linear_backward_weight(dev_bf16(dY), dev_bf16(X)))
