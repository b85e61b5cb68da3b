"""Weight gradient of a short reduction: one launch gives the bits of the two that it stands in for, masked and not."""
import ctypes

import pytest
import torch

import paper_2409_09708_amd as nm
from paper_2409_09708_amd.binding import load_library

from gpu_util import weight_grad_plan
from test_gpu_grad_short import one_launch

pytestmark = pytest.mark.gpu


def in_two_launches(dY, X, mask):
    (T, O), K = dY.shape, X.shape[1]
    dW = torch.full((O, K), 7.0, device="cuda")
    ws = torch.empty(nm.nm_backward_weight_workspace_bytes(O, K, T), dtype=torch.uint8, device="cuda")
    i64, ptr = ctypes.c_int64, ctypes.c_void_p
    call = load_library().nm_internal_weight_grad_two_launches
    assert 0 == call(ptr(dY.data_ptr()), i64(T), i64(O), i64(dY.stride(0)), ptr(X.data_ptr()), i64(K), i64(X.stride(0)),
                     ptr(mask.data_ptr() if mask is not None else None), ptr(dW.data_ptr()), i64(K), ptr(ws.data_ptr()),
                     ctypes.c_size_t(ws.nbytes), ptr(torch.cuda.current_stream().cuda_stream))
    return dW


# ranges of the reduction, and how many sums are added: that of the ranges, or of pairs of an even and an odd number of them; last
# steps that are whole, of one token and of others; ranges of unequal length
@pytest.mark.parametrize("T,K,O,ranges,sums", [
    (1, 8, 8, 1, 1), (33, 120, 136, 1, 1), (197, 768, 2304, 1, 1), (257, 520, 1032, 2, 2), (394, 1024, 4096, 3, 3),
    (500, 2048, 4096, 2, 1), (700, 2048, 2056, 3, 2), (788, 768, 3072, 6, 3), (801, 768, 3064, 6, 3), (900, 1664, 1272, 7, 4),
    (1000, 1152, 504, 8, 8), (1568, 768, 768, 12, 12), (1568, 768, 2304, 9, 5)])
def test_bits(T, K, O, ranges, sums):
    assert one_launch(T, K, O) and weight_grad_plan(T, K, O)[1:] == (ranges, sums)
    g = torch.Generator(device="cuda")
    g.manual_seed(9000 + T + O)
    X, dY = (torch.empty(T, n, dtype=torch.bfloat16, device="cuda").normal_(generator=g) for n in (K, O))
    X *= torch.logspace(-3, 3, T, device="cuda")[torch.randperm(T, generator=g, device="cuda")].bfloat16()[:, None]
    mask = nm.nm_prune(torch.empty(O, K, dtype=torch.bfloat16, device="cuda").normal_(generator=g), 2, 4)
    for m in (None, mask):
        two = in_two_launches(dY, X, m)
        assert torch.equal(nm.nm_linear_backward_weight(dY, X, mask=m).view(torch.int32), two.view(torch.int32))
    # (sums of ranges that are cut elsewhere have other bits)
    cut = [nm.nm_linear_backward_weight(dY[part], X[part], mask=mask) for part in (slice(0, T // 3), slice(T // 3, T))] if T > 2 else []
    assert not cut or not torch.equal(cut[0] + cut[1], two)
