"""Weights whose kernels need 2^32 lanes and more, the largest number one dimension of a launch can hold: masks from
scores (a lane per group) and the operand-order copy (a lane per 16 weights)."""
import pytest
import torch

import paper_2409_09708_amd as nm

pytestmark = pytest.mark.gpu


def need_free(nbytes):
    torch.cuda.empty_cache()
    if torch.cuda.mem_get_info()[0] < nbytes:
        pytest.skip("not enough free device memory")


def test_mask_from_scores():
    O, K = (1 << 16) + 3, 1 << 18  # 2^32 + 196608 groups of 4
    need_free(O * K * 4 + O * K // 8 + (8 << 30))
    score = torch.zeros((O, K), dtype=torch.float32, device="cuda")
    last = torch.randn((K,), generator=torch.Generator().manual_seed(3)).cuda()
    score[O - 1] = last
    mask = nm.nm_prune_scored(score, 1, 4)
    assert bool((mask[:O - 1] == 0x11111111).all())  # equal scores: the first of every group
    assert torch.equal(mask[O - 1:], nm.nm_prune_scored(last[None, :], 1, 4))
    del score, mask
    torch.cuda.empty_cache()


def test_operand_order_copy():
    O, K, N, M, T = (1 << 18) + 256, 1 << 18, 1, 16, 3  # 2^32 + 2^22 chunks of 16 weights
    need_free(O * K + O * K // 8 + O * K // 16 * 5 // 2 + (8 << 30))
    gen = torch.Generator(device="cuda").manual_seed(5)
    values = torch.empty((O, K // M), dtype=torch.bfloat16, device="cuda").normal_(0, 0.02, generator=gen)
    indices = torch.randint(-2 ** 31, 2 ** 31 - 1, (O, K // M // 8), dtype=torch.int32, device="cuda", generator=gen)
    X = torch.empty((T, K), dtype=torch.bfloat16, device="cuda").normal_(0, 1, generator=gen)
    ws = nm.nm_spmm_prepare(values, indices, K, N, M, T)
    y = nm.nm_linear_forward_prepared(values, indices, K, N, M, X, ws)
    rows = torch.tensor([0, 1, O // 2, O - 257, O - 256, O - 2, O - 1], device="cuda")
    W = nm.nm_unpack(values[rows].contiguous(), indices[rows].contiguous(), K, N, M).double()
    ref, B = X.double() @ W.t(), X.double().abs() @ W.abs().t()
    assert bool(((y[:, rows].double() - ref).abs() <= (K // M + 2) * 2.0 ** -24 * B).all())
    del ws, values, indices, y
    torch.cuda.empty_cache()
