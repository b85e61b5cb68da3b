"""Pruning that writes the weight: the chunks per lane go by the size of the matrix.  Both sides of each border against the same
rows pruned a thousand at a time, with a matrix of its own and in place."""
import pytest
import torch

import paper_2409_09708_amd as nm

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,M", [(2, 4), (1, 8), (4, 16), (3, 8)])
@pytest.mark.parametrize("O", [2048, 2049, 16384, 16385])  # x 3072: 1536 blocks of 256 chunks of 16, 12288, and 192 chunks more
def test_prune_large(N, M, O):
    K = 3072
    g = torch.Generator(device="cuda")
    g.manual_seed(O)
    W = torch.empty(O, K, dtype=torch.bfloat16, device="cuda").normal_(0, 0.02, generator=g)
    out = torch.empty_like(W)
    mask = nm.nm_prune(W, N, M, W_masked=out)
    for r in range(0, O, 1000):
        rows, part = slice(r, min(r + 1000, O)), torch.empty_like(W[r:r + 1000])
        assert torch.equal(nm.nm_prune(W[rows], N, M, W_masked=part), mask[rows])
        assert torch.equal(part.view(torch.int16), out[rows].view(torch.int16))
    assert torch.equal(nm.nm_prune(W, N, M, W_masked=W), mask) and torch.equal(W.view(torch.int16), out.view(torch.int16))
