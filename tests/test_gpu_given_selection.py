"""Packing under a given selection (a mask, stored ranks) at the levels whose kept weights are compacted by networks: zeros
in the last place of a group (whose key is that of a pruned weight), chunks in which one group has too many or too few kept
weights (they take the other coder), runs that end inside a block of 256 chunks."""
import numpy as np
import pytest
import torch

import paper_2409_09708_amd as nm
from oracle import nm_oracle as orc
from paper_2409_09708_amd import workloads as wl

from gpu_util import dev_bf16, dev_words, host_bits, host_words

pytestmark = pytest.mark.gpu

LEVELS = [(1, 4), (2, 4), (1, 8), (2, 8), (4, 8), (1, 16), (2, 16), (4, 16)]


def selection(rng, O, K, N, M, uneven):
    """A random mask with N of M (uneven: some groups have another number), and the weights kept under it by the rule for
    such groups: the N lowest set positions, missing ones completed by the lowest unset positions as +0."""
    order = rng.random((O, K // M, M)).argsort(axis=2)
    keep = order < N
    if uneven:
        bad = rng.random((O, K // M)) < 0.02
        keep[bad] = rng.random((int(bad.sum()), M)) < 0.5
    kept, filled = np.zeros_like(keep), np.zeros_like(keep)
    for o, g in np.ndindex(O, K // M):
        on, off = np.flatnonzero(keep[o, g])[:N], np.flatnonzero(~keep[o, g])
        kept[o, g, on] = True
        filled[o, g, off[:N - len(on)]] = True
    flat = lambda a: a.reshape(O, K)
    return flat(keep), flat(kept | filled), flat(filled)


@pytest.mark.parametrize("N,M", LEVELS)
@pytest.mark.parametrize("O,uneven", [(1, False), (5, True), (87, True)])  # 6, 30 and 522 chunks
def test_pack_under_a_mask(N, M, O, uneven):
    K = 96 if (96 // M * N * {4: 2, 8: 3, 16: 4}[M]) % 32 == 0 else 256
    rng = np.random.default_rng(100 * N + M + O)
    W = wl.tie_heavy_weights(rng, O, K)
    W[:, M - 1::M] = np.where(rng.random(W[:, M - 1::M].shape) < 0.5, 0, W[:, M - 1::M])
    mask, legal, filled = selection(rng, O, K, N, M, uneven)
    values, indices = nm.nm_pack(dev_bf16(W), N, M, mask=dev_words(orc.mask_to_words(mask)))
    vals, idx = orc.nm_pack(np.where(filled, 0, W).astype(np.uint16), legal, N, M)
    assert np.array_equal(host_bits(values), vals) and np.array_equal(host_words(indices), idx)


@pytest.mark.parametrize("N,M", LEVELS)
def test_pack_ranked_batched_and_ranks_that_are_no_permutation(N, M):
    K = 256
    rng = np.random.default_rng(10 * N + M)
    Ws = [wl.tie_heavy_weights(rng, O, K) for O in (1, 32, 67)]  # 16, 512 and 1072 chunks
    devs = [dev_bf16(W) for W in Ws]
    ranks = [nm.nm_rank(d, M) for d in devs]
    ranks[2][5:9] = torch.from_numpy(rng.integers(0, 256, size=(4, K // 2), dtype=np.uint8)).cuda()
    for W, rank, (values, indices) in zip(Ws, ranks, nm.nm_pack_ranked_batched([(d, r, N, M) for d, r in zip(devs, ranks)])):
        nibbles = rank.cpu().numpy()
        keep = np.stack([nibbles & 15, nibbles >> 4], axis=2).reshape(W.shape) < N
        mask = dev_words(orc.mask_to_words(keep))
        v, i = nm.nm_pack(dev_bf16(W), N, M, mask=mask)
        assert torch.equal(values.view(torch.int16), v.view(torch.int16)) and torch.equal(indices, i)
        rows = keep.reshape(len(W), -1, M).sum(axis=2).min(axis=1) == N  # (those the checker takes as they are)
        rows &= keep.reshape(len(W), -1, M).sum(axis=2).max(axis=1) == N
        vals, idx = orc.nm_pack(W[rows], keep[rows], N, M)
        assert np.array_equal(host_bits(values)[rows], vals) and np.array_equal(host_words(indices)[rows], idx)
