"""Masks from supplied scores and the dense weight back from the packed form, at the sizes where their kernels' lane
maps change: rows that end inside a mask word, row starts that are no whole 16-byte pieces, one row, every M, and the
contiguous form of the unpacking at index runs of 4 to 64 bits per 16 weights."""
import numpy as np
import pytest
import torch

import paper_2409_09708_amd as nm
from oracle import nm_oracle as orc
from paper_2409_09708_amd import workloads as wl

from gpu_util import dev_bf16, dev_words, host_bits, host_words

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("O,K,pitch,first,N,M", [
    (1, 4, 4, 0, 1, 4), (1, 16, 16, 0, 5, 16), (65, 36, 36, 0, 3, 4), (65, 36, 39, 0, 2, 4), (129, 64, 68, 1, 2, 8),
    (33, 40, 40, 0, 7, 8), (33, 48, 50, 2, 4, 16), (700, 96, 96, 0, 1, 16), (300, 768, 772, 4, 2, 4)])
def test_mask_from_scores_lane_maps(O, K, pitch, first, N, M):
    rng = np.random.default_rng(O * 1000 + K)
    s = rng.integers(-6, 7, size=(O * pitch + first + 16,)).astype(np.float32)
    s[rng.random(s.shape) < 0.04] = np.nan
    s[rng.random(s.shape) < 0.04] = -0.0
    s[rng.random(s.shape) < 0.04] = -np.inf
    dev = torch.from_numpy(s).cuda()
    view = torch.as_strided(dev, (O, K), (pitch, 1), first)
    ref = orc.nm_mask_from_scores(np.lib.stride_tricks.as_strided(s[first:], (O, K), (pitch * 4, 4)), N, M)
    assert np.array_equal(host_words(nm.nm_prune_scored(view, N, M)), orc.mask_to_words(ref))


# contiguous rows of whole words: one word, a last block that is partly filled, and both sides of four groups of 4 per lane
@pytest.mark.parametrize("O,K,N,M", [(1, 32, 2, 4), (3, 32, 1, 8), (5, 32, 3, 16), (33, 96, 3, 4), (65, 160, 5, 8), (67, 224, 9, 16),
                                     (2048, 4096, 2, 4), (2051, 4096, 1, 4), (1025, 8224, 3, 4)])
def test_mask_from_scores_contiguous(O, K, N, M):
    rng = np.random.default_rng(O * 1000 + K)
    s = rng.integers(-6, 7, size=(O, K)).astype(np.float32)
    for value in (np.nan, -0.0, -np.inf, np.inf):
        s[rng.random(s.shape) < 0.04] = value
    got = host_words(nm.nm_prune_scored(torch.from_numpy(s).cuda(), N, M))
    assert np.array_equal(got, orc.mask_to_words(orc.nm_mask_from_scores(s, N, M)))


@pytest.mark.parametrize("O,K,N,M", [(8, 64, 2, 4), (8, 128, 1, 16), (4, 64, 16, 16), (4, 128, 3, 8), (12, 256, 7, 8),
                                     (4, 128, 13, 16), (257, 64, 1, 4), (3, 1024, 1, 8), (5, 192, 8, 16)])
def test_unpack_contiguous(O, K, N, M):
    W = wl.tie_heavy_weights(np.random.default_rng(O + K + N), O, K)
    vals, idx = orc.nm_pack(W, orc.nm_mask(W, N, M), N, M)
    back = nm.nm_unpack(dev_bf16(vals), dev_words(idx), K, N, M)
    assert np.array_equal(host_bits(back), orc.nm_unpack(vals, idx, K, N, M))
