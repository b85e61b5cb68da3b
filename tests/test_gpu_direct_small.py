"""Up to 16 or 32 tokens the one-launch kernel takes four spans of 256 reduction positions at a time: reductions that end at, before
and behind four spans, tokens at the edges of the tile, both summation orders; the bytes of a prepared and of a batched call."""
import numpy as np
import pytest
import torch

import paper_2409_09708_amd as nm
from oracle import nm_oracle as orc
from paper_2409_09708_amd import workloads as wl
from gpu_util import check_output, dev_bf16, host_output, product_route

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,M", [(1, 4), (3, 4), (1, 8), (2, 8), (3, 8), (4, 8), (1, 16), (2, 16), (4, 16)])
@pytest.mark.parametrize("T,K,O", [(1, 64, 36), (8, 768, 1000), (15, 1024, 33), (16, 1088, 64), (16, 2304, 20), (9, 1040, 31),
                                   (17, 1024, 32), (31, 1088, 100), (32, 2304, 33), (33, 320, 72)])
def test_few_tokens(T, K, O, N, M):
    assert product_route("plain", T, K, O, N, M)[0] == "direct"
    rng = np.random.default_rng(1000 * T + K + N * M)
    X, W = wl.draw_activations(rng, T, K), wl.draw_weights(rng, O, K)
    bias = rng.standard_normal(O).astype(np.float32)
    Yref, B = orc.nm_linear_from_bits(X, W, N, M, bias=bias)
    v, i = nm.nm_pack(dev_bf16(W), N, M)
    Xd, bd = dev_bf16(X), torch.from_numpy(bias).cuda()
    ws = nm.nm_spmm_prepare(v, i, K, N, M, T)
    for dt in (torch.float32, torch.bfloat16):
        y = nm.nm_linear_forward(v, i, K, N, M, Xd, bias=bd, out_dtype=dt)
        check_output(host_output(y), Yref, B + np.abs(bias)[None, :], K // M * N + 1, dt == torch.float32, (T, K, O, N, M))
        if product_route("prepared", T, K, O, N, M)[0] in ("tiled", "ragged"):
            assert torch.equal(y, nm.nm_linear_forward_prepared(v, i, K, N, M, Xd, ws, bias=bd, out_dtype=dt))
        if K % 64 == 0 and O % 4 == 0 and N != 3:
            p = nm.nm_linear_forward(v, i, K, N, M, Xd, bias=bd, out_dtype=dt, from_packed=True)
            check_output(host_output(p), Yref, B + np.abs(bias)[None, :], K // M * N + 1, dt == torch.float32, (T, K, O, N, M))
            q = torch.zeros_like(p)
            nm.nm_linear_forward_prepared_batched([(v, i, K, N, M, Xd, None, bd, q)])
            assert torch.equal(p, q)


@pytest.mark.parametrize("T,K,O,N,M", [(32, 512, 32752, 4, 8), (32, 512, 32768, 4, 8), (28, 1024, 32752, 4, 8), (28, 1024, 32768, 4, 8),
                                       (29, 1024, 32768, 4, 16), (25, 2048, 32768, 4, 16), (16, 1024, 21856, 3, 4), (9, 1024, 21824, 3, 4),
                                       (16, 2048, 98304, 4, 8), (24, 2048, 98304, 4, 8), (24, 2048, 98272, 4, 8)])
def test_large_weights(T, K, O, N, M):
    """The tokens of a block by the size of the weight: the bytes are those of its first and last rows alone, which are few."""
    g = torch.Generator(device="cuda")
    g.manual_seed(T + O)
    W, X = (torch.empty(n, K, dtype=torch.bfloat16, device="cuda").normal_(generator=g) for n in (O, T))
    v, i = nm.nm_pack(W, N, M)
    for packed in (False, True) if N == 4 else (False,):
        assert product_route("packed" if packed else "plain", T, K, O, N, M)[0] == "direct"
        y = nm.nm_linear_forward(v, i, K, N, M, X, from_packed=packed)
        for rows in (slice(0, 72), slice(O - 72, O)):
            part = nm.nm_linear_forward(v[rows], i[rows], K, N, M, X, from_packed=packed)
            assert torch.equal(y[:, rows], part)
