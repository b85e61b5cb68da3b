"""The second form of the kernel that decodes the weight itself (blocks of 64 out-features x 128 tokens): the bytes of a prepared
call and the oracle's bounds at the edges of its tiles, spans, chunks and rows."""
import numpy as np
import pytest
import torch

import paper_2409_09708_amd as nm
from oracle import nm_oracle as orc
from paper_2409_09708_amd import workloads as wl
from gpu_util import check_output, dev_bf16, host_output, product_route

pytestmark = pytest.mark.gpu

LEVELS = [(1, 4), (3, 4), (1, 8), (2, 8), (3, 8), (4, 8), (1, 16), (2, 16), (4, 16)]


def takes(T, K, O, N, M):
    kernel, tile = product_route("plain", T, K, O, N, M)
    return kernel == "direct" and tile[:2] == (64, 128)


# one and several spans of 128, a last span of one step, of a part of one, of half a chunk; tiles one short of full, full and one
# over in both directions
@pytest.mark.parametrize("N,M", LEVELS)
@pytest.mark.parametrize("T,K,O", [(1025, 64, 1096), (1664, 128, 769), (1663, 192, 768), (1151, 448, 832), (1153, 576, 1025),
                                   (1664, 208, 705), (1024, 328, 1088), (1000, 72, 1030), (1152, 872, 1001)])
def test_bytes_of_a_prepared_call(T, K, O, N, M):
    if K % M:
        pytest.skip("K is no whole number of groups")
    assert takes(T, K, O, N, M)
    rng = np.random.default_rng(7 * T + K + N * M)
    X = wl.draw_activations(rng, T, K)
    W = wl.tie_heavy_weights(rng, O, K) if (T + O) % 2 else wl.draw_weights(rng, O, K)
    bias = rng.standard_normal(O).astype(np.float32)
    v, i = nm.nm_pack(dev_bf16(W), N, M)
    bd = torch.from_numpy(bias).cuda()
    wide = torch.full((T, K + 16), float("nan"), dtype=torch.bfloat16, device="cuda")  # what lies behind a row is never used
    Xd = wide[:, 8:K + 8]
    Xd.copy_(dev_bf16(X))
    ws = nm.nm_spmm_prepare(v, i, K, N, M, T)
    rows = np.unique(np.concatenate([np.arange(8), np.arange(120, 136), np.arange(T - 8, T)]))
    Yref, B = orc.nm_linear_from_bits(X[rows], W, N, M, bias=bias)
    for dt, pad in ((torch.float32, 4), (torch.bfloat16, 8), (torch.float32, 1), (torch.bfloat16, 3)):
        out = torch.full((T + 1, O + 2 * pad), 7.0, dtype=dt, device="cuda")
        y = nm.nm_linear_forward(v, i, K, N, M, Xd, bias=bd, out=out[:T, pad:pad + O])
        assert bool((out[T] == 7).all() and (out[:, :pad] == 7).all() and (out[:, pad + O:] == 7).all())
        assert torch.equal(y, nm.nm_linear_forward_prepared(v, i, K, N, M, Xd, ws, bias=bd, out_dtype=dt))
        some = y[torch.from_numpy(rows).cuda()]
        check_output(host_output(some), Yref, B + np.abs(bias)[None, :], K // M * N + 1, dt == torch.float32, (T, K, O, N, M, dt))


@pytest.mark.parametrize("T,K,O,N,M", [(1152, 1000, 1001, 2, 8), (1152, 1000, 1001, 4, 8), (1664, 256, 768, 1, 16), (1664, 256, 768, 4, 8)])
def test_activations_that_are_not_finite(T, K, O, N, M):
    assert takes(T, K, O, N, M)
    g = torch.Generator(device="cuda")
    g.manual_seed(T + N)
    W, X = (torch.empty(n, K, dtype=torch.bfloat16, device="cuda").normal_(generator=g) for n in (O, T))
    X[3, 5], X[T - 1, K - 1], X[130, K // 2], X[131, 0] = float("inf"), float("-inf"), float("nan"), float("inf")
    v, i = nm.nm_pack(W, N, M)
    ws = nm.nm_spmm_prepare(v, i, K, N, M, T)
    for dt, bits in ((torch.float32, torch.int32), (torch.bfloat16, torch.int16)):
        y = nm.nm_linear_forward(v, i, K, N, M, X, out_dtype=dt)
        p = nm.nm_linear_forward_prepared(v, i, K, N, M, X, ws, out_dtype=dt)
        assert torch.equal(torch.isnan(y), torch.isnan(p))
        assert torch.equal(torch.nan_to_num(y).view(bits), torch.nan_to_num(p).view(bits))


def test_fixed_scratch_and_capture():
    T, K, O, N, M = 1576, 768, 1000, 2, 8
    assert takes(T, K, O, N, M)
    g = torch.Generator(device="cuda")
    g.manual_seed(1)
    W = torch.empty(O, K, dtype=torch.bfloat16, device="cuda").normal_(generator=g)
    X = torch.empty(T, K, dtype=torch.bfloat16, device="cuda").normal_(generator=g)
    v, i = nm.nm_pack(W, N, M)
    y = nm.nm_linear_forward(v, i, K, N, M, X)
    assert torch.equal(y, nm.nm_linear_forward_static(v, i, K, N, M, X))
    out = torch.zeros_like(y)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        nm.nm_linear_forward_static(v, i, K, N, M, X, out=out)
    for _ in range(3):
        X.normal_(generator=g)
        want = nm.nm_linear_forward(v, i, K, N, M, X)
        out.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, want)
