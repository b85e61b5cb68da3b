"""One prepared layer whose reduction is cut, used by several calls at once: a product alone reads the workspace and never writes
it, so the layers of a batched call may share one, calls on two streams do not disturb each other, and a graph keeps scratch
of its own.  The bytes are those of a call with a workspace to itself throughout."""
import numpy as np
import pytest
import torch

import paper_2409_09708_amd as nm
from paper_2409_09708_amd import workloads as wl
from gpu_util import dev_bf16

pytestmark = pytest.mark.gpu

# (T, K, O, N, M): 64 x 64 and 128 x 128 tiles, with an operand copy and from the packed layout
LAYERS = [(197, 4096, 1024, 2, 4), (197, 4096, 1024, 1, 8), (788, 5120, 1280, 4, 8), (130, 4160, 90, 2, 16)]


def layer(T, K, O, N, M, inputs):
    rng = np.random.default_rng(9300 + T + O)
    v, i = nm.nm_pack(dev_bf16(wl.draw_weights(rng, O, K)), N, M)
    ws = nm.nm_spmm_prepare(v, i, K, N, M, T)
    scratch = nm.load_library().nm_prepared_scratch_bytes(O, K, N, M, T)
    assert 2 * T * O * 4 <= scratch < ws.numel() + 256
    ws[ws.numel() - scratch:] = 0x5A  # (a workspace that the plain call fills ends in the partial sums)
    Xs = [dev_bf16(wl.draw_activations(rng, T, K)) for _ in range(inputs)]
    return v, i, ws, Xs, [nm.nm_linear_forward(v, i, K, N, M, X) for X in Xs]


@pytest.mark.parametrize("T,K,O,N,M", LAYERS)
def test_products_leave_the_workspace_alone(T, K, O, N, M):
    v, i, ws, (Xa, Xb), (ya, yb) = layer(T, K, O, N, M, 2)
    before = ws.clone()
    assert torch.equal(nm.nm_linear_forward_prepared(v, i, K, N, M, Xa, ws), ya)
    assert torch.equal(nm.nm_linear_forward_prepared(v, i, K, N, M, Xa, ws, stream=torch.cuda.current_stream()), ya)
    outs = [torch.zeros_like(ya), torch.zeros_like(yb)]
    nm.nm_linear_forward_prepared_batched([(v, i, K, N, M, X, ws, None, y) for X, y in zip((Xa, Xb), outs)])
    assert torch.equal(outs[0], ya) and torch.equal(outs[1], yb)
    # without scratch, or with too little of it: the uncut product, as from a workspace that holds the operand copy only
    operand = nm.nm_spmm_workspace_bytes(O, K, N, M, T) - nm.load_library().nm_prepared_scratch_bytes(O, K, N, M, T)
    uncut = nm.nm_linear_forward(v, i, K, N, M, Xa, workspace=torch.empty((max(operand, 256),), dtype=torch.uint8, device="cuda"))
    args = (v.data_ptr(), i.data_ptr(), O, K, N, M, Xa.data_ptr(), T, K, None, outs[0].data_ptr(), O, 0, ws.data_ptr(), ws.numel())
    lib, s = nm.load_library(), torch.cuda.current_stream().cuda_stream
    some = torch.empty((4096,), dtype=torch.uint8, device="cuda")
    for status in (lambda: lib.nm_linear_forward_prepared(*args, s),
                   lambda: lib.nm_linear_forward_prepared_scratch(*args, some.data_ptr(), some.numel(), s)):
        outs[0].zero_()
        assert status() == 0 and torch.equal(outs[0], uncut)
    assert torch.equal(ws, before)


@pytest.mark.parametrize("T,K,O,N,M", LAYERS)
def test_two_streams_share_a_prepared_layer(T, K, O, N, M):
    v, i, ws, Xs, expected = layer(T, K, O, N, M, 2)
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    named = [[torch.zeros_like(y) for _ in range(10)] for y in expected]
    torch.cuda.synchronize()
    outs = [[], []]
    for turn in range(10):
        for n, s in enumerate(streams):
            with torch.cuda.stream(s):
                outs[n].append(nm.nm_linear_forward_prepared(v, i, K, N, M, Xs[n], ws))
            if turn % 2:
                nm.nm_linear_forward_prepared(v, i, K, N, M, Xs[n], ws, out=named[n][turn], stream=s)
            else:
                nm.nm_linear_forward_prepared_batched([(v, i, K, N, M, Xs[n], ws, None, named[n][turn])], stream=s)
    torch.cuda.synchronize()
    for got, y in zip(outs, expected):
        assert all(torch.equal(g, y) for g in got)
    for got, y in zip(named, expected):
        assert all(torch.equal(g, y) for g in got)


def test_a_graph_of_a_cut_layer_replays():
    T, K, O, N, M = LAYERS[1]
    v, i, ws, (X, Xb), (y, yb) = layer(T, K, O, N, M, 2)
    out, both = torch.zeros_like(y), [torch.zeros_like(y), torch.zeros_like(y)]
    descs = nm.forward_descs([(v, i, K, N, M, X, ws, None, both[0]), (v, i, K, N, M, Xb, ws, None, both[1])])

    def calls():
        nm.nm_linear_forward_prepared(v, i, K, N, M, X, ws, out=out)
        nm.nm_linear_forward_prepared_batched(descs)
    calls()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        calls()
    for _ in range(3):
        for t in (out, *both):
            t.zero_()
        other = torch.full((T * O * 16,), 3.0, device="cuda")  # eager work between the replays takes memory of its own
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, y) and torch.equal(both[0], y) and torch.equal(both[1], yb)
        assert torch.equal(nm.nm_linear_forward_prepared(v, i, K, N, M, Xb, ws), yb) and bool((other == 3.0).all())
