"""Native marshalling of the training products and of the int8 layer against the Python functions it stands in for."""
import pytest
import torch

import paper_2409_09708_amd as nm
from paper_2409_09708_amd import binding
from test_gpu_calls import in_python, matrix


def test_declines_what_python_has_to_judge():
    calls = binding._native()
    W, q = torch.zeros(8, 64, dtype=torch.bfloat16), torch.zeros(8, 64, dtype=torch.int8)
    words = torch.zeros(8, 2, dtype=torch.int32)
    for done in (calls.backward_input(W, W, None, None, None, None), calls.backward_weight(W, W, None, None, None, None, None),
                 calls.forward_i8(q, words, None, 2, 4, q, 1.0, None, None, None, None, None, None, 0), calls.backward_input(W),
                 calls.backward_weight(), calls.forward_i8(q)):
        assert done is NotImplemented
    with pytest.raises(ValueError, match="must be a device tensor"):
        nm.nm_linear_backward_input(W, W)
    with pytest.raises(ValueError, match="must be a device tensor"):
        nm.nm_linear_forward_i8(q, words, 2, 4, q)


def same(ours, theirs):
    for a, b in zip(ours, theirs, strict=True):
        assert a.dtype == b.dtype and a.shape == b.shape and a.stride() == b.stride() and a.device == b.device
        assert torch.equal(a.contiguous().view(torch.uint8), b.contiguous().view(torch.uint8))


@pytest.mark.gpu
@pytest.mark.parametrize("T,K,O,pitch", [(5, 64, 64, 0), (197, 384, 256, 8), (300, 100, 33, 0), (2048, 512, 768, 0)])
def test_training_products(monkeypatch, T, K, O, pitch):
    W, X, dY = matrix(O, K, torch.bfloat16, pitch, 1), matrix(T, K, torch.bfloat16, pitch, 2), matrix(T, O, torch.bfloat16, pitch, 3)
    mask = nm.nm_prune(W, 2, 4)
    side = torch.cuda.Stream()

    def run(stream):
        outs = []
        for dt in (None, torch.float32, torch.bfloat16):
            dX = torch.zeros(T, K + pitch, dtype=dt or torch.float32, device="cuda")[:, :K]
            dW = torch.zeros(O, K + pitch, dtype=dt or torch.float32, device="cuda")[:, :K]
            torch.cuda.synchronize()
            own = torch.empty(max(1, nm.nm_backward_weight_workspace_bytes(O, K, T)), dtype=torch.uint8, device="cuda")
            outs += [nm.nm_linear_backward_input(W, dY, out_dtype=dt, stream=stream), nm.nm_linear_backward_input(W, dY, out=dX, stream=stream),
                     nm.nm_linear_backward_weight(dY, X, mask=mask, out_dtype=dt, stream=stream),
                     nm.nm_linear_backward_weight(dY, X, out=dW, workspace=own, stream=stream)]
            assert outs[-3] is dX and outs[-1] is dW
        torch.cuda.synchronize()
        return outs

    for stream in (None, side):
        same(run(stream), in_python(monkeypatch, lambda: run(stream)))
    assert binding._CALLS.backward_input(W, dY, None, None, None, None) is not NotImplemented
    assert binding._CALLS.backward_weight(dY, X, mask, None, None, None, None) is not NotImplemented


@pytest.mark.gpu
@pytest.mark.parametrize("T,K,O", [(5, 128, 64), (197, 384, 256), (37, 96, 33)])
def test_int8_layers(monkeypatch, T, K, O):
    g = torch.Generator(device="cuda")
    g.manual_seed(T)
    draw = lambda r, c: torch.randint(-127, 128, (r, c), dtype=torch.int8, device="cuda", generator=g)
    Wq, Xq, mask = draw(O, K), draw(T, K), nm.nm_prune(matrix(O, K, torch.bfloat16, 0, 1), 2, 8)
    scale, bias = matrix(1, O, torch.float32, 0, 2).view(O), matrix(1, O, torch.float32, 0, 3).view(O)
    v, i = nm.nm_pack_i8(Wq, mask, 2, 8)
    ws = nm.nm_i8_prepare(Wq, mask, 2, 8, T)

    def run():
        outs = []
        for dt in (None, torch.bfloat16, torch.int32):
            out = torch.zeros(T, O, dtype=dt or torch.float32, device="cuda")
            outs += [nm.nm_linear_forward_i8(Wq, mask, 2, 8, Xq, x_scale=0.5, w_scale=scale, bias=bias, out_dtype=dt),
                     nm.nm_linear_forward_i8_packed(v, i, K, 2, 8, Xq, out=out),
                     nm.nm_linear_forward_i8(Wq, mask, 2, 8, Xq, x_scale=2)]
            if ws is not None:
                outs += [nm.nm_linear_forward_i8_prepared(Wq, mask, 2, 8, Xq, ws, x_scale=0.5, bias=bias, out_dtype=dt),
                         nm.nm_linear_forward_i8_packed_prepared(v, i, K, 2, 8, Xq, ws, w_scale=scale, out_dtype=dt)]
        return outs

    same(run(), in_python(monkeypatch, run))
    assert binding._CALLS.forward_i8(Wq, mask, None, 2, 8, Xq, 1.0, scale, None, None, None, None, None, 0) is not NotImplemented


@pytest.mark.gpu
def test_refusals():
    W, X, dY = matrix(64, 128, torch.bfloat16, 0, 1), matrix(16, 128, torch.bfloat16, 0, 2), matrix(16, 64, torch.bfloat16, 0, 3)
    with pytest.raises(ValueError):
        nm.nm_linear_backward_input(W, X)
    with pytest.raises(ValueError):
        nm.nm_linear_backward_input(W, dY, out_dtype=torch.float16)
    with pytest.raises(ValueError):
        nm.nm_linear_backward_weight(dY, X[:8])
    with pytest.raises(ValueError):
        nm.nm_linear_backward_weight(dY, X, mask=torch.zeros(64, 5, dtype=torch.int32, device="cuda"))
    with pytest.raises(ValueError):
        nm.nm_linear_backward_weight(dY, X, out=torch.zeros(64, 127, device="cuda"))
    Wq, mask = torch.zeros(64, 128, dtype=torch.int8, device="cuda"), nm.nm_prune(W, 2, 4)
    with pytest.raises(ValueError):
        nm.nm_linear_forward_i8(Wq, mask, 2, 4, Wq[:, :64])
    with pytest.raises(ValueError):
        nm.nm_linear_forward_i8_prepared(Wq, mask, 2, 4, Wq, None)
    with pytest.raises(ValueError):
        nm.nm_linear_forward_i8(Wq, mask, 2, 4, Wq, w_scale=torch.zeros(63, device="cuda"))
