"""The native marshalling of the per-layer calls against the Python functions it stands in for: the same bytes from both for
every form that it takes, and everything else left to Python."""
import numpy as np
import pytest
import torch

import paper_2409_09708_amd as nm
from paper_2409_09708_amd import binding


class _Declines:
    def __getattr__(self, name):
        return lambda *args: NotImplemented


def in_python(monkeypatch, call):
    binding._native()
    with monkeypatch.context() as m:
        m.setattr(binding, "_CALLS", _Declines())
        return call()


def test_declines_what_python_has_to_judge():
    calls = binding._native()
    W = torch.zeros(8, 64, dtype=torch.bfloat16)
    i32 = torch.zeros(8, 4, dtype=torch.int32)
    for done in (calls.prune(W, 2, 4, None, None), calls.prune_scored(W.float(), 2, 4, None), calls.pack(W, 2, 4, None, None),
                 calls.unpack(W, i32, 128, 2, 4, None), calls.prune("W", 2, 4, None, None), calls.prune(None, 2, 4, None, None),
                 calls.forward(W, i32, 128, 2, 4, W, None, None, None, None, None, 0), calls.pack(W, 2, 4)):
        assert done is NotImplemented
    with pytest.raises(ValueError, match="W must be a device tensor"):
        nm.nm_prune(W, 2, 4)
    with pytest.raises(KeyError):
        calls.bind({}, None, None)


def matrix(rows, cols, dtype, pitch, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    t = torch.empty(rows, cols + pitch, dtype=dtype, device="cuda").normal_(generator=g)
    return t[:, :cols]


@pytest.mark.gpu
@pytest.mark.parametrize("O,K,pitch", [(64, 128, 0), (64, 128, 8), (1, 64, 0), (5, 96, 32)])
def test_compression_calls(monkeypatch, O, K, pitch):
    W, score = matrix(O, K, torch.bfloat16, pitch, 1), matrix(O, K, torch.float32, pitch, 2)
    side = torch.cuda.Stream()

    def run(grad, stream):
        Wg = W.detach().requires_grad_(grad)
        Wm = torch.zeros(O, K + pitch, dtype=torch.bfloat16, device="cuda")[:, :K]
        mask = nm.nm_prune(Wg, 2, 8, W_masked=Wm, stream=stream)
        scored = nm.nm_prune_scored(score, 2, 4, stream=stream)
        v, i = nm.nm_pack(Wg, 2, 8, mask=mask, stream=stream)
        v4, i4 = nm.nm_pack(Wg, 1, 4, stream=stream)
        dense = nm.nm_unpack(v, i, K, 2, 8, stream=stream)
        torch.cuda.synchronize()
        return [mask, Wm, scored, v, i, v4, i4, dense]

    for grad, stream in ((False, None), (True, None), (False, side)):
        torch.cuda.synchronize()
        ours, theirs = run(grad, stream), in_python(monkeypatch, lambda: run(grad, stream))
        for a, b in zip(ours, theirs):
            assert a.dtype == b.dtype and a.shape == b.shape and a.stride() == b.stride() and a.device == b.device
            assert not a.requires_grad and torch.equal(a.contiguous().view(torch.uint8), b.contiguous().view(torch.uint8))
    assert binding._CALLS.prune(W, 2, 8, None, None) is not NotImplemented


@pytest.mark.gpu
@pytest.mark.parametrize("T,K,O", [(1, 64, 64), (197, 384, 256), (37, 100, 33), (300, 2048, 192)])
@pytest.mark.parametrize("out_dtype", [None, torch.float32, torch.bfloat16])
@pytest.mark.parametrize("bias,pitch", [(False, 0), (True, 8)])
def test_products(monkeypatch, T, K, O, out_dtype, bias, pitch):
    W, X = matrix(O, K, torch.bfloat16, 0, 1), matrix(T, K, torch.bfloat16, pitch, 2)
    b = matrix(1, O, torch.float32, 0, 3).view(O) if bias else None
    v, i = nm.nm_pack(W, 2, 4)
    ws = nm.nm_spmm_prepare(v, i, K, 2, 4, T)

    def run():
        out = torch.zeros(T, O + pitch, dtype=out_dtype or torch.float32, device="cuda")[:, :O]
        calls = [nm.nm_linear_forward(v, i, K, 2, 4, X, bias=b, out_dtype=out_dtype),
                 nm.nm_linear_forward(v, i, K, 2, 4, X, bias=b, out=out),
                 nm.nm_linear_forward_prepared(v, i, K, 2, 4, X, ws, bias=b, out_dtype=out_dtype),
                 nm.nm_linear_forward_static(v, i, K, 2, 4, X, bias=b, out_dtype=out_dtype)]
        if K % 64 == 0 and T <= 208 and O % 4 == 0:
            calls.append(nm.nm_linear_forward(v, i, K, 2, 4, X, bias=b, out_dtype=out_dtype, from_packed=True))
        assert calls[1] is out
        return calls

    for a, c in zip(run(), in_python(monkeypatch, run)):
        assert a.dtype == c.dtype and a.shape == c.shape and torch.equal(a, c)
    assert binding._CALLS.forward(v, i, K, 2, 4, X, b, out_dtype, None, ws, None, 1) is not NotImplemented


@pytest.mark.gpu
def test_refusals_and_wrapped_tensors():
    W, X = matrix(64, 128, torch.bfloat16, 0, 1), matrix(16, 128, torch.bfloat16, 0, 2)
    v, i = nm.nm_pack(W, 2, 4)
    with pytest.raises(nm.NmError):
        nm.nm_pack(W, 5, 4)
    with pytest.raises(nm.NmError):
        nm.nm_prune(W, 2, 6)
    with pytest.raises(ValueError):
        nm.nm_linear_forward(v, i, 64, 2, 4, X)
    with pytest.raises(ValueError):
        nm.nm_linear_forward(v, i, 128, 2, 4, X.float())
    with pytest.raises(ValueError):
        nm.nm_linear_forward_prepared(v, i, 128, 1, 4, X, None)
    with pytest.raises(ValueError):
        nm.nm_linear_forward(v, i, 128, 2, 4, X, out=torch.empty(16, 65, device="cuda"))
    with pytest.raises(ValueError):
        nm.nm_linear_forward(v, i, 128, 2, 4, X, out_dtype=torch.float16)
    calls = binding._native()

    class Sub(torch.Tensor):
        pass

    assert calls.prune(W.as_subclass(Sub), 2, 4, None, None) is NotImplemented
    assert calls.prune(W, np.int64(2), 4, None, None) is NotImplemented
    assert calls.prune(W.t(), 2, 4, None, None) is NotImplemented
    with torch.overrides.BaseTorchFunctionMode():
        assert calls.prune(W, 2, 4, None, None) is NotImplemented
    seen = []
    torch.func.vmap(lambda w: (seen.append(calls.prune(w, 2, 4, None, None)), w)[1])(W.view(1, 64, 128))
    assert seen == [NotImplemented]
