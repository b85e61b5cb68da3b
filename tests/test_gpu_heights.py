"""The tile heights of the persistent product kernel (128 to 256 tokens): shapes that take each of them, with tokens off
the tile edge, odd and even step counts, a bias and every output type; the same bytes alone and inside a batched call,
whose launch may use another height."""
import numpy as np
import pytest
import torch

import paper_2409_09708_amd as nm
from oracle import nm_oracle as orc
from paper_2409_09708_amd import workloads as wl
from gpu_util import check_output, dev_bf16, dev_words, host_output, int8_route, product_route

pytestmark = pytest.mark.gpu

# (T, K, O) by operand form and tokens per tile: odd and even step counts, T and O off the tile edge
SPARSE = {128: (16565, 320, 136), 160: (16413, 128, 392), 192: (13733, 320, 520), 224: (16409, 192, 648), 256: (19586, 128, 520)}
DENSE = {128: (16525, 192, 136), 160: (16654, 128, 392), 192: (13625, 192, 520), 224: (16414, 128, 648), 256: (19713, 192, 520)}
CASES = ([(s, lv, tokens) for tokens, s in SPARSE.items() for lv in ((2, 4), (1, 8))] +
         [(s, lv, tokens) for tokens, s in DENSE.items() for lv in ((4, 8), (8, 8))])
OTHERS = [(s, lv, None) for lv in ((2, 4), (1, 8), (4, 8), (8, 8))  # whichever kernel
          for s in ((12001, 192, 768), (15873, 128, 768), (6301, 64, 2560), (5500, 320, 3072), (8200, 192, 2048), (16384, 128, 1024))]
SPARSE_I8 = {128: (16451, 512, 136), 160: (16444, 384, 136), 192: (13658, 384, 528), 224: (16368, 384, 520), 256: (19889, 384, 520)}
DENSE_I8 = {128: (4164, 512, 136), 160: (16826, 256, 264), 192: (13702, 256, 520), 224: (16392, 256, 520), 256: (19280, 256, 520)}
INT8_CASES = [(s, lv, t) for t, s in SPARSE_I8.items() for lv in ((2, 4), (1, 8))] + [(s, (4, 8), t) for t, s in DENSE_I8.items()]
INT8_OTHERS = [(s, lv, None) for lv in ((2, 4), (4, 8))
               for s in ((12001, 384, 768), (15873, 512, 768), (6301, 640, 2560), (8200, 1024, 2048))]


@pytest.mark.parametrize("shape,level,tokens", CASES + OTHERS)
def test_products(shape, level, tokens):
    (T, K, O), (N, M) = shape, level
    if tokens is not None:
        kernel, tile = product_route("prepared", T, K, O, N, M)
        assert kernel == "persistent" and tile[1] == tokens
    rng = np.random.default_rng(12000 + N * 17 + M + T)
    X, W = wl.draw_activations(rng, T, K), wl.draw_weights(rng, O, K)
    bias = rng.standard_normal(O).astype(np.float32)
    Yref, B = orc.nm_linear_from_bits(X, W, N, M, bias=bias)
    B = B + np.abs(bias)[None, :]
    v, i = nm.nm_pack(dev_bf16(W), N, M)
    Xd, bd = dev_bf16(X), torch.from_numpy(bias).cuda()
    y = nm.nm_linear_forward(v, i, K, N, M, Xd, bias=bd)
    check_output(host_output(y), Yref, B, K // M * N + 1, True, (T, K, O, N, M))
    out = torch.full((T + 1, O), 7.0, dtype=torch.bfloat16, device="cuda")
    ws = nm.nm_spmm_prepare(v, i, K, N, M, T)
    nm.nm_linear_forward_prepared(v, i, K, N, M, Xd, ws, bias=bd, out=out[:T])
    check_output(host_output(out[:T]), Yref, B, K // M * N + 1, False, (T, K, O, N, M))
    assert bool((out[T] == 7).all())
    # beside a layer with many more tiles: another height, the same sums
    T2 = 40000
    X2 = dev_bf16(wl.draw_activations(rng, T2, K))
    ws2 = nm.nm_spmm_prepare(v, i, K, N, M, T2)
    y2 = torch.empty((T2, O), dtype=torch.bfloat16, device="cuda")
    both = torch.zeros((T, O), dtype=torch.float32, device="cuda")
    nm.nm_linear_forward_prepared_batched([(v, i, K, N, M, Xd, ws, bd, both), (v, i, K, N, M, X2, ws2, None, y2)])
    assert torch.equal(both, y)


@pytest.mark.parametrize("shape,level,tokens", INT8_CASES + INT8_OTHERS)
def test_int8_products(shape, level, tokens):
    (T, K, O), (N, M) = shape, level
    assert tokens is None or int8_route(T, K, O, N, M) == ("persistent", tokens)
    rng = np.random.default_rng(12500 + N + T)
    xq, wq = wl.draw_int8(rng, T, K), wl.draw_int8(rng, O, K)
    mask = orc.nm_mask(wl.f32_to_bf16_bits(wq.astype(np.float32)), N, M)
    words = dev_words(orc.mask_to_words(mask))
    acc = nm.nm_linear_forward_i8(torch.from_numpy(wq).cuda(), words, N, M, torch.from_numpy(xq).cuda(), out_dtype=torch.int32)
    ref = xq.astype(np.float32) @ (wq * mask).astype(np.float32).T  # exact: |sums| < 1024 * 127 * 127 < 2^24
    assert K * 127 * 127 < 2 ** 24 and np.array_equal(acc.cpu().numpy(), ref.astype(np.int32))
    scale = torch.from_numpy(rng.random(O).astype(np.float32)).cuda()
    bias = torch.from_numpy(rng.standard_normal(O).astype(np.float32)).cuda()
    y = nm.nm_linear_forward_i8(torch.from_numpy(wq).cuda(), words, N, M, torch.from_numpy(xq).cuda(), x_scale=0.02,
                                w_scale=scale, bias=bias)
    expect = torch.addcmul(bias.double(), acc.double(), (0.02 * scale).double())  # one rounding of the fused multiply-add
    assert (y.double() - expect).abs().max().item() <= 2.0 ** -23 * expect.abs().max().item()
    # bfloat16 rows leave by a write-out of their own: the rounding of the fp32 output, bit for bit, and nothing past the last row
    out = torch.full((T + 1, O), 7.0, dtype=torch.bfloat16, device="cuda")
    nm.nm_linear_forward_i8(torch.from_numpy(wq).cuda(), words, N, M, torch.from_numpy(xq).cuda(), x_scale=0.02, w_scale=scale,
                            bias=bias, out=out[:T])
    assert torch.equal(out[:T], y.bfloat16()) and bool((out[T] == 7).all())
