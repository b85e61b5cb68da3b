"""GPU parity of products whose operands fit no tile: a reduction that is no multiple of 64, rows of X that start at any
element, outputs whose rows are not whole 16-byte pieces."""
import numpy as np
import pytest
import torch

import paper_2409_09708_amd as nm
from oracle import nm_oracle as orc
from paper_2409_09708_amd import workloads as wl
from gpu_util import check_output, dev_bf16, host_output

pytestmark = pytest.mark.gpu


def layer(seed, T, K, O, N, M):
    rng = np.random.default_rng(seed)
    X, W = wl.draw_activations(rng, T, K), wl.draw_weights(rng, O, K)
    bias = rng.standard_normal(O).astype(np.float32)
    Yref, B = orc.nm_linear_from_bits(X, W, N, M, bias=bias)
    v, i = nm.nm_pack(dev_bf16(W), N, M)
    return X, v, i, torch.from_numpy(bias).cuda(), Yref, B + np.abs(bias)[None, :]


# K just above one step, half a step, a step but four, one group past a step; O and T off every tile edge; a few tiles
# (64 x 64) and enough for the 128 x 128 ones
@pytest.mark.parametrize("N,M", [(1, 4), (2, 4), (3, 4), (4, 4), (2, 8), (4, 8), (8, 8), (1, 16), (2, 16), (4, 16), (16, 16)])
@pytest.mark.parametrize("T,K,O", [(1, 80, 1), (67, 96, 65), (130, 176, 131), (197, 1072, 77), (2049, 144, 2047)])
def test_reductions_off_the_step(T, K, O, N, M):
    X, v, i, bias, Yref, B = layer(11000 + N * 17 + M + T + K, T, K, O, N, M)
    Xd = dev_bf16(X)
    y = nm.nm_linear_forward(v, i, K, N, M, Xd, bias=bias)
    check_output(host_output(y), Yref, B, K // M * N + 1, True, (T, K, O, N, M))
    y16 = nm.nm_linear_forward(v, i, K, N, M, Xd, bias=bias, out_dtype=torch.bfloat16)
    check_output(host_output(y16), Yref, B, K // M * N + 1, False, (T, K, O, N, M))
    ws = nm.nm_spmm_prepare(v, i, K, N, M, T)
    assert ws is not None
    assert torch.equal(y, nm.nm_linear_forward_prepared(v, i, K, N, M, Xd, ws, bias=bias))


@pytest.mark.parametrize("K", [68, 100, 124, 132, 252])  # multiples of 4 only
def test_reductions_that_end_inside_a_piece(K):
    T, O, N, M = 70, 66, 2, 4
    X, v, i, bias, Yref, B = layer(11500 + K, T, K, O, N, M)
    y = nm.nm_linear_forward(v, i, K, N, M, dev_bf16(X), bias=bias)
    check_output(host_output(y), Yref, B, K // M * N + 1, True, K)


# X and Y as views: rows that start on 16-, 8-, 4- and 2-byte boundaries; what lies beside the view (NaN around X, a
# guard value around Y) is neither read into a sum nor written
@pytest.mark.parametrize("offset,pad", [(0, 8), (4, 12), (2, 6), (1, 7), (3, 1)])
@pytest.mark.parametrize("K,N,M", [(104, 2, 8), (192, 4, 8), (192, 1, 4), (192, 2, 4), (192, 4, 4)])
@pytest.mark.parametrize("T", [75, 4200])
def test_views_of_any_alignment(offset, pad, K, N, M, T):
    O = 263 if T < 4000 else 2051
    X, v, i, bias, Yref, B = layer(11700 + K + N + T, T, K, O, N, M)
    wide = torch.full((T, K + offset + pad), float("nan"), dtype=torch.bfloat16, device="cuda")
    wide[:, offset:offset + K] = dev_bf16(X)
    out = torch.full((T, O + 2), 7.0, dtype=torch.bfloat16, device="cuda")
    nm.nm_linear_forward(v, i, K, N, M, wide[:, offset:offset + K], bias=bias, out=out[:, 1:O + 1])
    check_output(host_output(out[:, 1:O + 1].contiguous()), Yref, B, K // M * N + 1, False, (offset, pad, K, N, M, T))
    assert bool((out[:, 0] == 7).all()) and bool((out[:, O + 1] == 7).all())


def test_without_a_workspace_the_same_product():
    T, K, O, N, M = 50, 200, 40, 2, 8
    X, v, i, bias, Yref, B = layer(11900, T, K, O, N, M)
    y = nm.nm_linear_forward(v, i, K, N, M, dev_bf16(X), bias=bias, from_packed=True)
    check_output(host_output(y), Yref, B, K // M * N + 1, True, "gather kernel")
    y = nm.nm_linear_forward_prepared(v, i, K, N, M, dev_bf16(X), None, bias=bias)
    check_output(host_output(y), Yref, B, K // M * N + 1, True, "prepared, no workspace")
    y = nm.nm_linear_forward_static(v, i, K, N, M, dev_bf16(X), bias=bias)
    check_output(host_output(y), Yref, B, K // M * N + 1, True, "fixed scratch")


def test_ragged_layers_packed_and_prepared_in_one_call():
    rng = np.random.default_rng(11950)
    specs = [(100, 96, 256, 2, 8), (100, 160, 512, 4, 8), (70, 72, 30, 1, 4), (64, 128, 256, 1, 8)]
    Ws = [dev_bf16(wl.draw_weights(rng, O, K)) for _, K, O, _, _ in specs]
    packed, wss = nm.nm_pack_prepare_batched([(W, N, M, T) for W, (T, _, _, N, M) in zip(Ws, specs)])
    for W, (v, i), ws, (T, K, O, N, M) in zip(Ws, packed, wss, specs):
        alone = nm.nm_spmm_prepare(v, i, K, N, M, T)
        assert torch.equal(ws, alone), (T, K, O, N, M)


# X in whole 16-byte pieces with a reduction that ends inside a step, on each tile of that form: 1 to 7 pieces in the last
# step, steps fewer and more than the stages; the rows' neighbours and what follows the last row are NaN
@pytest.mark.parametrize("N,M", [(2, 8), (4, 8)])
@pytest.mark.parametrize("T,K,O", [(67, 72, 65), (130, 248, 131), (789, 1000, 1272), (2999, 200, 761), (2999, 968, 761)])
def test_whole_pieces_and_a_short_last_step(T, K, O, N, M):
    X, v, i, bias, Yref, B = layer(11980 + N + T + K, T, K, O, N, M)
    flat = torch.full((T * (K + 16) + 64,), float("nan"), dtype=torch.bfloat16, device="cuda")
    for pitch in (K, K + 16):
        view = torch.as_strided(flat, (T, K), (pitch, 1), 8)
        view.copy_(dev_bf16(X))
        y = nm.nm_linear_forward(v, i, K, N, M, view, bias=bias)
        check_output(host_output(y), Yref, B, K // M * N + 1, True, (T, K, O, N, M, pitch))
        flat.fill_(float("nan"))


# An infinity or NaN among the activations: products that reach the zero-padded operand give what the gather gives, which
# never reads an activation at a pruned position (without a workspace these views run it).  The forms are the
# asynchronous copies and the registers, on both tiles, and an output whose rows the persistent kernel cannot write.
@pytest.mark.parametrize("N,M", [(1, 4), (2, 8), (4, 8), (1, 16), (6, 16)])
@pytest.mark.parametrize("T,K,O,offset", [(67, 80, 65, 0), (70, 80, 64, 0), (67, 176, 65, 1), (2049, 176, 2047, 0), (2049, 176, 2047, 1),
                                          (130, 192, 131, 2), (12001, 192, 771, 0)])
def test_activations_that_are_not_finite(T, K, O, offset, N, M):
    rng = np.random.default_rng(11990 + T + K + N + M)
    X = dev_bf16(wl.draw_activations(rng, T, K))
    X[:, 5] = float("inf")
    X[T // 2, 17] = float("nan")
    X[T - 1, :] = float("-inf")
    v, i = nm.nm_pack(dev_bf16(wl.draw_weights(rng, O, K)), N, M)
    bias = torch.from_numpy(rng.standard_normal(O).astype(np.float32)).cuda()
    wide = torch.zeros((T, K + 9), dtype=torch.bfloat16, device="cuda")
    one = wide[:, 1:K + 1]  # a view that is multiplied by the gather kernel when there is no workspace
    one.copy_(X)
    view = X
    if offset:
        wide2 = torch.zeros((T, K + 10), dtype=torch.bfloat16, device="cuda")
        view = wide2[:, offset:offset + K]
        view.copy_(X)
    ref = nm.nm_linear_forward(v, i, K, N, M, one, bias=bias, from_packed=True)
    y = nm.nm_linear_forward(v, i, K, N, M, view, bias=bias)
    assert torch.equal(torch.isnan(y), torch.isnan(ref))
    assert torch.equal(torch.isinf(y), torch.isinf(ref)) and torch.equal(y[torch.isinf(y)], ref[torch.isinf(ref)])
    assert bool(torch.isfinite(y).any())
    # finite sums: two orders of an fp32 sum of terms + 1 products, each within (terms + 2) 2^-24 sum |x w| of the exact one
    finite = torch.where(torch.isfinite(X), X, torch.zeros_like(X))
    B = finite.double().abs() @ nm.nm_unpack(v, i, K, N, M).double().abs().t() + bias.double().abs()
    ok = torch.isfinite(ref)
    assert bool(((y.double() - ref.double()).abs()[ok] <= 2 * (K // M * N + 3) * 2.0 ** -24 * B[ok]).all())
    y16 = nm.nm_linear_forward(v, i, K, N, M, view, bias=bias, out_dtype=torch.bfloat16)
    assert torch.equal(torch.isnan(y16), torch.isnan(ref)) and torch.equal(torch.isinf(y16), torch.isinf(ref.bfloat16()))


# The call on the fixed scratch, at operand copies that fit it and that are larger: 16 blocks of 256 out-features fit at
# K = 1000 in the dense form, 29 in the 2:4 form
@pytest.mark.parametrize("T,K,O,N,M", [(70, 1000, 4096, 4, 8), (70, 1000, 4097, 4, 8), (300, 1000, 8448, 4, 8),
                                       (70, 1000, 7425, 2, 8), (70, 4004, 3001, 3, 4)])
@pytest.mark.parametrize("out_dtype", [torch.float32, torch.bfloat16])
def test_fixed_scratch_writes_the_same_bytes(T, K, O, N, M, out_dtype):
    X, v, i, bias, _, _ = layer(12100 + O + N, T, K, O, N, M)
    Xd = dev_bf16(X)
    y = nm.nm_linear_forward(v, i, K, N, M, Xd, bias=bias, out_dtype=out_dtype)
    out = torch.full((T, O + 3), 7.0, dtype=out_dtype, device="cuda")
    nm.nm_linear_forward_static(v, i, K, N, M, Xd, bias=bias, out=out[:, 1:O + 1])
    assert torch.equal(out[:, 1:O + 1], y)
    assert bool((out[:, 0] == 7).all() and (out[:, O + 1:] == 7).all())


# Outputs of a few columns, on either side of the widths where the write-out changes (16 columns; a wave's 32 or 64), by
# every kernel that writes rows of any alignment; what lies beside the view stays
@pytest.mark.parametrize("cols", [1, 3, 4, 13, 15, 16, 17, 31, 33, 65])
@pytest.mark.parametrize("out_dtype", [torch.float32, torch.bfloat16])
def test_narrow_outputs(cols, out_dtype):
    T, K = 133, 128
    rng = np.random.default_rng(12300 + cols)
    Xd = dev_bf16(wl.draw_activations(rng, T, K))
    W = dev_bf16(wl.draw_weights(rng, cols, K))
    out = torch.full((T + 1, cols + 3), 7.0, dtype=out_dtype, device="cuda")

    def same(view, ref, B, terms):
        bound = (terms + 2) * 2.0 ** -24 * B + (2.0 ** -8 * ref.abs() if out_dtype == torch.bfloat16 else 0)
        assert bool(((view.double() - ref).abs() <= bound).all())
        assert bool((out[:, 0] == 7).all() and (out[:, 1 + view.shape[1]:] == 7).all() and (out[view.shape[0]:] == 7).all())
        out.fill_(7.0)

    for N, M in ((2, 4), (1, 8), (4, 8)):
        v, i = nm.nm_pack(W, N, M)
        Ws = nm.nm_unpack(v, i, K, N, M).double()
        ws = nm.nm_spmm_prepare(v, i, K, N, M, T)
        y = nm.nm_linear_forward_prepared(v, i, K, N, M, Xd, ws, out=out[:T, 1:cols + 1])
        same(y, Xd.double() @ Ws.t(), Xd.double().abs() @ Ws.abs().t(), K // M * N)
    # weight gradient: rows of `cols` columns; input gradient likewise
    dY = dev_bf16(wl.draw_activations(rng, T, 96))
    Xn = dev_bf16(wl.draw_activations(rng, T, cols))
    if cols % 8 == 0:
        dW = nm.nm_linear_backward_weight(dY, Xn, out=out[:96, 1:cols + 1])
        same(dW, dY.double().t() @ Xn.double(), dY.double().abs().t() @ Xn.double().abs(), T)
        Wd = dev_bf16(wl.draw_weights(rng, 96, cols))
        dX = nm.nm_linear_backward_input(Wd, dY, out=out[:T, 1:cols + 1])
        same(dX, dY.double() @ Wd.double(), dY.double().abs() @ Wd.double().abs(), 96)
    # int8: the rescaled sums, one rounding of a fused multiply-add
    Xq, Wq = torch.from_numpy(wl.draw_int8(rng, T, K)).cuda(), torch.from_numpy(wl.draw_int8(rng, cols, K)).cuda()
    mask = nm.nm_prune(Wq.to(torch.bfloat16), 2, 4)
    y = nm.nm_linear_forward_i8(Wq, mask, 2, 4, Xq, x_scale=0.25, out=out[:T, 1:cols + 1])
    kept = ((mask[:, :, None] >> torch.arange(32, device="cuda")) & 1).reshape(cols, -1)[:, :K]
    ref = 0.25 * (Xq.double() @ (Wq * kept).double().t())
    same(y, ref, ref.abs(), 1)
