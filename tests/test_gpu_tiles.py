"""The tiles of the tiled product kernel a single layer may take (64 x 64 to 128 x 128, two to four LDS stages): one
shape per tile and operand form, tokens and out-features off the tile edge, both weight orders, both output types; the
same bytes as inside a batched call, which may use another tile."""
import numpy as np
import pytest
import torch

import paper_2409_09708_amd as nm
from oracle import nm_oracle as orc
from paper_2409_09708_amd import workloads as wl
from gpu_util import check_output, dev_bf16, host_output, product_route

pytestmark = pytest.mark.gpu

# (T, K, O) by operand form and tile (out-features, tokens, stages)
SPARSE = {(64, 64, 3): (397, 192, 504), (128, 64, 3): (789, 192, 1272), (128, 128, 3): (2999, 512, 760),
          (64, 64, 4): (397, 3072, 504), (128, 64, 4): (789, 2048, 1272), (128, 128, 4): (2999, 2048, 760),
          (128, 128, 2): (2999, 192, 760)}
DENSE = {(64, 64, 3): (397, 192, 504), (128, 64, 3): (789, 192, 1272), (128, 128, 3): (2999, 1600, 760),
         (64, 64, 4): (397, 2048, 504), (128, 64, 4): (789, 2112, 1272), (128, 128, 4): (2999, 2048, 760),
         (128, 128, 2): (8133, 192, 584)}
CASES = ([(s, lv, tile) for tile, s in SPARSE.items() for lv in ((2, 4), (1, 8))] +
         [(s, lv, tile) for tile, s in DENSE.items() for lv in ((4, 8), (4, 4))])
OTHERS = [((2999, 192, 760), lv, None) for lv in ((4, 8), (4, 4))]  # whichever tile


@pytest.mark.parametrize("shape,level,tile", CASES + OTHERS)
def test_products(shape, level, tile):
    (T, K, O), (N, M) = shape, level
    assert tile is None or product_route("prepared", T, K, O, N, M) == ("tiled", tile)
    rng = np.random.default_rng(13000 + N * 17 + M + T)
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
    both = [torch.empty((T, O), dtype=torch.float32, device="cuda") for _ in range(2)]
    nm.nm_linear_forward_prepared_batched([(v, i, K, N, M, Xd, ws, bd, b) for b in both])
    assert torch.equal(both[0], y) and torch.equal(both[1], y)


@pytest.mark.parametrize("blocks,T", [(1, 197), (2, 197), (3, 130)])
def test_batched_calls_with_narrow_tiles(blocks, T):
    # few layers of unequal depth: the deep ones take tiles of 64 out-features, ragged in both directions; the same bytes
    # as the single calls
    rng = np.random.default_rng(13500 + blocks + T)
    levels = [(2, 4), (4, 8), (1, 8), (4, 4), (2, 8), (4, 16), (1, 16)]
    descs, singles = [], []
    for n in range(4 * blocks):
        K, O = ((768, 2304), (768, 776), (768, 3072), (3072, 776))[n % 4]
        N, M = levels[(n + n // 4) % 7]
        X = dev_bf16(wl.draw_activations(rng, T, K))
        v, i = nm.nm_pack(dev_bf16(wl.draw_weights(rng, O, K)), N, M)
        ws = nm.nm_spmm_prepare(v, i, K, N, M, T)
        out = torch.full((T + 1, O), 7.0, dtype=torch.bfloat16 if n % 2 else torch.float32, device="cuda")
        singles.append(nm.nm_linear_forward_prepared(v, i, K, N, M, X, ws, out_dtype=out.dtype))
        descs.append((v, i, K, N, M, X, ws, None, out))
    nm.nm_linear_forward_prepared_batched([d[:8] + (d[8][:T],) for d in descs])
    for d, y in zip(descs, singles):
        assert torch.equal(d[8][:T], y) and bool((d[8][T] == 7).all()), d[2:5]
