"""Plain calls of large layers whose output rows are no whole 16-byte pieces: one launch, and what a prepared call gives, also for
activations that are not finite at positions that are pruned."""
import pytest
import torch

import paper_2409_09708_amd as nm
from gpu_util import product_route

pytestmark = pytest.mark.gpu


# O that is no whole number of pieces in both output types and in bfloat16 alone; aligned O in rows of an odd pitch
@pytest.mark.parametrize("T,K,O,N,M,pitch", [(1280, 64, 3241, 1, 4, 0), (5471, 64, 641, 1, 16, 0), (5400, 128, 645, 2, 8, 0),
                                             (770, 128, 4636, 4, 8, 0), (1408, 128, 3200, 3, 8, 1)])
def test_infinities_at_pruned_positions(T, K, O, N, M, pitch):
    kernel, tile = product_route("plain", T, K, O, N, M)
    assert kernel == "direct" and tile[:2] == (64, 128) and ((O + 127) // 128) * ((T + 127) // 128) > 256
    g = torch.Generator(device="cuda")
    g.manual_seed(T + N)
    W, X = (torch.empty(n, K, dtype=torch.bfloat16, device="cuda").normal_(generator=g) for n in (O, T))
    places = [(0, 3), (T // 2, K - 1), (T - 1, K // 2)]
    for n, (t, k) in enumerate(places):
        X[t, k] = (float("inf"), float("-inf"), float("nan"))[n]
    v, i = nm.nm_pack(W, N, M)
    kept = nm.nm_unpack(v, i, K, N, M) != 0
    ws = nm.nm_spmm_prepare(v, i, K, N, M, T)
    for dt, bits in ((torch.float32, torch.int32), (torch.bfloat16, torch.int16)):
        y, p = (torch.zeros(T, O + pitch, dtype=dt, device="cuda")[:, :O] for _ in range(2))
        nm.nm_linear_forward(v, i, K, N, M, X, out=y)
        nm.nm_linear_forward_prepared(v, i, K, N, M, X, ws, out=p)
        if dt == torch.bfloat16 or O % 4 or pitch:  # (rows of whole pieces: the matrix instructions may multiply by a zero)
            for t, k in places:
                assert bool((torch.isfinite(y[t]) == ~kept[:, k]).all()), (t, k, dt)
        assert torch.equal(torch.isnan(y), torch.isnan(p))
        assert torch.equal(torch.nan_to_num(y).view(bits), torch.nan_to_num(p).view(bits))
