"""dX of few tokens: the transposed copy and the tiled kernel where the scratch for it is there, the same bits without."""
import numpy as np
import pytest
import torch

import paper_2409_09708_amd as nm
from oracle import nm_oracle as orc
from paper_2409_09708_amd import workloads as wl
from paper_2409_09708_amd.binding import load_library
from gpu_util import check_output, dev_bf16, host_output


def test_scratch_is_beside_what_is_required():
    lib = load_library()
    for O, K, T in ((3072, 768, 197), (2304, 768, 1576), (768, 768, 20), (256, 256, 3152), (4096, 1024, 788)):
        assert lib.nm_backward_input_workspace_bytes(O, K, T) == 0
        assert lib.nm_backward_input_scratch_bytes(O, K, T) == (K + 255) // 256 * 256 * O * 2
    for O, K, T in ((512, 3456, 495), (800, 768, 197), (64, 904, 5388), (0, 64, 1)):  # its own kernel is faster, or no whole steps
        assert lib.nm_backward_input_scratch_bytes(O, K, T) == 0
    for O, K, T in ((768, 768, 12608), (2304, 768, 12608)):
        assert lib.nm_backward_input_scratch_bytes(O, K, T) == lib.nm_backward_input_workspace_bytes(O, K, T) > 0


# one and several tiles of 64 x 64 and larger, edges in both directions; rows of dX that are no whole pieces stay with the other kernel
@pytest.mark.gpu
@pytest.mark.parametrize("T,K,O", [(1, 64, 256), (63, 200, 320), (65, 264, 576), (197, 768, 768), (130, 1000, 1024), (1577, 384, 1152),
                                   (20, 100, 512)])
def test_input_gradient(T, K, O):
    rng = np.random.default_rng(T + K + O)
    dY, W = wl.draw_activations(rng, T, O), wl.draw_weights(rng, O, K)
    if K % 8 == 0:
        assert load_library().nm_backward_input_scratch_bytes(O, K, T) > 0
    mask = orc.nm_mask(W, 2, 4)
    Wm = torch.empty(O, K, dtype=torch.bfloat16, device="cuda")
    nm.nm_prune(dev_bf16(W), 2, 4, W_masked=Wm)
    dYd = dev_bf16(dY)
    dXref, _, B, _ = orc.nm_linear_backward(dY, np.zeros((T, K), np.uint16), W, mask)
    for dt in (torch.float32, torch.bfloat16):
        out = torch.full((T + 1, K + 8), 7.0, dtype=dt, device="cuda")
        y = nm.nm_linear_backward_input(Wm, dYd, out=out[:T, :K])
        plain = nm.nm_linear_backward_input(Wm, dYd, out_dtype=dt, workspace=torch.empty(8, dtype=torch.uint8, device="cuda"))
        assert bool((out[T] == 7).all() and (out[:, K:] == 7).all())
        if K % 8 == 0:
            assert torch.equal(y, plain)
        check_output(host_output(y.contiguous()), dXref, B, O, dt == torch.float32, (T, K, O, dt))

