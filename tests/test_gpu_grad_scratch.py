"""dW of a short reduction: no scratch where nothing is written to it."""
import pytest
import torch

import paper_2409_09708_amd as nm
from paper_2409_09708_amd import binding
from test_gpu_calls import in_python

# one launch, whose sums stay on the chip: (T, K, O)
SHORT = [(197, 768, 2304), (394, 1024, 4096), (788, 768, 3072), (1576, 768, 2304), (20, 64, 64)]
LONG = [(394, 256, 256), (3152, 768, 2304), (50432, 768, 768)]


def test_scratch_is_what_the_kernels_use():
    lib = binding.load_library()
    for T, K, O in SHORT:
        assert lib.nm_backward_weight_scratch_bytes(O, K, T) == 0 < lib.nm_backward_weight_workspace_bytes(O, K, T)
    for T, K, O in LONG:
        assert lib.nm_backward_weight_scratch_bytes(O, K, T) == lib.nm_backward_weight_workspace_bytes(O, K, T) > 0
        call = lambda ws, size: lib.nm_linear_backward_weight_scratch(4096, T, O, O, 4096, K, K, None, 4096, K, 0, ws, size, None)
        need = lib.nm_backward_weight_scratch_bytes(O, K, T)
        assert call(None, 0) == 6 and call(4096, need - 1) == 6 and call(4096 + 16, need) == 6
    assert lib.nm_backward_weight_scratch_bytes(0, 64, 16) == 0 and lib.nm_backward_weight_scratch_bytes(30, 64, 100) == 0
    assert lib.nm_linear_backward_weight_scratch(None, 16, 64, 64, 4096, 64, 64, None, 4096, 64, 0, None, 0, None) == 1


@pytest.mark.gpu
@pytest.mark.parametrize("T,K,O", SHORT + LONG[:1])
def test_calls_without_scratch(monkeypatch, T, K, O):
    g = torch.Generator(device="cuda")
    g.manual_seed(T + O)
    X, dY = (torch.empty(T, n, dtype=torch.bfloat16, device="cuda").normal_(generator=g) for n in (K, O))
    ws = torch.empty(nm.nm_backward_weight_workspace_bytes(O, K, T), dtype=torch.uint8, device="cuda")
    want = nm.nm_linear_backward_weight(dY, X, workspace=ws)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    for run in (lambda call: call(), lambda call: in_python(monkeypatch, call)):
        for key in [k for k in binding._WORKSPACES if k[2] == side.cuda_stream]:
            del binding._WORKSPACES[key]
        got = run(lambda: nm.nm_linear_backward_weight(dY, X, stream=side))
        side.synchronize()
        assert torch.equal(got, want)
        assert any(k[2] == side.cuda_stream for k in binding._WORKSPACES) == ((T, K, O) in LONG)
