"""The scratch tensor that a stream's calls share: one that is replaced stays out of the allocator's hands until its stream is done with
it, also where that is the default stream and the tensor was allocated while another one was current."""
import types

import pytest

from paper_2409_09708_amd import binding


@pytest.mark.parametrize("handle", [0, 0x5000])
def test_a_replaced_tensor_is_in_use_on_its_stream(monkeypatch, handle):
    marked = []

    class Tensor:
        def __init__(self, size):
            self.size = size

        def numel(self):
            return self.size

        def record_stream(self, stream):
            marked.append((self, stream))

    cuda = types.SimpleNamespace(current_device=lambda: 0, ExternalStream=lambda h, device: ("external", h, device),
                                 default_stream=lambda device: ("default", 0, device))
    torch = types.SimpleNamespace(cuda=cuda, uint8=None, empty=lambda shape, dtype, device: Tensor(shape[0]))
    for name, value in (("_torch", lambda: torch), ("_stream_handle", lambda stream: handle), ("_WORKSPACES", {})):
        monkeypatch.setattr(binding, name, value)
    device = types.SimpleNamespace(type="cuda", index=0)
    first = binding._workspace(100, device)
    assert binding._workspace(1 << 20, device) is first and marked == []
    assert binding._workspace(1 << 21, device) is not first
    assert marked == [(first, ("external", handle, 0) if handle else ("default", 0, 0))]
