"""The build of the native marshalling beside the library, and what is loaded of it."""
import sysconfig

import pytest
import torch

from paper_2409_09708_amd import binding


@pytest.mark.parametrize("module,name,value", [(torch, "__version__", "1.0.0"),
                                               (sysconfig, "get_config_var", lambda name: "cpython-30-other")])
def test_calls_built_for_another_torch_or_python_are_not_loaded(monkeypatch, module, name, value):
    binding._native()
    monkeypatch.setattr(binding, "_CALLS", None)
    monkeypatch.setattr(module, name, value)
    with pytest.raises(RuntimeError, match="build it"):
        binding._native()
    assert binding._CALLS is None
