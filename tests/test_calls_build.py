"""The build of the native marshalling beside the library, and what is loaded of it."""
import subprocess
import sysconfig

import pytest
import torch

from paper_2409_09708_amd import binding
from paper_2409_09708_amd import build as nm_build


@pytest.mark.parametrize("module,name,value", [(torch, "__version__", "1.0.0"),
                                               (sysconfig, "get_config_var", lambda name: "cpython-30-other")])
def test_calls_built_for_another_torch_or_python_are_not_loaded(monkeypatch, module, name, value):
    binding._native()
    monkeypatch.setattr(binding, "_CALLS", None)
    monkeypatch.setattr(module, name, value)
    with pytest.raises(RuntimeError, match="build it"):
        binding._native()
    assert binding._CALLS is None


def test_library_is_linked_where_the_marshalling_cannot_be_built(monkeypatch, tmp_path):
    def run(cmd, **kw):  # the compilers, but for the one that fails
        if "nm_calls.cpp" in " ".join(cmd):
            return subprocess.CompletedProcess(cmd, 1, "", "no torch headers")
        open(cmd[cmd.index("-o") + 1], "w").close()
        return subprocess.CompletedProcess(cmd, 0, "", "")

    monkeypatch.setattr(nm_build.subprocess, "run", run)
    monkeypatch.setattr(nm_build, "PKG_DIR", str(tmp_path))
    monkeypatch.setattr(nm_build, "LIB_PATH", str(tmp_path / "lib.so"))
    with pytest.raises(RuntimeError, match="no torch headers"):
        nm_build.build_library()
    assert (tmp_path / "lib.so").exists()


def test_rocm_headers_are_those_of_the_compiler_found(monkeypatch, tmp_path):
    seen = []
    monkeypatch.setattr(nm_build, "hipcc", lambda: str(tmp_path / "rocm" / "bin" / "hipcc"))
    monkeypatch.setattr(nm_build.subprocess, "run", lambda cmd, **kw: seen.extend(cmd) or subprocess.CompletedProcess(cmd, 1, "", ""))
    with pytest.raises(RuntimeError):
        nm_build.compile_calls("nm_calls.cpp", str(tmp_path / "calls.so"))
    assert f"-I{tmp_path}/rocm/include" in seen and "-I/opt/rocm/include" not in seen
