"""The build without a host compiler or without torch's headers (no compilation
is run): the library does not need either."""
import os
import shutil

import pytest

from paper_2608_10805_amd import build


@pytest.mark.parametrize("missing", ["g++", "headers"])
def test_the_library_builds_without_the_wrapper_s_toolchain(missing, monkeypatch, tmp_path, capsys):
    compiled, stale = [], tmp_path / "_wtconv_torch.so"
    stale.write_text("")
    monkeypatch.setattr(build, "TORCH_LIB", str(stale))
    monkeypatch.setattr(build, "_compile", lambda sources, lib, extra, verbose: compiled.append(lib))
    monkeypatch.setattr(build.subprocess, "run", lambda *a, **k: pytest.fail("nothing else may be compiled"))
    if missing == "g++":
        monkeypatch.setattr(shutil, "which", lambda name: None)
    else:
        exists = os.path.exists
        monkeypatch.setattr(os.path, "exists", lambda p: exists(p) and not str(p).endswith("extension.h"))
    assert build.build() == build.LIB
    assert compiled == [build.LIB, build.PROBE_LIB]
    assert not stale.exists()
    assert "left out" in capsys.readouterr().out
