"""The library works where _marshal.so is not there or does not load (another Python, no host compiler,
no headers): the ctypes path is complete."""
import os

import pytest
import torch

import paper_2504_19925_amd as symi
from paper_2504_19925_amd import binding, build


@pytest.mark.parametrize("what", ["absent", "unloadable"])
def test_calls_go_through_ctypes(what, tmp_path, monkeypatch):
    cfg = symi.SymiCfg.make(64, 8, 2, 128, 256, 16, 4, 0, "f32")
    monkeypatch.setenv("SYMI_LIB", symi.lib_path())
    monkeypatch.setattr(binding, "_HERE", str(tmp_path))
    monkeypatch.setattr(binding, "_LIB", None)
    monkeypatch.setattr(binding, "_marshal", {})
    if what == "unloadable":
        (tmp_path / "_marshal.so").write_bytes(b"of another machine")
        with pytest.warns(UserWarning, match="ctypes"):
            symi.lib()
    assert symi.symi_validate(cfg) == 0 and symi.symi_workspace_bytes(cfg) > 0
    assert binding._marshal == {}
    z = torch.zeros(64, 8)
    with pytest.raises(symi.SymiError, match="logits: expected a GPU tensor"):
        symi.symi_route(symi.SymiCtx(None, cfg, 0), z, z, z, z)


def test_build_goes_on_without_a_host_compiler(tmp_path, monkeypatch):
    old = tmp_path / "_marshal.so"
    old.write_bytes(b"an older one")
    monkeypatch.setattr(build, "MARSHAL_LIB", str(old))
    monkeypatch.setenv("CXX", str(tmp_path / "no-such-compiler"))
    assert build.build_marshal(verbose=False) is False
    assert not os.path.exists(old)
