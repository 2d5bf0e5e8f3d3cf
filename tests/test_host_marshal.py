"""Without the native half of binding.py, or with one of another torch: what loads, and what says how to build it."""
import subprocess
import sys

import pytest

from paper_2511_04283_amd import binding as B
from paper_2511_04283_amd import build


def test_module_imports_without_its_native_half():
    """As without the library: structures and cameras are there, the first call that needs it names the command."""
    code = """
import sys
sys.modules["paper_2511_04283_amd._marshal"] = None   # (an import finds nothing)
from paper_2511_04283_amd import binding as B, scenes
assert B.make_camera(scenes.Camera(16, 16, 8.0, 8.0, 8.0, 8.0)).width == 16
for call in (B.load_library, lambda: B._addresses(B.fs_gaussians(), 0, (), (), ())):
    try:
        call()
    except RuntimeError as e:
        assert "paper_2511_04283_amd.build" in str(e), e
    else:
        raise SystemExit("loaded")
"""
    subprocess.run([sys.executable, "-c", code], check=True, cwd=build.ROOT)


def test_the_one_of_another_torch_is_built_again(monkeypatch):
    assert B.load_marshal().stamp == build.marshal_stamp()
    monkeypatch.setattr(build, "marshal_stamp", lambda: "built against torch 0.0.0")
    monkeypatch.setattr(B, "_marshal", None)
    assert build.is_stale()
    with pytest.raises(RuntimeError, match="paper_2511_04283_amd.build"):
        B.load_marshal()
