"""The binding's native calls are an addition: a package without them, or with those of another torch, loads and goes through ctypes."""
import os
import shutil
import subprocess
import sys

import paper_1911_02150_amd.binding as binding


def test_package_without_native_calls(tmp_path):
    """What build_library() alone makes."""
    package = os.path.dirname(binding.__file__)
    shutil.copytree(package, tmp_path / "paper_1911_02150_amd", ignore=shutil.ignore_patterns("_calls*", "csrc", "__pycache__"))
    code = ("import paper_1911_02150_amd.binding as b, os; b.load_library(); "
            f"assert os.path.dirname(b.__file__) == {str(tmp_path / 'paper_1911_02150_amd')!r}; assert b._native is None; print(b.status_string(2))")
    done = subprocess.run([sys.executable, "-c", code], cwd=tmp_path, capture_output=True, text=True, timeout=300)
    assert done.returncode == 0 and done.stdout.strip(), done.stderr


def test_native_calls_of_another_torch(monkeypatch):
    lib = binding.load_library()
    assert binding._load_native(lib) is not None
    monkeypatch.setattr(binding.torch, "__version__", "0.0")
    assert binding._load_native(lib) is None
