"""The binding's native call path is optional (CPU): without it the package imports and
its calls go through the Python checks; without torch the build ends with the library."""
import importlib.util
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PACKAGE = os.path.join(ROOT, "paper_2609_04105_amd")

WITHOUT_BINDING = """
import sys, warnings
sys.modules["paper_2609_04105_amd._binding"] = None   # import raises ImportError
with warnings.catch_warnings(record=True) as seen:
    warnings.simplefilter("always")
    import paper_2609_04105_amd as fa
assert any(w.category is RuntimeWarning and "_binding" in str(w.message) for w in seen), seen
import torch
x = torch.zeros(1, 1, 128, 64)
for call in (lambda: fa.quantize_qkv(x, x, x), lambda: fa.attention_mxfp4(x, x, x), lambda: fa.forward_bf16(x, x, x),
             lambda: fa.forward_mxfp4(*[x] * 6)):
    try:
        call()
    except ValueError as e:
        assert "must be a GPU tensor" in str(e), e
    else:
        raise AssertionError("a CPU tensor was accepted")
"""


def test_package_works_without_the_native_call_path():
    run = subprocess.run([sys.executable, "-c", WITHOUT_BINDING], cwd=ROOT, capture_output=True, text=True, timeout=300)
    assert run.returncode == 0, run.stderr


@pytest.mark.parametrize("torch_spec", ["absent", "no headers"])
def test_build_without_torch_leaves_the_binding_out(tmp_path, monkeypatch, torch_spec):
    spec = importlib.util.spec_from_file_location("_fp4attn_build_test", os.path.join(PACKAGE, "build.py"))
    build = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(build)
    stale = tmp_path / "_binding.so"
    stale.write_bytes(b"")
    monkeypatch.setattr(build, "BINDING", str(stale))
    found = None
    if torch_spec == "no headers":
        found = importlib.util.spec_from_loader("torch", None, is_package=True)
        found.submodule_search_locations = [str(tmp_path)]
    monkeypatch.setattr(build.importlib.util, "find_spec", lambda name: found)
    assert build._build_binding() is False
    assert not stale.exists()
