"""The package with and without the extension of its calls (csrc/py_calls.cpp): missing or built for another torch it is left out, with a warning, and ctypes serves alone."""
import shutil
import subprocess
import sys
from pathlib import Path

import pytest

PKG = Path(__file__).resolve().parent.parent / "paper_1805_12549_amd"

CHECK = """
import sys, warnings
import torch
if {other}:
    torch.__version__ = "0.0.1"
with warnings.catch_warnings(record=True) as said:
    warnings.simplefilter("always")
    from {package} import binding as B
said = [str(w.message) for w in said if "_calls.so" in str(w.message)]
print(B._calls is not None, len(said), B.cg_last_error() is not None, *said)
"""


@pytest.mark.skipif(not (PKG / "libcg_conv.so").exists() or not (PKG / "_calls.so").exists(), reason="needs the built library")
@pytest.mark.parametrize("case,starts", [("whole", "True 0 True"), ("missing", "False 1 True"), ("other_torch", "False 1 True"), ("broken", "False 1 True")])
def test_import(tmp_path, case, starts):
    copy = tmp_path / PKG.name
    copy.mkdir()
    for f in ("__init__.py", "binding.py", "libcg_conv.so", "_calls.so"):
        shutil.copy(PKG / f, copy / f)
    if case == "missing":
        (copy / "_calls.so").unlink()
    elif case == "broken":
        (copy / "_calls.so").write_bytes(b"not a library")
    r = subprocess.run([sys.executable, "-c", CHECK.format(other=case == "other_torch", package=PKG.name)], cwd=tmp_path, capture_output=True, text=True,
                       timeout=300)
    assert r.returncode == 0 and r.stdout.startswith(starts), (r.stdout, r.stderr[-2000:])


@pytest.mark.skipif(not (PKG / "libcg_conv.so").exists() or not (PKG / "_calls.so").exists(), reason="needs the built library")
def test_forward_takes_a_layer_only():
    """(an object of another type was read as a layer)"""
    from paper_1805_12549_amd import binding as B
    for other in (None, 0, object(), "layer"):
        with pytest.raises(TypeError, match="Layer"):
            B._calls.forward(other, None, None, None, None, False, False)
