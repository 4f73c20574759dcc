"""The library and the extension of its calls are put in place together or not at all."""
import shutil
import subprocess

import pytest

from paper_1805_12549_amd import build


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="needs hipcc")
def test_nothing_is_replaced_where_the_extension_does_not_build(tmp_path, monkeypatch):
    monkeypatch.setattr(build, "SOURCES", ["kernels_counts.hip"])
    monkeypatch.setattr(build, "calls_command", lambda *_: ["false"])
    for name in ("LIB", "CALLS"):
        path = tmp_path / getattr(build, name).name
        path.write_bytes(b"of the build before")
        monkeypatch.setattr(build, name, path)
    with pytest.raises(subprocess.CalledProcessError):
        build.build()
    assert sorted(p.name for p in tmp_path.iterdir()) == ["_calls.so", "libcg_conv.so"]
    assert all(p.read_bytes() == b"of the build before" for p in tmp_path.iterdir())
