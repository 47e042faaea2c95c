"""The build's own checks: a library or marshalling module that is missing, or older
than a source, is not up to date; an import without the marshalling module says so."""
import os
import subprocess
import sys

import pytest

from paper_2604_11947_amd import build as B

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_up_to_date_knows_the_marshalling_module(tmp_path, monkeypatch):
    files = {k: tmp_path / k for k in ("lib.so", "marshal.so", "a.hip", "marshal.cpp")}
    for f in files.values():
        f.write_text("x")
        os.utime(f, (1000, 1000))
    monkeypatch.setattr(B, "lib_path", lambda variant="bf16": str(files["lib.so"]))
    monkeypatch.setattr(B, "MARSHAL", str(files["marshal.so"]))
    monkeypatch.setattr(B, "SRC_MARSHAL", str(files["marshal.cpp"]))
    monkeypatch.setattr(B, "DEPS", [str(files["a.hip"])])
    assert B.up_to_date()
    for src in ("a.hip", "marshal.cpp"):
        os.utime(files[src], (2000, 2000))
        assert not B.up_to_date(), src
        os.utime(files[src], (1000, 1000))
    files["marshal.so"].unlink()
    assert not B.up_to_date()


@pytest.mark.parametrize("blocked", [False, True])
def test_import_without_the_marshalling_module_warns(blocked):
    code = "import sys; m = 'paper_2604_11947_amd'; "
    code += "sys.modules[m + '._marshal'] = None; " if blocked else ""
    code += "import paper_2604_11947_amd.resbm as R; assert (R._marshal is None) == " + str(blocked)
    p = subprocess.run([sys.executable, "-c", code], cwd=ROOT, capture_output=True, text=True)
    assert p.returncode == 0, p.stderr
    assert ("native argument marshalling not loaded" in p.stderr) == blocked
