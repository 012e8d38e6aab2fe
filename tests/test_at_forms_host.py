"""The arithmetic behind the Axilrod-Teller matrix form, on the host: the linear
forms split tr(ABC) exactly, and the block order is a bijection."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.skipif(shutil.which("g++") is None, reason="no host C++ compiler")
def test_forms_and_block_order(tmp_path):
    exe = str(tmp_path / "check_at_forms")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-I", os.path.join(ROOT, "paper_1610_07394_amd", "csrc"),
                           "-o", exe, os.path.join(ROOT, "tests", "host", "check_at_forms.cpp")])
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and r.stdout.strip() == "ok", r.stdout
