"""Paths that open but are no model file are errors of the call, not of the process: a directory, an
empty file, a file shorter than its header."""
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.parametrize("what", ["directory", "empty", "short"])
def test_no_model_file(tmp_path, what):
    path = tmp_path / "model.bin"
    if what == "directory":
        path.mkdir()
    else:
        path.write_bytes(b"" if what == "empty" else b"DPAMDv01" + bytes(100))
    code = ("from paper_2602_02234_amd import load\n"
            "for prec in (0, 1):\n"
            "    assert load().dp_check_model_file(%r, prec, None, None) == -2\n" % str(path).encode())
    r = subprocess.run([sys.executable, "-c", code], cwd=ROOT, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-500:]


@pytest.mark.gpu
def test_directory_is_no_message_passing_model(tmp_path):
    from paper_2602_02234_amd import DPError, GnnModel, RepModel
    for load in (GnnModel, RepModel):
        with pytest.raises(DPError, match="DP_ERR_MODEL_FILE"):
            load(str(tmp_path))
